// Full-vocabulary support: steps 1 and 2 of the verifier (Sec. 5.1 ratio order and prefix psi, Sec. 6
// H*, alpha*, outer residuals of Thm 6.2, records, truncation sets of Alg. 1) for a draft distribution
// without top-k or with a top-k above GR_MAX_SUPPORT, where the support (up to V tokens) does not fit LDS.
//
// Every per-token array lives in a per-handle HBM workspace, row-major with stride V + 2; one
// workgroup works through a row (256 threads; 512 or 1024 on long rows), but where a row's slices, buckets or chunks are shared out.  The
// arithmetic that decides integers (prefix sums, F, the running masses of the truncation sets) is the same sequential fp64 arithmetic as on the
// LDS-resident path.
#include <algorithm>
#include <type_traits>

#include "gr_internal.h"

namespace gr {

namespace {

constexpr int kScanThreads = 512;                  // of the kernel that takes the prefix sums
constexpr int kChunkRanks = 4096;                  // ranks per workgroup of the kernel that scatters by token id ...
constexpr int kChunkLds = 40 * 1024;               // ... and the LDS that a workgroup of 256 threads reserves, for four of them to a compute unit: the rows that are in
                                                   // work at a time then stay in their XCD's L2
// The sort by q of a support's candidates and of the truncation sets: elements of 8 bytes, the key in the high bits and the token id in the low ones.
template <int NT, int R = 4>
struct Sort32Lds {
    static constexpr int kWavesNT = NT / 64;
    static constexpr int kItems = R;               // elements per thread and tile
    static constexpr int kTile = NT * kItems;
    unsigned long long tile[kTile];                // the tile in digit order
    unsigned long long wcnt[kWavesNT][64];         // per wave: 256 counters of 16 bits, four to a word
    int hist[4][256];
    int start[256];                                // first place of each digit in the tile
    int dest[256];                                 // output slot of the tile's place 0, per digit
    int skip[4];
};

// Stable least-significant-digit radix sort of one row's `count` elements by their bits from `lo` on, 8 bits per pass and
// at most four passes, between a and b; returns the buffer that holds the result.  A pass moves tiles of kTile elements: every wave ranks 64 kItems
// consecutive ones among themselves (ballots, and counters that are its own, so no barrier lies between its
// rounds), wave 0 turns the counters into places, and the tile goes through LDS into digit order, so that the
// elements of one digit leave as one run and not one by one.  Three barriers per tile.
// A run is 128 bytes on average with four elements per thread and 1024 threads, 256 bytes with eight (see kLongRow).
// Bound: 16 bytes of traffic per element and pass, and the latency of a tile's three barriers (1024 rows of 128256
// tokens, four passes: 18 GB in 5.3 ms, 3.4 TB/s where a device copy reaches 5.2).  All threads call.
template <int NT, int R>
__device__ unsigned long long* block_sort32(unsigned long long* a, unsigned long long* b, int count, Sort32Lds<NT, R>& S, int lo = 32,
                                           int passes = 4) {
    constexpr int kTile = Sort32Lds<NT, R>::kTile;
    constexpr int kSortItems = R, NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int c = tid; c < 4 * 256; c += NT) (&S.hist[0][0])[c] = 0;
    if (tid < 4) S.skip[tid] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < count; i0 += 4 * NT) {
        unsigned keys[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { const int i = i0 + u * NT + tid; keys[u] = i < count ? static_cast<unsigned>(a[i] >> lo) : 0u; }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool valid = i0 + u * NT + tid < count;
            const unsigned key = keys[u];
            const unsigned long long vm = __ballot(valid);
            if (vm == 0ull) continue;                           // wave-uniform; lane 0 is valid otherwise
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= passes) break;
                const int d = static_cast<int>((key >> (8 * j)) & 255u);
                const int d0 = __builtin_amdgcn_readfirstlane(d);
                if (__ballot(valid && d == d0) == vm) {         // one digit in the whole wave: one update
                    if (lane == 0) atomicAdd(&S.hist[j][d0], __popcll(vm));
                } else if (valid) {
                    atomicAdd(&S.hist[j][d], 1);
                }
            }
        }
    }
    __syncthreads();
    for (int c = tid; c < 4 * 256; c += NT) if ((&S.hist[0][0])[c] == count) S.skip[c >> 8] = 1;
    __syncthreads();

    for (int pass = 0; pass < passes; ++pass) {
        if (S.skip[pass]) continue;
        const int shift = lo + 8 * pass;
        int next[4] = {0, 0, 0, 0};                             // wave 0: next output slot of digits 4 lane .. 4 lane + 3
        if (wv == 0) {
            int tot = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { next[j] = tot; tot += S.hist[pass][4 * lane + j]; }
            const int incl = wave_scan_i(tot);
#pragma unroll
            for (int j = 0; j < 4; ++j) next[j] += incl - tot;
        }
        unsigned short* mycnt = reinterpret_cast<unsigned short*>(&S.wcnt[wv][0]);
        unsigned long long en[kSortItems];
#pragma unroll
        for (int j = 0; j < kSortItems; ++j) {
            const int i = wv * 64 * kSortItems + j * 64 + lane;
            en[j] = i < count ? a[i] : 0ull;
        }
        for (int t0 = 0; t0 < count; t0 += kTile) {
            unsigned long long e[kSortItems]; int rank[kSortItems];
            const int first = t0 + wv * 64 * kSortItems + lane;
#pragma unroll
            for (int j = 0; j < kSortItems; ++j) {
                e[j] = en[j];
                const int i = first + kTile + j * 64;
                en[j] = i < count ? a[i] : 0ull;
            }
            S.wcnt[wv][lane] = 0ull;                            // read last before the barrier that ended the previous tile's second phase
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < kSortItems; ++j) {
                const bool valid = first + j * 64 < count;
                const int d = static_cast<int>((e[j] >> shift) & 255ull);
                unsigned long long peers = __ballot(valid);     // lanes of this wave that hold the same digit
#pragma unroll
                for (int bb = 0; bb < 8; ++bb) {
                    const bool bit = (d >> bb) & 1;
                    const unsigned long long m = __ballot(valid && bit);
                    peers &= bit ? m : ~m;
                }
                const int before = mycnt[d];
                const int below = __popcll(peers & ((1ull << lane) - 1ull));
                rank[j] = before + below;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
                if (valid && below == 0) mycnt[d] = static_cast<unsigned short>(before + __popcll(peers));
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            if (wv == 0) {
                // four digits per lane: the waves' counts become offsets (16-bit fields: a tile holds at most 8192)
                unsigned long long run = 0ull;
#pragma unroll 4
                for (int w = 0; w < NW; ++w) { const unsigned long long c = S.wcnt[w][lane]; S.wcnt[w][lane] = run; run += c; }
                int c[4]; int tot = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) { c[j] = static_cast<int>((run >> (16 * j)) & 0xFFFFull); tot += c[j]; }
                int at = wave_scan_i(tot) - tot;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    S.start[4 * lane + j] = at; S.dest[4 * lane + j] = next[j] - at;
                    at += c[j]; next[j] += c[j];
                }
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < kSortItems; ++j) {
                if (first + j * 64 < count) {
                    const int d = static_cast<int>((e[j] >> shift) & 255ull);
                    S.tile[S.start[d] + mycnt[d] + rank[j]] = e[j];
                }
            }
            __syncthreads();
            const int cnt = min(kTile, count - t0);
#pragma unroll
            for (int j = 0; j < kSortItems; ++j) {
                const int i = j * NT + tid;
                if (i < cnt) { const unsigned long long x = S.tile[i]; b[S.dest[static_cast<int>((x >> shift) & 255ull)] + i] = x; }
            }
        }
        __syncthreads();
        unsigned long long* t = a; a = b; b = t;
    }
    return a;
}
__device__ __forceinline__ unsigned long long pack32(unsigned key, int id) {
    return (static_cast<unsigned long long>(key) << 32) | static_cast<unsigned>(id);
}
__device__ __forceinline__ int packed_id(unsigned long long e) { return static_cast<int>(static_cast<unsigned>(e)); }

// wtot: LDS, the counts of the workgroup's 4 NW groups of 64 tokens in token order (NW <= 16: one per lane).  offs[j] = the
// count before this wave's group of round j; returns the count of all groups.  (A loop over the groups in every thread
// cost a row of 8193 tokens cut to 9 36 of its 100 us in a workgroup of 16 waves.)
template <int NW>
__device__ __forceinline__ int group_offsets(const int* wtot, int (&offs)[4]) {
    static_assert(4 * NW <= 64, "one group per lane");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int v = lane < 4 * NW ? wtot[lane] : 0;
    const int incl = wave_scan_i(v);
#pragma unroll
    for (int j = 0; j < 4; ++j) offs[j] = __shfl(incl - v, j * NW + wv);
    return __builtin_amdgcn_readlane(incl, 4 * NW - 1);
}

// chist[4096]: members per magnitude class of a positive float (its bit pattern >> 19: exponent and four mantissa
// bits; every member lies below the class's upper edge, so count x edge bounds the class's mass).  Classes are
// dropped from the bottom while that bound stays within `budget`; returns the lowest class that stays (0 when every
// class would fit: nothing is dropped then).  dscan: LDS double[kThreads], bsel: LDS int.  All threads
// call; the first kThreads of them own the classes.
__device__ int class_threshold(const int* chist, double budget, double* dscan, int* bsel) {
    const int tid = threadIdx.x;
    // thread t owns classes 16 t .. 16 t + 15; prefix of the bounds over the threads, serially by thread 0
    double local = 0.0;
    if (tid < kThreads) {
        for (int c = 16 * tid; c < 16 * tid + 16; ++c)
            local += static_cast<double>(chist[c]) * static_cast<double>(__uint_as_float((static_cast<unsigned>(c) + 1u) << 19));
        dscan[tid] = local;
    }
    if (tid == 0) *bsel = 4096;
    __syncthreads();
    if (tid == 0) {
        double run = 0.0;
#pragma unroll 32
        for (int t = 0; t < kThreads; ++t) { const double v = dscan[t]; dscan[t] = run; run += v; }
    }
    __syncthreads();
    if (tid < kThreads) {
        double run = dscan[tid];                                 // bound on the mass of all classes below 16 tid
        for (int c = 16 * tid; c < 16 * tid + 16; ++c) {
            run += static_cast<double>(chist[c]) * static_cast<double>(__uint_as_float((static_cast<unsigned>(c) + 1u) << 19));
            if (run > budget) { atomicMin(bsel, c); break; }     // class c cannot be dropped whole
        }
    }
    __syncthreads();
    const int b = *bsel;
    __syncthreads();
    return b == 4096 ? 0 : b;
}

// The lowest class c (4096: none) with enough(mass of the classes below it), the mass bounded from below: count x lower edge.
template <class F>
__device__ int definite_class(const int* chist, F enough, double* dscan, int* bsel) {
    const int tid = threadIdx.x;
    auto least = [&](int c) { return static_cast<double>(chist[c]) * static_cast<double>(__uint_as_float(static_cast<unsigned>(c) << 19)); };
    if (tid < kThreads) {
        double local = 0.0;
        for (int c = 16 * tid; c < 16 * tid + 16; ++c) local += least(c);
        dscan[tid] = local;
    }
    if (tid == 0) *bsel = 4096;
    __syncthreads();
    if (tid == 0) {
        double run = 0.0;
#pragma unroll 32
        for (int t = 0; t < kThreads; ++t) { const double v = dscan[t]; dscan[t] = run; run += v; }
    }
    __syncthreads();
    if (tid < kThreads) {
        double run = dscan[tid];
        for (int c = 16 * tid; c < 16 * tid + 16; ++c) {
            if (enough(run)) { atomicMin(bsel, c); break; }
            run += least(c);
        }
    }
    __syncthreads();
    const int b = *bsel;
    __syncthreads();
    return b;
}

__device__ void mark_bad(const FullParams& fp, int row, double ptot, double qtot) {
    RowInfo info;
    info.support = 0; info.h = 0; info.status = GR_ROW_BAD; info.iterations = 0;
    info.alpha_star = __longlong_as_double(0x7ff8000000000000ll);
    info.res_total = 0.0; info.p_total = ptot; info.q_total = qtot; info.node_tokens = 0.0; info.p_ref = 0.0; info.inv_temp = 0.0; info.q_ref = 0.0;
    fp.info[row] = info;
    fp.accept_prob[row] = __uint_as_float(0x7fc00000u);
    fp.status[row] = GR_ROW_BAD;
}

// Workgroups of a kernel that goes through all rows in chunks of kChunkRanks ranks: a launch of chunk_grid() workgroups of one dimension.  A chunk
// reads or writes by token id, anywhere in its row's arrays, so the chunks of a row should share an L2: with eight rows or more to each XCD
// (workgroups go round the XCDs) a row's chunks stay on one.
__host__ __device__ inline bool rows_to_xcds(int B) { return B >= 64; }
inline unsigned chunk_grid(int B, int chunks) { return static_cast<unsigned>(rows_to_xcds(B) ? (B + 7) / 8 * 8 : B) * static_cast<unsigned>(chunks); }
__device__ __forceinline__ void chunk_of(int B, int chunks, int& row, int& chunk) {
    const unsigned g = blockIdx.x;
    if (rows_to_xcds(B)) { row = static_cast<int>((g >> 3) / chunks * 8 + (g & 7u)); chunk = static_cast<int>((g >> 3) % chunks); }
    else { row = static_cast<int>(g / chunks); chunk = static_cast<int>(g % chunks); }
}

// The order's key of a token: rising keys are falling ratios, ties go by the token id.  Rows given as probabilities: the correctly rounded quotient
// (p = 0 gives an infinity: first); as logits: q/p is proportional to exp((d - t) / T), so d - t (exact in float64; a masked target gives +inf).
struct RatioKey {
    bool lg; double inv_temp, inv_temp_q;
    __device__ __forceinline__ unsigned long long operator()(float qv, float pv) const {
        const double ratio = lg ? logit_ratio_key(static_cast<double>(qv), static_cast<double>(pv), inv_temp_q, inv_temp)
                                : static_cast<double>(qv) / static_cast<double>(pv);
        return lg ? ~mono64(ratio) : ~static_cast<unsigned long long>(__double_as_longlong(ratio));
    }
};
// Buckets of the order: kBucket tokens on average at most (while there are buckets enough), kBucketCap in the LDS of the workgroup that sorts one.
// With kSamplesPerBucket samples to a bucket, four in a million are of twice the average.  Rows of more than 131072 tokens have 4096 samples for all their
// buckets, so that more of these end above the cap: one in 1500 at 262144 tokens, one in 24 at a million; at 4 million, with 2048 buckets for all, two of
// five, and beyond that most.  Those go by sorted stretches (one row of 2^18 / 2^20 / 2^22 / 2^24 - 1 tokens, the call: 1463 us, 4.1, 16.0 and 67 ms; with the
// tokens of a bucket compared all with all 2117 us, 5.4, 28 and 294 ms).
constexpr int kBucket = 1024, kBucketCap = 2048, kSamplesPerBucket = 32, kLogBuckets = 11;
__host__ __device__ inline int log_buckets(int tokens) {
    int l = 0;
    while (tokens > kBucketCap && l < kLogBuckets && (kBucket << l) < tokens) ++l;   // up to the cap one workgroup takes them whole
    return l;
}
// What the order's kernels hand on about a row's buckets, in arrays that later kernels fill.
constexpr int kMaxSlices = 32;
struct SplitView {
    unsigned long long* key; int* id;                            // the splitters
    unsigned short* bucket;                                      // of a token
    int* count;                                                  // [slices, buckets]
    int* first;                                                  // the first rank of each bucket, and of the end
    __device__ SplitView(const FullParams& fp, int row) {
        const size_t at = row * (static_cast<size_t>(fp.V) + 2);
        key = reinterpret_cast<unsigned long long*>(fp.rho + at); id = fp.blk + at;
        bucket = reinterpret_cast<unsigned short*>(fp.blo + at);
        count = reinterpret_cast<int*>(fp.weight + at); first = fp.val0 + at;
    }
};
static_assert((kMaxSlices + 1) * 2 * sizeof(int) <= kBucket * sizeof(double), "the counts of a row's slices lie in its weights");
template <int NT>
struct SplitLds {
    static constexpr int kLogBuckets = NT >= 1024 ? gr::kLogBuckets : 4;   // the small workgroup takes rows of up to 16384 tokens
    static constexpr int kSamples = NT >= 1024 ? 4096 : kSamplesPerBucket << kLogBuckets;
    unsigned long long key[kSamples];
    int id[kSamples];
};

// Sorts `size` (a power of two, at least 64) keys with their ids in LDS, by key and then id.  All threads call; barriers at both ends.
template <int NT>
__device__ void block_bitonic(unsigned long long* key, int* id, int size) {
    for (int k = 2; k <= size; k *= 2)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < size / 2; t += NT) {
                const int i = 2 * t - (t & (j - 1)), o = i + j;
                const unsigned long long a = key[i], b = key[o];
                const int ia = id[i], ib = id[o];
                const bool behind = a > b || (a == b && ia > ib);
                if (behind == ((i & k) == 0)) { key[i] = b; key[o] = a; id[i] = ib; id[o] = ia; }
            }
        }
    __syncthreads();
}
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
    auto least = [](unsigned long long a, int lo, int hi) { return min(a, (static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) | static_cast<unsigned>(lo)); };
    v = least(v, dpp_move<kDppXor1>(static_cast<int>(v)), dpp_move<kDppXor1>(static_cast<int>(v >> 32)));
    v = least(v, dpp_move<kDppXor2>(static_cast<int>(v)), dpp_move<kDppXor2>(static_cast<int>(v >> 32)));
    v = least(v, dpp_move<kDppHalfMirror>(static_cast<int>(v)), dpp_move<kDppHalfMirror>(static_cast<int>(v >> 32)));
    v = least(v, dpp_move<kDppMirror>(static_cast<int>(v)), dpp_move<kDppMirror>(static_cast<int>(v >> 32)));
    const int lo = static_cast<int>(v), hi = static_cast<int>(v >> 32);
    unsigned long long r = ~0ull;
#pragma unroll
    for (int l = 0; l < 64; l += 16) r = least(r, __builtin_amdgcn_readlane(lo, l), __builtin_amdgcn_readlane(hi, l));
    return r;
}

// What adding a run of terms one after the other does to a running sum, from its rounding alone.  While the sum stays in one
// binade it is a whole number of units u, and acc + x rounds to acc + r u with r depending on x and, where x lies halfway between
// two units, on whether acc / u is even.  So a run of terms is two sums (exact, both whole numbers of u) and the parity they
// leave, one for an even start and one for an odd one, and runs compose: sequential sums, bit for bit, by a scan.
struct RunSum { double d[2]; int par; };                       // par: bit s = the parity that a start of parity s ends with
__device__ __forceinline__ RunSum compose(const RunSum& a, const RunSum& b) {
    RunSum r;
    r.d[0] = a.d[0] + ((a.par & 1) ? b.d[1] : b.d[0]);
    r.d[1] = a.d[1] + ((a.par & 2) ? b.d[1] : b.d[0]);
    r.par = ((b.par >> (a.par & 1)) & 1) | (((b.par >> ((a.par >> 1) & 1)) & 1) << 1);
    return r;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_step(RunSum& v) {
    RunSum a;                                                  // a lane without a source: the empty run
    a.d[0] = dpp_shift<CTRL, ROWS>(v.d[0], 0.0); a.d[1] = dpp_shift<CTRL, ROWS>(v.d[1], 0.0); a.par = dpp_shift<CTRL, ROWS>(v.par, 2);
    v = compose(a, v);
}

}  // namespace

// ---- kernel 1: row sums and validity, the support (all positive entries of q, or the k largest) in
// token order where it is cut, the splitters of its order by decreasing q/p (ties by id).
// The key of the order is the correctly rounded float64 quotient q/p: for float32 inputs two different
// ratios differ by at least 2^-48 relative, so their quotients differ and keep their order, and equal
// ratios give equal quotients -- the same order as the exact cross-product comparison (Sec. 5.1).
//
// This kernel splits the support into buckets of some kBucket tokens by splitters, keys with their token ids from a sorted sample of the row (so
// that equal ratios can be split too); the next two kernels move the tokens there, and full_bucket_kernel puts each bucket in order.  The elements keep p and q
// beside the id: no kernel gathers them.  Where the support is sparse or cut, its list is sampled and not the row.
// Bound: memory, and the quotients.  1024 rows of 128256 tokens, n = 8: four sorting passes over elements of 8 bytes by one workgroup per row and a
// gather of the pairs took 6.1 + 1.6 ms; support 0.44, count 0.72, scatter 0.78 and buckets 1.5 ms take their place.  One row 1555 -> 748 us the call,
// 16 rows 2412 -> 1485, 64 rows cut by a nucleus of 32000 tokens 314 -> 274; 64 rows whose draft logits are the target's but for noise of 1e-2 / 1e-4 / 1e-6
// 1902 / 1899 / 2112 -> 1053 / 1145 / 1330 (ratios that are few or close crowd in their buckets' cells and go by the bitonic sort).
template <int NT, bool CUT, int R = 4>
__global__ __launch_bounds__(NT, CUT ? 1 : 8) void full_support_kernel(FullParams fp) {
    constexpr int kWaves = NT / 64;                              // this workgroup's waves
    constexpr int kThreads = NT;
    __shared__ union { std::conditional_t<CUT, Sort32Lds<NT, R>, char> sort; SplitLds<NT> split; } lds;
    auto& S = lds.sort;
    __shared__ double red[kWaves];
    __shared__ int wtot[4 * kWaves];
    __shared__ double dscan[gr::kThreads];
    __shared__ int bsel;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int V = fp.V;
    const size_t vs = static_cast<size_t>(V) + 2;
    const float* pr = fp.p + static_cast<size_t>(row) * V;
    const float* qr = fp.q + static_cast<size_t>(row) * V;
    unsigned long long* k0 = fp.key0 + row * vs; unsigned long long* k1 = fp.key1 + row * vs;
    const bool lg = fp.logits != 0;
    const bool cut = CUT && fp.tail_mass > 0.0;
    int positive = 0;                                            // tokens that the draft may take
    double ptot, qtot;
    double p_ref = 0.0, q_ref = 0.0, inv_temp = 0.0, inv_temp_q = 0.0;
    if (fp.logits) {
        // rows given as logits: the largest target and draft logit, then the target's softmax sum relative to it;
        // q needs no sum (it is renormalised over the support).  A NaN or +inf anywhere, or a temperature that is not
        // positive and finite, marks the row bad; -inf is a masked token.
        const float T = fp.temperature[row];
        const float Td = fp.draft_temperature ? fp.draft_temperature[row] : T;
        float tm = -__builtin_inff(), dm = -__builtin_inff(); int bad = !(T > 0.f) || !(T <= 3.0e38f) || !(Td > 0.f) || !(Td <= 3.0e38f);
        for (int i0 = tid; i0 < V; i0 += 4 * kThreads) {
            float pv[4], qv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int i = i0 + j * kThreads; pv[j] = i < V ? pr[i] : -__builtin_inff(); qv[j] = i < V ? qr[i] : -__builtin_inff(); }
#pragma unroll
            for (int j = 0; j < 4; ++j) { bad |= !(pv[j] + qv[j] < 3.0e38f); tm = fmaxf(tm, pv[j]); dm = fmaxf(dm, qv[j]); }
        }
        p_ref = block_max<kWaves>(static_cast<double>(tm), red);
        q_ref = block_max<kWaves>(static_cast<double>(dm), red);
        const int anybad = block_sum_i<kWaves>(bad, red);
        inv_temp = anybad ? 0.0 : 1.0 / static_cast<double>(T);
        inv_temp_q = anybad ? 0.0 : 1.0 / static_cast<double>(Td);
        double ps = 0.0;
        if (!anybad && p_ref > -3.0e38 && q_ref > -3.0e38)
            for (int i0 = tid; i0 < V; i0 += 4 * kThreads) {
                float pv[4], qv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) { const int i = i0 + j * kThreads; pv[j] = i < V ? pr[i] : -__builtin_inff(); qv[j] = i < V ? qr[i] : -__builtin_inff(); }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    ps += exp((static_cast<double>(pv[j]) - p_ref) * inv_temp);
                    positive += qv[j] > -3.0e38f;
                }
            }
        ptot = block_sum<kWaves>(ps, red); qtot = 1.0;
        if (anybad || !(ptot >= 1.0) || !(ptot < 1e300)) {
            if (tid == 0) mark_bad(fp, row, ptot, qtot);
            return;
        }
    } else {
        double ps = 0.0, qs = 0.0; int bad = 0;
        for (int i0 = tid; i0 < V; i0 += 4 * kThreads) {           // four tokens in flight
            float pv[4], qv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int i = i0 + j * kThreads; pv[j] = i < V ? pr[i] : 0.f; qv[j] = i < V ? qr[i] : 0.f; }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                bad |= !(qv[j] >= 0.f) | !(pv[j] >= 0.f);
                ps += static_cast<double>(pv[j]); qs += static_cast<double>(qv[j]);
                positive += qv[j] > 0.f;
            }
        }
        ptot = block_sum<kWaves>(ps, red);
        qtot = block_sum<kWaves>(qs, red);
        const int anybad = block_sum_i<kWaves>(bad, red);
        if (anybad || !(fabs(ptot - 1.0) <= 1e-3) || !(fabs(qtot - 1.0) <= 1e-3)) {
            if (tid == 0) mark_bad(fp, row, ptot, qtot);
            return;
        }
    }
    // With a top-k below the number of positive entries, or a nucleus cut (tail_mass > 0; Sec. 5.1: top-p/k
    // sampling of the draft restricts the domain): order the candidates by decreasing q (ties by token id)
    // and flag the first k' of them; the support is then the flagged tokens.
    int* member = fp.flag + row * vs;                       // by token id here; reused by rank later
    bool by_flag = false;
    positive = block_sum_i<kWaves>(positive, red);
    int kk = positive;                                      // the support's size
    const unsigned long long* sorted = nullptr;             // its tokens, where they are listed
    if (CUT || positive < V / 4) {
        // Nucleus cut: tokens are taken by decreasing q until their running sum reaches (1 - tail_mass) qtot.
        // Candidates first, so that only they are sorted: half of the budget tail_mass qtot goes to the tokens
        // below qmin = budget / (2 V) (fewer than V of them: below budget / 2 together), the other half to the
        // lowest occupied magnitude classes (exponent and four mantissa bits of q: every member is below the
        // class's upper edge, so count x edge bounds the class's mass).  Everything dropped here lies in the
        // tail that the exact walk below would leave out anyway.
        double qmin = 0.0; int bstar = 0;
        if constexpr (CUT) if (cut) {
            int* chist = reinterpret_cast<int*>(&S);             // 4096 classes = 16 KB of the sort's LDS
            static_assert(sizeof(S) >= 4096 * sizeof(int), "the class histogram borrows the sort's LDS");
            for (int c = tid; c < 4096; c += kThreads) chist[c] = 0;
            __syncthreads();
            const double budget = fp.tail_mass * qtot;
            qmin = 0.5 * budget / static_cast<double>(V);
            for (int i0 = tid; i0 < V; i0 += 4 * kThreads) {
                float qv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) { const int i = i0 + j * kThreads; qv[j] = i < V ? qr[i] : 0.f; }
#pragma unroll
                for (int j = 0; j < 4; ++j) if (static_cast<double>(qv[j]) >= qmin && qv[j] > 0.f) atomicAdd(&chist[__float_as_uint(qv[j]) >> 19], 1);
            }
            __syncthreads();
            bstar = class_threshold(chist, 0.5 * budget, dscan, &bsel);
        }
        int cnt = 0;
        for (int t0 = 0; t0 < V; t0 += 4 * kThreads) {           // 4 NT tokens per round
            float qv[4]; unsigned long long mask[4]; bool take[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int i = t0 + j * kThreads + tid; qv[j] = i < V ? qr[i] : (lg ? -__builtin_inff() : 0.f); }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                take[j] = (lg ? qv[j] > -3.0e38f : qv[j] > 0.f) && (!cut || (static_cast<double>(qv[j]) >= qmin && static_cast<int>(__float_as_uint(qv[j]) >> 19) >= bstar));
                mask[j] = __ballot(take[j]);
                if (lane == 0) wtot[j * kWaves + wv] = __popcll(mask[j]);
            }
            __syncthreads();
            int offs[4];
            const int run = group_offsets<kWaves>(wtot, offs);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = t0 + j * kThreads + tid;
                if (take[j]) {
                    const int off = cnt + offs[j] + __popcll(mask[j] & ((1ull << lane) - 1ull));
                    k0[off] = pack32(lg ? ~mono32(qv[j]) : ~__float_as_uint(qv[j]), i);   // ties: the sort is stable and this is token order
                }
                if (i < V) member[i] = 0;
            }
            cnt += run;
            __syncthreads();
        }
        sorted = k0;
        int keep = cnt;
        if constexpr (CUT) if (cnt > fp.k || (cut && cnt > 0)) {
            sorted = block_sort32(k0, k1, cnt, S);
            if (cut) {
                // the exact walk: running sums of q in the sorted order, added one after the other (wave 0), until
                // they reach (1 - tail_mass) qtot; the first rank that does is the last token of the support
                const double need = (1.0 - fp.tail_mass) * qtot;
                double carry = 0.0;
                double* xin = reinterpret_cast<double*>(&S.tile[0]); double* xout = xin + NT;   // the sort is done with its tile
                static_assert(sizeof(S.tile) >= (2 * NT + 1) * sizeof(double), "the walk borrows the sort's tile");
                if (tid == 0) bsel = cnt;                                // rank of the last kept token; cnt: never reached
                __syncthreads();
                for (int t0 = 0; t0 < cnt; t0 += kThreads) {
                    const int r = t0 + tid;
                    xin[tid] = r < cnt ? static_cast<double>(qr[packed_id(sorted[r])]) : 0.0;
                    __syncthreads();
                    const int todo = min(kThreads, (cnt - t0 + 15) & ~15);
                    if (wv == 0) wave_sequential_scan_padded<16>(xin, xout, todo, carry);       // 16: few registers, the others need theirs
                    __syncthreads();
                    if (r < cnt && xout[tid + 1] >= need) atomicMin(&bsel, r);
                    carry = xout[todo];
                    __syncthreads();
                    if (bsel < cnt) break;                               // uniform: read behind the barrier
                }
                keep = bsel < cnt ? bsel + 1 : cnt;
                __syncthreads();
            }
            if (fp.k < keep) keep = fp.k;
            for (int r = tid; r < keep; r += kThreads) member[packed_id(sorted[r])] = 1;
            by_flag = true;
        }
        __syncthreads();
        kk = keep;
    }
    if (kk == 0) {
        if (tid == 0) mark_bad(fp, row, ptot, qtot);
        return;
    }
    const RatioKey key_of{lg, inv_temp, inv_temp_q};
    SplitLds<NT>& L = lds.split;
    const int log_nb = log_buckets(kk), nb = 1 << log_nb;
    static_assert(SplitLds<NT>::kSamples >= kSamplesPerBucket << SplitLds<NT>::kLogBuckets || NT >= 1024, "samples for every bucket");
    __syncthreads();
    if (nb > 1) {
        // a token of every part of the support or the row, at a place that no pattern of the tokens follows
        const int ns = min(SplitLds<NT>::kSamples, kSamplesPerBucket * nb), of = sorted ? kk : V;
        int valid = 0;
        for (int t = tid; t < ns; t += NT) {
            const int lo = static_cast<int>(static_cast<long long>(t) * of / ns), hi = static_cast<int>(static_cast<long long>(t + 1) * of / ns);
            unsigned x = static_cast<unsigned>(t) * 0x9E3779B9u + 0x7F4A7C15u;
            x ^= x >> 15; x *= 0x85EBCA6Bu; x ^= x >> 13;
            const int at = lo + static_cast<int>(__umulhi(x, static_cast<unsigned>(max(hi - lo, 1))));
            const int id = sorted ? packed_id(sorted[at]) : at;
            const float qv = qr[id], pv = pr[id];
            const bool in = sorted || (lg ? qv > -3.0e38f : qv > 0.f);
            L.key[t] = in ? key_of(qv, pv) : ~0ull; L.id[t] = in ? id : 0x7fffffff;
            valid += in;
        }
        valid = block_sum_i<kWaves>(valid, red);                 // barriers inside
        block_bitonic<NT>(L.key, L.id, ns);                      // ns is a power of two
        const SplitView split(fp, row);
        for (int j = tid; j < nb - 1; j += NT) {
            const int at = static_cast<int>(static_cast<long long>(j + 1) * valid >> log_nb);
            split.key[j] = at < valid ? L.key[at] : ~0ull; split.id[j] = at < valid ? L.id[at] : 0x7fffffff;
        }
    }
    if (nb == 1 && sorted) {                                     // one bucket of listed tokens: here it is
        Element* elems = fp.elements() + row * vs;
        for (int r = tid; r < kk; r += NT) { const int id = packed_id(sorted[r]); elems[r] = Element{pr[id], qr[id], id}; }
        if (tid == 0) { const SplitView split(fp, row); split.first[0] = 0; split.first[1] = kk; }
    }
    if (tid == 0) {
        RowInfo info;
        info.support = kk; info.h = 0; info.status = GR_ROW_OK; info.iterations = 0;
        info.alpha_star = 0.0; info.res_total = 0.0; info.p_total = ptot; info.q_total = qtot; info.node_tokens = 0.0;
        info.p_ref = p_ref; info.inv_temp = inv_temp; info.q_ref = q_ref;
        fp.info[row] = info;
        // until the truncation kernel, for the next two: how to know the support, whether its elements are written
        fp.tcount[3 * row] = by_flag; fp.tcount[3 * row + 1] = nb == 1 && sorted;
    }
}

// ---- kernels 2 and 3: the bucket of every token and the buckets' sizes, then the elements.  A row is shared by the workgroups of its slices of
// `len` tokens; splitters and counters lie in LDS (`room` buckets).
constexpr int kCountThreads = 512, kLogCells = 10;
// Tokens from `from` on of a row, R to a thread: p, q, and whether the support has it.
template <int NT, int R>
struct Tokens {
    float p[R], q[R]; bool in[R];
    __device__ __forceinline__ void load(const FullParams& fp, int row, int from, int to, bool by_flag) {
        const float* pr = fp.p + static_cast<size_t>(row) * fp.V;
        const float* qr = fp.q + static_cast<size_t>(row) * fp.V;
        const int* member = fp.flag + row * (static_cast<size_t>(fp.V) + 2);
        int m[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = from + j * NT + static_cast<int>(threadIdx.x);
            q[j] = i < to ? qr[i] : -__builtin_inff(); p[j] = i < to ? pr[i] : 0.f;
            m[j] = by_flag && i < to ? member[i] : 0;
        }
#pragma unroll
        for (int j = 0; j < R; ++j) in[j] = by_flag ? m[j] != 0 : (fp.logits ? q[j] > -3.0e38f : q[j] > 0.f);
    }
};

// The search goes from the cell of a key, of 2^kLogCells equal ones over the splitters' range, whose splitters are counted: most cells hold one
// or none.  Bound: arithmetic, the quotient and the search.
__global__ __launch_bounds__(kCountThreads, 8) void full_count_kernel(FullParams fp, int slices, int len, int room) {
    extern __shared__ __align__(16) unsigned char full_lds[];
    constexpr int NT = kCountThreads, kCells = 1 << kLogCells;
    unsigned long long* key = reinterpret_cast<unsigned long long*>(full_lds);
    int* ids = reinterpret_cast<int*>(key + room); int* count = ids + room; int* below = count + room;   // below: kCells + 1 of them
    int row, slice;
    chunk_of(fp.B, slices, row, slice);
    if (row >= fp.B) return;
    const RowInfo info = fp.info[row];
    if (info.status == GR_ROW_BAD) return;
    const int tid = threadIdx.x;
    const size_t vs = static_cast<size_t>(fp.V) + 2;
    const int nb = 1 << log_buckets(info.support);
    const bool by_flag = fp.tcount[3 * row] != 0;
    const SplitView split(fp, row);
    for (int b = tid; b < nb; b += NT) {
        if (b < nb - 1) { key[b] = split.key[b]; ids[b] = split.id[b]; }
        count[b] = 0;
    }
    __syncthreads();
    unsigned long long base = 0ull;
    int shift = 0;
    if (nb > 1) {
        base = key[0];
        const unsigned long long range = key[nb - 2] - base;
        shift = max(0, 64 - kLogCells - (range ? __clzll(static_cast<long long>(range)) : 64));
        for (int c = tid; c <= kCells; c += NT) {
            const unsigned long long ahead = static_cast<unsigned long long>(c) << shift, from = ahead > ~base ? ~0ull : base + ahead;
            int b = 0;
            for (int step = nb >> 1; step > 0; step >>= 1) if (key[b + step - 1] < from) b += step;
            below[c] = c == 0 ? 0 : (c == kCells ? nb - 1 : b);
        }
        __syncthreads();
    }
    const RowValues val(fp, info, row);
    const RatioKey key_of{val.lg, val.inv_temp, val.inv_temp_q};
    double* rho_id = fp.rho_id + row * vs; int* rank_of = fp.rank_of + row * vs;
    const int end = min(fp.V, slice * len + len);
    for (int t0 = slice * len; t0 < end; t0 += 4 * NT) {
        Tokens<NT, 4> x;
        x.load(fp, row, t0, end, by_flag);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = t0 + j * NT + tid;
            if (x.in[j]) {
                int b = 0;                                       // the splitters that do not come after the token
                if (nb > 1) {
                    const unsigned long long k = key_of(x.q[j], x.p[j]);
                    const int c = k <= base ? 0 : static_cast<int>(min((k - base) >> shift, static_cast<unsigned long long>(kCells - 1)));
                    b = below[c];
                    for (int up = below[c + 1]; b < up;) {
                        const int mid = (b + up) >> 1;
                        const unsigned long long o = key[mid];
                        if (o < k || (o == k && ids[mid] <= i)) b = mid + 1; else up = mid;
                    }
                    split.bucket[i] = static_cast<unsigned short>(b);
                }
                atomicAdd(&count[b], 1);
            } else if (i < end) {
                // a token outside the support keeps all of p as residual
                rank_of[i] = -1;
                rho_id[i] = val.p(x.p[j]);
            }
        }
    }
    __syncthreads();
    for (int b = tid; b < nb; b += NT) split.count[slice * nb + b] = count[b];
}

// A tile of 8 NT tokens goes through LDS into bucket order, so that the elements of a bucket leave as one run: stores of single elements were
// spread over more lines than an L2 holds (1024 rows of 128256 tokens: 1840 us).
template <int NT>
__global__ __launch_bounds__(NT) void full_scatter_kernel(FullParams fp, int slices, int len, int room) {
    extern __shared__ __align__(16) unsigned char full_lds[];
    constexpr int R = 8, kTile = R * NT, NW = NT / 64;
    Element* tile = reinterpret_cast<Element*>(full_lds);
    // per bucket: tokens of the tile, its first place in the tile, the output slot of the tile's place 0, the next output slot
    int* count = reinterpret_cast<int*>(tile + kTile); int* start = count + room; int* dest = start + room; int* next = dest + room;
    unsigned short* where = reinterpret_cast<unsigned short*>(next + room);
    __shared__ int held;
    __shared__ int wsum[NW];
    int row, slice;
    chunk_of(fp.B, slices, row, slice);
    if (row >= fp.B || fp.info[row].status == GR_ROW_BAD || fp.tcount[3 * row + 1] != 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const size_t vs = static_cast<size_t>(fp.V) + 2;
    const int kk = fp.info[row].support, nb = 1 << log_buckets(kk);
    const bool by_flag = fp.tcount[3 * row] != 0;
    const SplitView split(fp, row);
    // exclusive sums over the buckets of what `of` gives for each, NT of them at a time; all threads call
    auto prefix = [&](auto of, auto put) {
        int run = 0;
        for (int b0 = 0; b0 < nb; b0 += NT) {
            const int b = b0 + tid, c = b < nb ? of(b) : 0, incl = wave_scan_i(c);
            if (lane == 63) wsum[wv] = incl;
            __syncthreads();
            int at = run + incl - c;
#pragma unroll
            for (int w = 0; w < NW; ++w) { const int x = wsum[w]; if (w < wv) at += x; run += x; }
            if (b < nb) put(b, at, c);
            if (b0 + NT < nb) __syncthreads();
        }
    };
    prefix([&](int b) { int all = 0; for (int s = 0; s < slices; ++s) all += split.count[s * nb + b]; return all; },
           [&](int b, int at, int) {
               if (slice == 0) { split.first[b] = at; if (b == 0) split.first[nb] = kk; }
               for (int s = 0; s < slice; ++s) at += split.count[s * nb + b];
               next[b] = at; count[b] = 0;
           });
    __syncthreads();
    Element* elems = fp.elements() + row * vs;
    const int end = min(fp.V, slice * len + len);
    int b[R];
    Tokens<NT, R> x;
    auto load = [&](int t0) {
        x.load(fp, row, t0, end, by_flag);
#pragma unroll
        for (int j = 0; j < R; ++j) { const int i = t0 + j * NT + tid; b[j] = nb > 1 && i < end ? split.bucket[i] : 0; }
    };
    load(slice * len);
    for (int t0 = slice * len; t0 < end; t0 += kTile) {
        int at[R];
#pragma unroll
        for (int j = 0; j < R; ++j) if (x.in[j]) at[j] = atomicAdd(&count[b[j]], 1);
        __syncthreads();
        prefix([&](int d) { return count[d]; },
               [&](int d, int from, int c) {
                   start[d] = from; dest[d] = next[d] - from; next[d] += c; count[d] = 0;
                   if (d == nb - 1) held = from + c;
               });
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (x.in[j]) {
                const int o = start[b[j]] + at[j];
                tile[o] = Element{x.p[j], x.q[j], t0 + j * NT + tid};
                where[o] = static_cast<unsigned short>(b[j]);
            }
        load(t0 + kTile);
        __syncthreads();
        for (int i = tid; i < held; i += NT) elems[dest[where[i]] + i] = tile[i];
    }
}

// ---- kernel 4: every bucket in order: token ids and pairs (p, q) by rank, and every token's rank.
//
// A token's place in its bucket is found through the key's place between the bucket's smallest and largest one: it goes to one of kCells cells,
// half a token each on average, and is compared with the others of its cell.  Where the keys lie too unevenly for that (kCrowded in a
// cell) the bucket is sorted; one above kBucketCap (the sample missed it, or the row has more than kBucket tokens to each of all buckets) goes by sorted
// stretches.  Buckets of a row share an XCD: the ranks go to 4 V bytes of it at random and stay in its L2 meanwhile.
constexpr int kBucketThreads = 512, kCells = 2048, kCrowded = 48;
__global__ __launch_bounds__(kBucketThreads, 8) void full_bucket_kernel(FullParams fp, int buckets) {
    constexpr int NT = kBucketThreads, PER = kBucketCap / NT, kWaves = NT / 64;
    __shared__ union { unsigned long long key[kBucketCap]; float2 pair[kBucketCap]; } A;
    __shared__ int ids[kBucketCap];
    __shared__ int cells[kCells];
    __shared__ unsigned long long wred[2][kWaves];
    __shared__ int wsum[kWaves], wmost[kWaves];
    int row, b;
    chunk_of(fp.B, buckets, row, b);
    if (row >= fp.B) return;
    const size_t vs = static_cast<size_t>(fp.V) + 2;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const SplitView split(fp, row);
    const RowInfo info = fp.info[row];
    const int at = split.first[b], count = split.first[b + 1] - at;
    if (info.status == GR_ROW_BAD || b >> log_buckets(info.support) != 0) return;
    const RowValues val(fp, info, row);
    const RatioKey key_of{val.lg, val.inv_temp, val.inv_temp_q};
    const Element* elems = fp.elements() + row * vs + at;
    int* order = fp.order + row * vs + at; float2* pairs = fp.pairs + row * vs + at; int* rank_of = fp.rank_of + row * vs;
    auto before = [](unsigned long long k0, int i0, unsigned long long k1, int i1) { return k0 < k1 || (k0 == k1 && i0 < i1); };
    if (count > kBucketCap) {
        // stretches of kBucketCap tokens, each put in order in LDS; every token of the bucket finds how many of it come before itself
        unsigned long long* key = fp.key0 + row * vs + at; int* rank = fp.byq + row * vs + at;   // later kernels fill them
        for (int i = tid; i < count; i += NT) { const Element e = elems[i]; key[i] = key_of(e.q, e.p); rank[i] = 0; }
        for (int t0 = 0; t0 < count; t0 += kBucketCap) {
            __syncthreads();
            for (int i = tid; i < kBucketCap; i += NT) {
                const bool in = t0 + i < count;
                A.key[i] = in ? key[t0 + i] : ~0ull; ids[i] = in ? elems[t0 + i].id : 0x7fffffff;
            }
            block_bitonic<NT>(A.key, ids, kBucketCap);
            for (int i = tid; i < count; i += NT) {
                const unsigned long long k = key[i];
                const int id = elems[i].id;
                int lo = 0;
#pragma unroll
                for (int step = kBucketCap / 2; step > 0; step >>= 1) if (before(A.key[lo + step - 1], ids[lo + step - 1], k, id)) lo += step;
                rank[i] += lo + before(A.key[lo], ids[lo], k, id);
            }
        }
        for (int i = tid; i < count; i += NT) {
            const Element e = elems[i];
            const int r = rank[i];
            order[r] = e.id; pairs[r] = make_float2(e.p, e.q); rank_of[e.id] = at + r;
        }
        return;
    }
    Element e[PER]; unsigned long long key[PER];
    unsigned long long kmin = ~0ull, kmax = 0ull;
    for (int c = tid; c < kCells; c += NT) cells[c] = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) if (j * NT + tid < count) e[j] = elems[j * NT + tid];
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (j * NT + tid < count) { key[j] = key_of(e[j].q, e[j].p); kmin = min(kmin, key[j]); kmax = max(kmax, key[j]); }
    kmin = wave_min_u64(kmin); kmax = ~wave_min_u64(~kmax);
    if (lane == 0) { wred[0][wv] = kmin; wred[1][wv] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { kmin = min(kmin, wred[0][w]); kmax = max(kmax, wred[1][w]); }
    // tokens of one ratio go by their ids
    const bool one = kmin == kmax;
    const unsigned long long range = one ? static_cast<unsigned long long>(fp.V) : kmax - kmin;
    const int shift = max(0, 32 - __clzll(static_cast<long long>(range)));
    // a ratio's pattern is even in its logarithm; the difference of two logits is the logarithm itself
    const double x0 = val.lg ? unmono64(~kmin) : 0.0, spread = val.lg ? x0 - unmono64(~kmax) : 0.0;
    const bool linear = val.lg && !one && spread > 1e-290 && spread < 1e300;
    const double per = linear ? 4294967040.0 / spread : 0.0;
    const unsigned top = linear ? 0xFFFFFFFFu : static_cast<unsigned>(range >> shift);
    const unsigned scale = top < kCells ? 0u : static_cast<unsigned>(static_cast<double>(kCells) * 4294967296.0 / (static_cast<double>(top) + 1.0));
    auto cell_of = [&](unsigned long long k, int id) {
        const unsigned v = linear ? static_cast<unsigned>((x0 - unmono64(~k)) * per)
                                  : static_cast<unsigned>((one ? static_cast<unsigned long long>(id) : k - kmin) >> shift);
        return static_cast<int>(scale ? __umulhi(v, scale) : v);
    };
    int cell[PER], slot[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) if (j * NT + tid < count) { cell[j] = cell_of(key[j], e[j].id); slot[j] = atomicAdd(&cells[cell[j]], 1); }
    __syncthreads();
    {
        int c[kCells / NT], tot = 0, most = 0;
#pragma unroll
        for (int j = 0; j < kCells / NT; ++j) { c[j] = cells[kCells / NT * tid + j]; tot += c[j]; most = max(most, c[j]); }
        const int incl = wave_scan_i(tot);
        const bool crowded = __ballot(most > kCrowded) != 0ull;
        if (lane == 63) { wsum[wv] = incl; wmost[wv] = crowded; }
        __syncthreads();
        int run = incl - tot;
        for (int w = 0; w < wv; ++w) run += wsum[w];
#pragma unroll
        for (int j = 0; j < kCells / NT; ++j) { cells[kCells / NT * tid + j] = run; run += c[j]; }
    }
    bool crowded = false;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) crowded |= wmost[w] != 0;
    __syncthreads();
    int rank[PER];
    if (!crowded) {
#pragma unroll
        for (int j = 0; j < PER; ++j) if (j * NT + tid < count) { const int o = cells[cell[j]] + slot[j]; A.key[o] = key[j]; ids[o] = e[j].id; }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (j * NT + tid < count) {
                const int from = cells[cell[j]], to = cell[j] + 1 < kCells ? cells[cell[j] + 1] : count;
                rank[j] = from;
                for (int o = from; o < to; ++o) rank[j] += before(A.key[o], ids[o], key[j], e[j].id);
            }
        __syncthreads();
    } else {
        int size = 64;
        while (size < count) size *= 2;
        for (int i = tid; i < size; i += NT) { A.key[i] = ~0ull; ids[i] = 0x7fffffff; }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) if (j * NT + tid < count) { A.key[j * NT + tid] = key[j]; ids[j * NT + tid] = e[j].id; }
        __syncthreads();
        block_bitonic<NT>(A.key, ids, size);
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (j * NT + tid < count) {
                int lo = 0;
                for (int step = size >> 1; step > 0; step >>= 1) if (before(A.key[lo + step - 1], ids[lo + step - 1], key[j], e[j].id)) lo += step;
                rank[j] = lo;
            }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (j * NT + tid < count) { A.pair[rank[j]] = make_float2(e[j].p, e[j].q); ids[rank[j]] = e[j].id; rank_of[e[j].id] = at + rank[j]; }
    __syncthreads();
    for (int i = tid; i < count; i += NT) { pairs[i] = A.pair[i]; order[i] = ids[i]; }
}

// ---- kernel 5: prefix sums in the order, F, H*, alpha*, suffix minima, residuals, records, blocks.
//
// Ascending, in tiles of 2048 ranks: the sequential sums P (waves 0-3) and Q (waves 4-7), eight terms per lane (RunSum).  A sum that leaves its binade inside the tile is right up to the lane where it
// does; the lanes behind it go again with the new unit (a row's sums double some 40 times, mostly in its first tile).  So one wave adds the
// first ranks of a row, where most of that happens: all of a row of up to 1024 ranks, 256 of a longer one.  No ranks / 256 / 512 / 1024 so, the
// call: 1 row of 300 tokens 128 / 119 / 114 / 114 us, 256 rows of 700 278 / 271 / 269 / 257, 1 row of 1500 157 / 154 / 156 / 161, 256 rows of 8192
// 502 / 493 / 499 / 504.
// Descending: F, its suffix minima G, residuals, records (F(m) <= G(m + 1); m = kk always) and the number of records behind
// every rank, in one pass: below H* the suffix minimum is F(h) throughout, so residuals and records there come out 0 and none,
// and h is the first record.
// Bound: memory (44 bytes per token: most tiles hold no record, and their ranks' blocks are written once, when the records are counted) and the two
// passes' barriers.  1024 rows of 128256 tokens: 2110 us with every rank's block written twice, 1900 now.
// One wave adding for each sum from LDS, and P, Q, F, the targets and the records' flags as arrays of their own: 9.5 ms for
// 1024 rows of 128256 tokens, 3.06 for 256.
__global__ __launch_bounds__(kScanThreads, 4) void full_scan_kernel(FullParams fp) {
    constexpr int NT = kScanThreads, NW = NT / 64, CW = NW / 2, E = 8, kTile = 64 * CW * E, PER = kTile / NT;
    static_assert(CW == 4 && PER == 4, "four waves per sum, four ranks per thread");
    constexpr int kRound = 32, kHead = 256, kWhole = 1024;     // ranks that one wave adds at the start of a row, and of a row that it adds alone
    static_assert(kHead % (kRound * E) == 0 && kWhole <= kTile, "rounds of the first tile, whole lanes");
    __shared__ double xs[2][kTile + kTile / E];                // a lane's eight terms, then its sums; one word of padding per lane
    __shared__ RunSum run[NW];
    __shared__ double upto[NW];
    __shared__ int stop[NW];
    __shared__ double wmin[2][NW];
    __shared__ int wcnt[2][NW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int V = fp.V, n = fp.n;
    const size_t vs = static_cast<size_t>(V) + 2;
    RowInfo info = fp.info[row];
    if (info.status == GR_ROW_BAD) return;
    const int kk = info.support;
    const RowValues val(fp, info, row);
    const float2* by_rank = fp.pairs + row * vs;
    double* P = fp.P + row * vs; double* Q = fp.Q + row * vs; double* rho = fp.rho + row * vs;
    int* blk = fp.blk + row * vs; int* blo = fp.blo + row * vs; int* bcount = fp.bcount + row * vs; int* behind = fp.val0 + row * vs;
    int* tile_rec = fp.flag + row * vs;                        // per tile: the records behind all of its ranks, -1 where it holds one itself
    auto pad = [](int i) { return i + (i >> 3); };

    const int chain = wv / CW, cw = wv % CW;
    double acc = 0.0;                                          // the running sum of this wave's chain
    if (tid == 0) { P[0] = 0.0; Q[0] = 0.0; }
    float2 x2[PER];                                            // the next tile's pairs are on their way while this one is added up
#pragma unroll
    for (int j = 0; j < PER; ++j) x2[j] = j * NT + tid < kk ? by_rank[j * NT + tid] : make_float2(0.f, 0.f);
    for (int t0 = 0; t0 < kk; t0 += kTile) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = j * NT + tid, r = t0 + i;
            const bool in = r < kk;
            xs[0][pad(i)] = in ? val.p(x2[j].x) : 0.0; xs[1][pad(i)] = in ? val.q(x2[j].y) : 0.0;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) { const int r = t0 + kTile + j * NT + tid; x2[j] = r < kk ? by_rank[r] : make_float2(0.f, 0.f); }
        __syncthreads();
        const int head = t0 > 0 ? 0 : (kk <= kWhole ? kWhole : kHead);   // ranks whose sums take the place of their terms here
        if (head) {
#pragma clang fp contract(off)
            if (cw == 0) {
                for (int i0 = 0; i0 < min(head, kk); i0 += kRound) {
                    double v[kRound];
#pragma unroll
                    for (int i = 0; i < kRound; ++i) v[i] = xs[chain][pad(i0 + i)];
#pragma unroll
                    for (int i = 0; i < kRound; ++i) { acc = acc + v[i]; v[i] = acc; }
                    if (lane == 0) {
#pragma unroll
                        for (int i = 0; i < kRound; ++i) xs[chain][pad(i0 + i)] = v[i];
                    }
                }
                if (lane == 0) upto[wv] = acc;
            }
            __syncthreads();
            acc = upto[chain * CW];
        }
        double x[E], sum[E];
        const int mine = (cw * 64 + lane) * (E + 1);
#pragma unroll
        for (int e = 0; e < E; ++e) { x[e] = xs[chain][mine + e]; sum[e] = x[e]; }
        if (t0 + head < kk) {
#pragma clang fp contract(off)
            for (int pos = head / E;;) {                       // the lanes of the chain from `pos` on
                const long long bits = __double_as_longlong(acc);
                const double unit = __longlong_as_double(bits & 0x7FF0000000000000ll), odd = __longlong_as_double((bits & 0x7FF0000000000000ll) | 1ll);
                const bool none = acc < 1e-290;                // nothing to speak of yet: the first term starts the sum
                const bool act = cw * 64 + lane >= pos;
                double a0 = unit, a1 = odd;
                if (act) {
#pragma unroll
                    for (int e = 0; e < E; ++e) { a0 = a0 + x[e]; a1 = a1 + x[e]; }
                }
                RunSum v;
                v.d[0] = a0 - unit; v.d[1] = a1 - odd;
                v.par = static_cast<int>(__double_as_longlong(a0) & 1ll) | (static_cast<int>(__double_as_longlong(a1) & 1ll) << 1);
                scan_step<0x111, 0xF>(v); scan_step<0x112, 0xF>(v); scan_step<0x114, 0xF>(v); scan_step<0x118, 0xF>(v);
                scan_step<0x142, 0xA>(v); scan_step<0x143, 0xC>(v);
                if (lane == 63) run[wv] = v;
                RunSum before;                                 // the lanes before this one
                before.d[0] = __shfl_up(v.d[0], 1); before.d[1] = __shfl_up(v.d[1], 1); before.par = __shfl_up(v.par, 1);
                if (lane == 0) { before.d[0] = 0.0; before.d[1] = 0.0; before.par = 2; }
                __syncthreads();
                double delta = 0.0;
                int s = static_cast<int>(bits & 1ll);
                for (int w = 0; w < cw; ++w) { const RunSum c = run[chain * CW + w]; delta = delta + (s ? c.d[1] : c.d[0]); s = (c.par >> s) & 1; }
                delta = delta + (s ? before.d[1] : before.d[0]);
                double t = none ? acc : acc + delta;
                const double start = t;
                if (act) {
#pragma unroll
                    for (int e = 0; e < E; ++e) { t = t + x[e]; sum[e] = t; }
                }
                const unsigned long long out = __ballot(act && (none ? t != start : !(t < 2.0 * unit)));
                const int last = out ? __ffsll(static_cast<long long>(out)) - 1 : 63;
                const double end = read_lane(t, last);
                if (lane == 0) { upto[wv] = end; stop[wv] = out ? cw * 64 + last + 1 : 0; }
                __syncthreads();
                int next[2];
                for (int c = 0; c < 2; ++c) {
                    next[c] = 64 * CW;
                    for (int w = 0; w < CW; ++w) {
                        if (c == chain) acc = upto[c * CW + w];
                        if (stop[c * CW + w]) { next[c] = stop[c * CW + w]; break; }
                    }
                }
                pos = next[chain];
                if (next[0] == 64 * CW && next[1] == 64 * CW) break;
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) xs[chain][mine + e] = sum[e];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int i = j * NT + tid, r = t0 + i;
            if (r < kk) { P[r + 1] = xs[0][pad(i)]; Q[r + 1] = xs[1][pad(i)]; }
        }
        __syncthreads();                                       // the next tile's terms take the place of these sums
    }
    __syncthreads();
    const double stot = Q[kk];
    // thread t holds four ranks, the last threads the first ones: what lies behind a rank is a scan over the threads
    double later = 1e300;                                      // min of F over the tiles above
    int nrec = 0;                                              // records in the tiles above
    const int ntile = kk / kTile + 1;
    double Pn[PER], Qn[PER];
    auto fetch = [&](int t) {
        const int m0 = t * kTile + (NT - 1 - tid) * PER;
#pragma unroll
        for (int j = 0; j < PER; ++j) { const bool in = t >= 0 && m0 + j <= kk; Pn[j] = in ? P[m0 + j] : 0.0; Qn[j] = in ? Q[m0 + j] : 0.0; }
    };
    fetch(ntile - 1);
    for (int t = ntile - 1, b = 0; t >= 0; --t, b ^= 1) {
#pragma clang fp contract(off)
        const int m0 = t * kTile + (NT - 1 - tid) * PER;
        double a[PER], s[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            a[j] = 1e300;
            if (m0 + j <= kk) a[j] = m0 + j == 0 ? 0.0 : Pn[j] - ipow(Qn[j] / stot, n);
        }
        fetch(t - 1);
        s[3] = a[3]; s[2] = fmin(a[2], s[3]); s[1] = fmin(a[1], s[2]); s[0] = fmin(a[0], s[1]);
        const double incl = wave_scan_min(s[0]);
        double after = __shfl_up(incl, 1);
        if (lane == 0) after = 1e300;
        if (lane == 63) wmin[b][wv] = incl;
        __syncthreads();
        double total = 1e300;
#pragma unroll
        for (int w = 0; w < NW; ++w) { const double x = wmin[b][w]; total = fmin(total, x); if (w < wv) after = fmin(after, x); }
        after = fmin(after, later);                            // G(m0 + 4)
        int rec[PER], cnt = 0;
#pragma unroll
        for (int j = PER - 1; j >= 0; --j) {
            const int m = m0 + j;
            const double g = fmin(s[j], after), gn = j < PER - 1 ? fmin(s[j < PER - 1 ? j + 1 : j], after) : after;   // G(m), G(m + 1)
            rec[j] = m <= kk && (m == kk || a[j] <= gn) ? 1 : 0;
            cnt += rec[j];
            if (m < kk) rho[m] = gn - g;
        }
        const int ci = wave_scan_i(cnt);
        if (lane == 63) wcnt[b][wv] = ci;
        __syncthreads();
        int c = nrec + ci - cnt, here = 0;                     // records behind this thread's ranks, and in this tile
#pragma unroll
        for (int w = 0; w < NW; ++w) { const int x = wcnt[b][w]; if (w < wv) c += x; here += x; }
        if (tid == 0) tile_rec[t] = here ? -1 : nrec;
        if (here)
#pragma unroll
            for (int j = PER - 1; j >= 0; --j) {
                const int m = m0 + j;
                if (m < kk) blk[m] = c;                        // for now the records behind token m
                if (rec[j]) { behind[c] = m; ++c; }
            }
        nrec += here;
        later = fmin(later, total);
    }
    __syncthreads();
    // records in rising order, and every token's block: the records up to its rank
    for (int t = 0; t < ntile; ++t) {
        const int c = tile_rec[t];
#pragma unroll
        for (int j = 0; j < PER; ++j) { const int m = t * kTile + j * NT + tid; if (m < kk) blk[m] = nrec - (c < 0 ? blk[m] : c); }
    }
    for (int i = tid; i <= nrec; i += NT) { bcount[i] = 0; if (i > 0) blo[i] = behind[nrec - i]; }
    if (tid == 0) {
#pragma clang fp contract(off)
        const int h = behind[nrec - 1];
        const double Fh = h == 0 ? 0.0 : P[h] - ipow(Q[h] / stot, n);
        info.h = h;
        info.alpha_star = 1.0 + Fh;
        info.res_total = -Fh;
        fp.info[row] = info;
        fp.nblk[row] = nrec - 1;
        fp.accept_prob[row] = static_cast<float>(1.0 + Fh);
    }
}

// ---- kernel 6: truncation sets (Alg. 1: fewest tokens by decreasing q with gamma_T <= tau inside H*,
// epsilon_T <= tau outside), size of every program, row status.
//
// Bound: the pass over q (twice, 4 bytes a token) and, where many tokens stay, their sort.  A workgroup of 256 threads that read
// q in ratio order as float64 and sorted by eight passes of 12 bytes took 7.2 ms for 1024 rows of 128256 tokens; this without the
// rows that are known to end above the cap before their sort, 4.5.
template <int NT>
__global__ __launch_bounds__(NT) void full_trunc_kernel(FullParams fp) {
    constexpr int kWaves = NT / 64;
    __shared__ Sort32Lds<NT> S;
    __shared__ int cnt_in, cnt_out, act_in, capped, bsel;
    __shared__ int wtot[4 * kWaves];
    __shared__ double dscan[gr::kThreads];
    __shared__ double red[kWaves];
    __shared__ double wx[2][64];
    __shared__ double wo[2][65];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int V = fp.V, n = fp.n;
    const size_t vs = static_cast<size_t>(V) + 2;
    const RowInfo info = fp.info[row];
    if (info.status == GR_ROW_BAD) return;
    const int kk = info.support, h = info.h;
    const RowValues val(fp, info, row);
    const bool lg = val.lg;
    const float* qr = fp.q + static_cast<size_t>(row) * V;
    const int* order = fp.order + row * vs; const int* rank_of = fp.rank_of + row * vs;
    const float2* by_rank = fp.pairs + row * vs;
    unsigned long long* k0 = fp.key0 + row * vs; unsigned long long* k1 = fp.key1 + row * vs;
    int* byq = fp.byq + row * vs;
    const double* Q = fp.Q + row * vs; const double* rho = fp.rho + row * vs;
    const int* blk = fp.blk + row * vs; const int* blo = fp.blo + row * vs;
    int* bcount = fp.bcount + row * vs;
    const double stot = Q[kk];
    auto qn = [&](int r) { return val.q(by_rank[r].y) / stot; };
    auto target = [&](int r) { return val.p(by_rank[r].x) - rho[r]; };

    // A large support is gone through in token order (its ties go to the lower id, and q is read as it lies), a small one by its ranks.
    const bool ids = kk > V / 8;
    const int count = ids ? V : kk;
    auto member = [&](int i) { return i < count && (!ids || kk == V || rank_of[i] >= 0); };
    auto raw = [&](int i) { return ids ? qr[i] : by_rank[i].y; };
    auto cls = [&](float q) { return static_cast<int>(__float_as_uint(lg ? static_cast<float>(val.q(q)) : q) >> 19); };
    // A token joins a truncation set only while the mass before it leaves more than tau.  The lowest-q tokens whose
    // normalised masses sum to at most tau / n can therefore never join: before any of them lies everything else of
    // its side, so what is left is at most Q^n - (Q - tau/n)^n <= tau.  They are left out of the sort (found, safely,
    // with the magnitude-class histogram: count x upper edge bounds a class's mass); the walk over the others is
    // the same arithmetic as before.
    int bstar = 0;
    if (fp.tau > 0.0) {
        int* chist = reinterpret_cast<int*>(&S);
        static_assert(sizeof(S) >= 4096 * sizeof(int), "the class histogram borrows the sort's LDS");
        for (int c = tid; c < 4096; c += NT) chist[c] = 0;
        __syncthreads();
        for (int i0 = tid; i0 < count; i0 += 4 * NT) {
            float qv[4]; bool in[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int i = i0 + j * NT; in[j] = member(i); qv[j] = i < count ? raw(i) : 0.f; }
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int c = in[j] ? cls(qv[j]) : 0; if (c > 0) atomicAdd(&chist[c], 1); }
        }
        __syncthreads();
        bstar = class_threshold(chist, (fp.tau / static_cast<double>(n)) * (1.0 - 1e-6) * stot, dscan, &bsel);   // the margin covers the rounding of q to float
    }
    // the tokens that stay: inside H* first, decreasing q (the leading 32 or 33 bits of an element), token id
    int kept = 0, kin = 0;
    for (int t0 = 0; t0 < count; t0 += 4 * NT) {
        float qv[4]; bool take[4]; unsigned long long mask[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int i = t0 + j * NT + tid; take[j] = member(i); qv[j] = i < count ? raw(i) : 0.f; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            take[j] = take[j] && (bstar == 0 || cls(qv[j]) >= bstar);
            mask[j] = __ballot(take[j]);
            if (lane == 0) wtot[j * kWaves + wv] = __popcll(mask[j]);
        }
        __syncthreads();
        int offs[4];
        const int run = group_offsets<kWaves>(wtot, offs);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = t0 + j * NT + tid;
            if (take[j]) {
                const int id = ids ? i : order[i], r = ids ? rank_of[i] : i;
                const bool in = r < h;
                kin += in;
                // q < 2, so bit 31 of ~bits(q) is always set: it carries the class instead; a draft logit's pattern needs all 32 bits
                k0[kept + offs[j] + __popcll(mask[j] & ((1ull << lane) - 1ull))] =
                    lg ? (static_cast<unsigned long long>(~mono32(qv[j])) << 31) | (in ? 0ull : 0x8000000000000000ull) | static_cast<unsigned>(id)
                       : pack32((~__float_as_uint(qv[j]) & 0x7FFFFFFFu) | (in ? 0u : 0x80000000u), id);
            }
        }
        kept += run;
        __syncthreads();
    }
    const int kept_in = block_sum_i<kWaves>(kin, red);
    if (tid == 0) { cnt_in = 0; cnt_out = 0; act_in = 0; capped = 0; }
    __syncthreads();
    // Many tokens that stay are a sort of their own, and most such rows end above the cap.  A token whose class leaves more than tau
    // in the classes below it joins its set whatever the order within the classes, so where those alone exceed the cap, the row does.
    // The large workgroup only: the small one's LDS holds one histogram of the two, and its rows have at most 8192 tokens to sort.
    if constexpr (NT >= 1024) {
        if (kept > NT) {
            int* chist = reinterpret_cast<int*>(&S);
            static_assert(sizeof(S) >= 2 * 4096 * sizeof(int), "one histogram for each side");
            for (int c = tid; c < 2 * 4096; c += NT) chist[c] = 0;
            __syncthreads();
            for (int r0 = tid; r0 < kk; r0 += 4 * NT) {
                float qv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) { const int r = r0 + j * NT; qv[j] = r < kk ? by_rank[r].y : 0.f; }
#pragma unroll
                for (int j = 0; j < 4; ++j) { const int r = r0 + j * NT; if (r < kk) atomicAdd(&chist[(r < h ? 0 : 4096) + cls(qv[j])], 1); }
            }
            __syncthreads();
            const double more = fp.tau * (1.0 + 1e-6) + 1e-12, Qh = Q[h] / stot;
            const int c_in = definite_class(chist, [&](double m) { return ipow(Qh, n) - ipow(fmax(Qh - m / stot, 0.0), n) > more; }, dscan, &bsel);
            const int c_out = definite_class(chist + 4096, [&](double m) { return 1.0 - ipow(1.0 - m / stot, n) > more; }, dscan, &bsel);
            for (int r0 = 0; r0 < kk; r0 += 4 * NT) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = r0 + j * NT + tid;
                    const float2 x = r < kk ? by_rank[r] : make_float2(0.f, 0.f);
                    const bool in = r < kk && cls(x.y) >= (r < h ? c_in : c_out) && val.p(x.x) - rho[min(r, kk - 1)] > 0.0;
                    if (in && r < h) { atomicAdd(&act_in, 1); }
                    else if (in) {
                        const int bl = blk[r];
                        if (blo[bl + 1] - blo[bl] >= 2) {
                            const int lead = __builtin_amdgcn_readfirstlane(bl);
                            const unsigned long long same = __ballot(bl == lead);
                            if (bl == lead) { if (lane == __ffsll(static_cast<long long>(same)) - 1 && atomicAdd(&bcount[bl], __popcll(same)) + __popcll(same) > fp.max_T) capped = 1; }
                            else if (atomicAdd(&bcount[bl], 1) + 1 > fp.max_T) capped = 1;
                        }
                    }
                }
                __syncthreads();
                const bool over = act_in > fp.max_T || capped != 0;
                __syncthreads();
                if (over) {
                    if (tid == 0) {
                        fp.tcount[3 * row] = 0; fp.tcount[3 * row + 1] = 0; fp.tcount[3 * row + 2] = 0;
                        RowInfo out = info;
                        out.status = GR_ROW_TRUNC_CAP;
                        fp.info[row] = out;
                        fp.status[row] = GR_ROW_TRUNC_CAP;
                    }
                    return;
                }
            }
            for (int b = tid; b <= fp.nblk[row] + 1; b += NT) bcount[b] = 0;   // the walk counts again
            if (tid == 0) act_in = 0;
            __syncthreads();
        }
    }
    const int id_shift = lg ? 31 : 32;
    auto id_of = [&](unsigned long long e) { return static_cast<int>(e & ((1ull << id_shift) - 1ull)); };
    if (kept <= NT) {
        // few of them, the common case: every thread counts what comes before its own
        const unsigned long long mine = tid < kept ? k0[tid] : ~0ull;
        S.tile[tid] = mine;
        __syncthreads();
        if (tid < kept) {
            int at = 0;
#pragma unroll 8
            for (int o = 0; o < kept; ++o) at += S.tile[o] < mine;
            byq[at] = rank_of[id_of(mine)];
        }
    } else {
        unsigned long long* e = k0;
        auto other = [&]() { return e == k0 ? k1 : k0; };
        if (!ids) e = block_sort32(e, other(), kept, S, 0, 3);   // ids below 2^24
        e = block_sort32(e, other(), kept, S, id_shift);
        if (lg) e = block_sort32(e, other(), kept, S, 63, 1);
        for (int i = tid; i < kept; i += NT) byq[i] = rank_of[id_of(e[i])];
    }
    __syncthreads();
    const double Qh = Q[h] / stot;
    // wave 0 walks H* by decreasing q, wave 1 the other tokens: a token joins T while the mass before
    // it leaves more than tau (running sums added one after the other, as a sequential loop would).
    // The walk only counts; the ranks and masses of the next two rounds are already on their way.  Inside H* it ends, the row
    // capped, with more active tokens than a program may have.
    if (wv < 2) {
#pragma clang fp contract(off)
        const int first = wv == 0 ? 0 : kept_in;                 // the tokens of H* that stayed come first
        const int len = wv == 0 ? kept_in : kept - kept_in;
        const double bound = wv == 0 ? ipow(Qh, n) : 1.0;
        double acc = wv == 0 ? 0.0 : Qh;
        int taken = 0, active = 0;
        bool done = false;
        int r1 = (lane < len) ? byq[first + lane] : 0;                        // ranks of round 0
        int r2 = (64 + lane < len) ? byq[first + 64 + lane] : 0;              // ranks of round 1
        double m1 = (lane < len) ? qn(r1) : 0.0;                              // masses of round 0
        for (int base = 0; base < len && !done; base += 64) {
            const bool valid = base + lane < len;
            const double mine = m1;
            const bool act = wv == 0 && valid && target(r1) > 0.0;
            m1 = (base + 64 + lane < len) ? qn(r2) : 0.0;
            r1 = r2;
            r2 = (base + 128 + lane < len) ? byq[first + base + 128 + lane] : 0;
            // running sums through a wave-private LDS strip (broadcast reads; see the padded scan)
            wx[wv][lane] = mine;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
            wave_sequential_scan_padded<32>(wx[wv], wo[wv], 64, acc);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
            const double before = wo[wv][lane];
            acc = wo[wv][64];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
            const double bn = (before > 0.0) ? ipow(before, n) : 0.0;
            const bool in = valid && (bound - bn > fp.tau);
            const unsigned long long out_mask = __ballot(valid && !in);
            int upto = 64;                                       // lanes below `upto` join T
            if (out_mask) { upto = __ffsll(static_cast<long long>(out_mask)) - 1; done = true; }
            taken += __popcll(__ballot(valid && lane < upto));
            active += __popcll(__ballot(act && lane < upto));
            done = done || active > fp.max_T;
        }
        if (lane == 0) { if (wv == 0) { cnt_in = taken; act_in = active; } else cnt_out = taken; }
    }
    __syncthreads();
    // count the active tokens of every program outside H*
    {
        const int nout = cnt_out;
        for (int i0 = tid; i0 < nout; i0 += 4 * NT) {
            int r[4]; double t[4]; int bl[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { const int i = i0 + j * NT; r[j] = i < nout ? byq[kept_in + i] : -1; }
#pragma unroll
            for (int j = 0; j < 4; ++j) { t[j] = r[j] >= 0 ? target(r[j]) : 0.0; bl[j] = r[j] >= 0 ? blk[r[j]] : 0; }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (t[j] > 0.0 && blo[bl[j] + 1] - blo[bl[j]] >= 2) {
                    const int old = atomicAdd(&bcount[bl[j]], 1);
                    if (old + 1 > fp.max_T) capped = 1;
                }
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int status = (act_in > fp.max_T || capped) ? GR_ROW_TRUNC_CAP : GR_ROW_OK;
        fp.tcount[3 * row] = cnt_in; fp.tcount[3 * row + 1] = cnt_out; fp.tcount[3 * row + 2] = kept_in;
        RowInfo out = info;
        out.status = status;
        fp.info[row] = out;
        fp.status[row] = status;
    }
}

// ---- kernel 7: the dense per-token arrays that the verify and slice kernels read, of the rows within the cap: start weights by
// rank (target / Pr[token drawn within its system], inner ones in the slack's gauge) and the residuals by token id.
// Bound: memory.  Inside the programs kernel, one workgroup of 512 threads to a compute unit, these arrays were
// most of the 4.8 ms for 1024 rows of 128256 tokens.
__global__ __launch_bounds__(kThreads) void full_dense_kernel(FullParams fp, int chunks) {
    int row, chunk;
    chunk_of(fp.B, chunks, row, chunk);
    if (row >= fp.B) return;
    const int n = fp.n;
    const size_t vs = static_cast<size_t>(fp.V) + 2;
    const RowInfo info = fp.info[row];
    const int kk = info.support, h = info.h;
    if (info.status != GR_ROW_OK || chunk * kChunkRanks >= kk) return;
    const RowValues val(fp, info, row);
    const float2* by_rank = fp.pairs + row * vs;
    const int* order = fp.order + row * vs; const int* blk = fp.blk + row * vs; const int* blo = fp.blo + row * vs;
    const double* Q = fp.Q + row * vs; const double* rho = fp.rho + row * vs;
    double* weight = fp.weight + row * vs; double* rho_id = fp.rho_id + row * vs;
    const double stot = Q[kk];
    const int end = min(kk, (chunk + 1) * kChunkRanks);
    for (int r0 = chunk * kChunkRanks + static_cast<int>(threadIdx.x); r0 < end; r0 += 4 * kThreads) {   // four independent chains of gathers per thread in flight
        int hi[4], id[4]; double top[4], rv[4]; float2 x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = r0 + j * kThreads;
            const bool ok = r < end;
            hi[j] = ok && r >= h ? blk[r] : 0;
            x[j] = ok ? by_rank[r] : make_float2(0.f, 0.f); rv[j] = ok ? rho[r] : 0.0; id[j] = ok ? order[r] : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int r = r0 + j * kThreads; hi[j] = (r < h || r >= end) ? h : blo[hi[j] + 1]; }
#pragma unroll
        for (int j = 0; j < 4; ++j) top[j] = Q[hi[j]] / stot;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = r0 + j * kThreads;
            if (r < end) {
                const double t = val.p(x[j].x) - rv[j];
                const double gauge = (r < h) ? ipow(top[j], n) / info.res_total : 1.0;
                weight[r] = (t > 0.0) ? gauge * t / pow_diff(top[j], val.q(x[j].y) / stot, n) : 0.0;
                rho_id[id[j]] = rv[j];
            }
        }
    }
}

// Workgroups of 1024 threads take rows of more than two of the sort's tiles of 4096 tokens; shorter rows would leave most of one
// idle.  One of them fills a compute unit, so where rows wait for one (more of them than compute units) and a nucleus cut
// leaves little to sort, the row must be longer (cut of 1e-3; 1024 against 256 threads, the call when one kernel ordered the whole row): 1024 rows of
// 8193 tokens 795 and 707 us, of 12289 840 and 779, of 16384 959 and 950, of 24000 968 and 1010, of 50021 1504 and 1725.
// Rows of more than kLongRow tokens sort their candidates in tiles of eight elements per thread: half the barriers, twice the run; a shorter row loses more to
// its last tile.  The call, four / eight: 1024 rows of 128256 tokens with a nucleus cut of 1e-8 11602 / 11359 us, 256 of them with a top-k of 1000 1493 / 1342.
constexpr int kLongRow = 65536;
constexpr int scatter_lds(int threads, int buckets) { return 8 * threads * static_cast<int>(sizeof(Element) + sizeof(unsigned short)) + buckets * 16; }
// The LDS of the kernel that moves the elements lies above the default limit.
hipError_t full_kernel_setup() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(full_scatter_kernel<1024>), hipFuncAttributeMaxDynamicSharedMemorySize,
                               scatter_lds(1024, 1 << kLogBuckets));
}
static void launch_full_order(const FullParams& fp, hipStream_t stream) {
    const bool crowded = fp.tail_mass > 0.0 && fp.B > 256 && fp.V <= 16384;
    const bool small = fp.V <= 8192 || crowded;
    if (fp.k < fp.V || fp.tail_mass > 0.0) {
        if (fp.V > kLongRow) hipLaunchKernelGGL((full_support_kernel<1024, true, 8>), dim3(fp.B), dim3(1024), 0, stream, fp);
        else if (!small) hipLaunchKernelGGL((full_support_kernel<1024, true>), dim3(fp.B), dim3(1024), 0, stream, fp);
        else hipLaunchKernelGGL((full_support_kernel<kThreads, true>), dim3(fp.B), dim3(kThreads), 0, stream, fp);
    } else if (!small) hipLaunchKernelGGL((full_support_kernel<1024, false>), dim3(fp.B), dim3(1024), 0, stream, fp);
    else hipLaunchKernelGGL((full_support_kernel<kThreads, false>), dim3(fp.B), dim3(kThreads), 0, stream, fp);
    const int buckets = 1 << log_buckets(fp.V);
    auto slices = [&](int groups, int least) { return std::max(1, std::min(std::min(kMaxSlices, groups / fp.B), fp.V / least)); };
    const int count = small ? slices(2048, 1024) : slices(1024, 4096);
    const int len = (fp.V + count - 1) / count;
    hipLaunchKernelGGL(full_count_kernel, dim3(chunk_grid(fp.B, count)), dim3(kCountThreads), buckets * 16 + ((1 << kLogCells) + 1) * 4, stream, fp, count, len, buckets);
    if (small) hipLaunchKernelGGL(full_scatter_kernel<kThreads>, dim3(chunk_grid(fp.B, count)), dim3(kThreads), scatter_lds(kThreads, buckets), stream, fp, count, len, buckets);
    else hipLaunchKernelGGL(full_scatter_kernel<1024>, dim3(chunk_grid(fp.B, count)), dim3(1024), scatter_lds(1024, buckets), stream, fp, count, len, buckets);
    hipLaunchKernelGGL(full_bucket_kernel, dim3(chunk_grid(fp.B, buckets)), dim3(kBucketThreads), 0, stream, fp, buckets);
}

void launch_full_prologue(const FullParams& fp, hipStream_t stream) {
    launch_full_order(fp, stream);
    const int chunks = (fp.V + kChunkRanks - 1) / kChunkRanks;
    hipLaunchKernelGGL(full_scan_kernel, dim3(fp.B), dim3(kScanThreads), 0, stream, fp);
    if (fp.V > 8192) hipLaunchKernelGGL(full_trunc_kernel<1024>, dim3(fp.B), dim3(1024), 0, stream, fp);
    else hipLaunchKernelGGL(full_trunc_kernel<kThreads>, dim3(fp.B), dim3(kThreads), 0, stream, fp);
    hipLaunchKernelGGL(full_dense_kernel, dim3(chunk_grid(fp.B, chunks)), dim3(kThreads), kChunkLds, stream, fp, chunks);
}

}  // namespace gr
