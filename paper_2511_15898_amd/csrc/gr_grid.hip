// Acceptance grid over supports that do not fit LDS (the first experiment of Sec. 7 runs the top-k size up to the whole vocabulary): the
// minimum over prefixes of the ratio order of F(m) = P_m - Q_m^n (Thm 3.1, Sec. 5.1) for every top-k size and draft count, without
// that order.
//
// The tokens of a row go into bins by their ratio q/p, with sums of p and q per bin and top-k size.  F at the bins' edges needs no more;
// inside a bin the slope p/q of the path m -> (Q_m, P_m) rises within the bin's own bounds, so P lies above two lines, one from each
// end, and F, which is concave along a line, above its value where they meet.  A bin that may hold a smaller F than the best edge is cut
// again, with the bins of a round shared out to all such intervals, until none is left; the tokens of one ratio are one line, so an
// interval of one ratio never is.  Rows of language models end after one round, or two where the draft is almost the target.
//
// Sums are of whole numbers of 2^-62 (p and q sum to 1.001 at most), so the result does not depend on the order of the additions.  The acceptance's error
// against sums of more bits, n = 1 and 8, rows of 300 to 128256 tokens of eight kinds (targets and drafts of language models, cooled, near one another, apart
// down to acceptances of 1e-10): 1e-16 to 1.4e-15, as far as float64 carries P - Q^n; sums in float64 along the order 2e-16 to 4e-15, whole numbers cut
// off below the unit up to 6e-14.
//
// One workgroup per row.  Bound: instruction issue of the third of three passes over the row (class, ratio, bin and three LDS additions per token), which takes
// half of the launch; the first runs at the memory's rate.  Two radix sorts per row (by q/p and by q), gathers and masked prefix scans took 3877 us for 256
// rows of 128256 tokens, six sizes and ten draft counts, this 258 of a kernel trace, 210 to 266 the call on different cards.  The call with sorts and now: 256
// rows whose drafts are almost the target 4082 and 516 us, of 8192 tokens 336 and 90, one row of 128256 tokens 1773 and 156, of 300 tokens and one size 46 and 22, with
// eight sizes and eight draft counts 50 and 35.  Slower than the sorts where many cells meet few tokens: that row with twelve counts and a draft that is almost
// the target 51 and 53, 1024 rows of 300 tokens with eight sizes and 16 counts 134 and 143 (eight counts 129 and 127).
#include "gr_internal.h"

namespace gr {

namespace {

constexpr int kNT = 1024, kNW = kNT / 64;
constexpr int kBins = 512, kBinsLog = 9;
constexpr int kMaxOpen = 64;                       // intervals cut in one round: eight bins each at least
constexpr int kClasses = 2048;                     // of q: exponent and four bits of the mantissa
constexpr int kList = 8192;                        // keys that the search for the top-k thresholds holds in LDS
constexpr unsigned long long kInf = 0x7ff0000000000000ull;

constexpr int kMaxHeavy = 2048;                   // so many tokens of the classes of largest q at most are kept at hand
constexpr int kItems = kSweepMaxK * kBins / kNT;   // bins of a thread, one of every other top-k size

// The place of a digit's counter: the lanes that look for a digit each own a run of them.
__host__ __device__ constexpr int padded(int digit) { return digit + (digit >> 5); }

// An interval of the order's keys that is still open: [lo, hi), and what lies before it of every top-k size.
struct Interval { unsigned long long lo, hi, tokens; double P[kSweepMaxK], Q[kSweepMaxK]; };
static_assert(sizeof(Interval) <= 2 * kFullBytesPerToken, "an interval holds two tokens at least: their bytes of the workspace hold it");

struct GridLds {
    union {
        // per top-k size and bin: sums in units of 2^-62, then P and Q at the bin's last place (rows padded: the sizes of a bin lie in different banks)
        struct { union { unsigned long long sum[2][kSweepMaxK][kBins + 2]; double at[2][kSweepMaxK][kBins + 2]; }; int count[kSweepMaxK][kBins]; };
        struct { unsigned long long keys[kList]; int hist[kSweepMaxK][padded(256)]; int classes[padded(kClasses)]; };   // classes: the wanted ones, once counted
    };
    Element heavy[kMaxHeavy];
    Interval open[kMaxOpen];
    int shift[kMaxOpen];                           // bin of a key of open[i]: (key - lo) >> shift[i]
    unsigned long long prefix[kSweepMaxK];         // the search: the threshold's digits so far; then the thresholds
    int need[kSweepMaxK], bucket[kSweepMaxK];
    double best[kSweepMaxK][kSweepMaxN], limit[kSweepMaxK][kSweepMaxN];   // limit: what a smaller F has to be below
    double low[kSweepMaxN][kNW][16];               // of a wave's groups of four lanes
    double mass[kSweepMaxK], inv_mass[kSweepMaxK];
    double red[kNW];
    int flag[kBins];
    int wcount[kNW];
    int listed, heavies, inside, heavy_class;
};

// The order's key of a token: rising keys are falling ratios; p = 0 gives +inf, which comes first.  The quotient is rounded correctly, so two
// different ratios of float32 values have different keys.
__device__ __forceinline__ unsigned long long ratio_key(float q, float p) {
    const double r = p > 0.f ? static_cast<double>(q) / static_cast<double>(p) : __builtin_inf();
    return kInf - static_cast<unsigned long long>(__double_as_longlong(r));
}
// Whether what a token's values have below a unit counts as one: even over the tokens, the same for a token at every look.
__device__ __forceinline__ float odds_of(int id) { return static_cast<float>(static_cast<unsigned>(id) * 0x9E3779B1u) * 0x1p-32f; }
// v in units of 2^-62, v in [0, 2).  Values of 2^-39 and more are whole; the fraction that a smaller one leaves counts as a unit with that probability,
// so that a sum of many small values errs by half a unit times the root of their number, and not by half a unit each.
__device__ __forceinline__ unsigned long long fixed62(float v, float odds) {
    const float a = v * 0x1p30f, t = __builtin_amdgcn_fractf(a) * 0x1p32f;            // both exact
    return (static_cast<unsigned long long>(static_cast<unsigned>(a)) << 32) + static_cast<unsigned>(t) + (__builtin_amdgcn_fractf(t) > odds);
}
// Bins of the first round, by the ratio's place x in 32nds of an octave: 32 to an octave from 2^-5 to 2^5, where thresholds lie (a token is taken up to
// a ratio of about 1 / n, in the support's own scale), two to an octave out to 2^-53 and 2^52, one for what lies beyond on either side, and one for
// the ratios that are not finite.
__device__ __forceinline__ int bin_of(int x) {
    const int u = x < -160 ? max(0, 96 + ((x + 160) >> 4)) : (x < 160 ? 256 + x : min(510, 416 + ((x - 160) >> 4)));
    return kBins - 1 - u;
}
__device__ __forceinline__ int first_bin(unsigned long long key) {
    const unsigned long long r = kInf - key;
    return r == kInf ? 0 : bin_of(static_cast<int>(r >> 47) - (1023 << 5));
}
// The same from a float32 quotient of a few units in the last place, where that cannot lie on the other side of an edge; -1 where it might.
__device__ __forceinline__ int quick_bin(float q, float p) {
    const unsigned r = __float_as_uint(q * __builtin_amdgcn_rcpf(p));
    const bool sure = min(__float_as_uint(p), __float_as_uint(q)) > 0x0d800000u && ((r + 8u) & 0x3FFFFu) > 16u;   // both above 2^-100
    return sure ? bin_of(static_cast<int>(r >> 18) - (127 << 5)) : -1;
}
// The smallest pattern of a ratio in bin u (counted by rising ratios), 0..kBins.
__device__ __forceinline__ unsigned long long first_edge(int u) {
    if (u <= 0) return 0ull;
    if (u >= 511) return u == 511 ? kInf : kInf + 1ull;
    const int x = u < 96 ? 16 * (u - 96) - 160 : (u < 416 ? u - 256 : 16 * (u - 416) + 160);
    return static_cast<unsigned long long>(x + (1023 << 5)) << 47;
}

// Every token of a row: f(p, q, id).  Long rows: four to a thread and step, two steps in flight where vectors can read them.  A short row takes
// one copy of f for all of its tokens: it waits for instructions that no wave has fetched before more than for anything else (one row of 300 tokens,
// eight sizes and eight draft counts 55 us with the long rows' loops, 42 with this one; 256 rows of 128256 tokens 313 us with this one).
constexpr int kFewTokens = 16384;
template <bool P, class F>
__device__ __forceinline__ void each_token(const float* pr, const float* qr, int V, F f) {
    const int tid = threadIdx.x;
    if (V <= kFewTokens) {
        float p = 0.f, q = 0.f;
        if (tid < V) { if (P) p = pr[tid]; q = qr[tid]; }
#pragma unroll 1
        for (int i = tid; i < V; i += kNT) {
            const float pv = p, qv = q;
            if (i + kNT < V) { if (P) p = pr[i + kNT]; q = qr[i + kNT]; }
            f(pv, qv, i);
        }
        return;
    }
    if (((reinterpret_cast<size_t>(pr) | reinterpret_cast<size_t>(qr)) & 15u) == 0) {
        const int whole = V & ~3;
        constexpr int U = 2;
        for (int i0 = 4 * tid; i0 < whole; i0 += U * 4 * kNT) {
            float4 a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * 4 * kNT;
                if (i < whole) { if (P) a[u] = *reinterpret_cast<const float4*>(pr + i); b[u] = *reinterpret_cast<const float4*>(qr + i); }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = i0 + u * 4 * kNT;
                if (i < whole) {
                    f(P ? a[u].x : 0.f, b[u].x, i); f(P ? a[u].y : 0.f, b[u].y, i + 1);
                    f(P ? a[u].z : 0.f, b[u].z, i + 2); f(P ? a[u].w : 0.f, b[u].w, i + 3);
                }
            }
        }
        if (whole + tid < V) f(P ? pr[whole + tid] : 0.f, qr[whole + tid], whole + tid);
        return;
    }
    for (int i0 = tid; i0 < V; i0 += 4 * kNT) {
        float a[4], b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int i = i0 + j * kNT; a[j] = P && i < V ? pr[i] : 0.f; b[j] = i < V ? qr[i] : 0.f; }
#pragma unroll
        for (int j = 0; j < 4; ++j) if (i0 + j * kNT < V) f(a[j], b[j], i0 + j * kNT);
    }
}

// One more at a counter in LDS, for the lanes that are here: by one of them where all name the same (flat drafts).
__device__ __forceinline__ void count_one(int* counters, int at) {
    const unsigned long long here = __ballot(true);
    if (__ballot(at == __builtin_amdgcn_readfirstlane(at)) != here) atomicAdd(&counters[at], 1);
    else if ((threadIdx.x & 63) == __ffsll(static_cast<long long>(here)) - 1) atomicAdd(&counters[at], __popcll(here));
}

// One wave: the digit of `hist` (DIGITS of them) that holds the need-th largest key; returns it, with the keys still needed from it and
// how many it holds.
template <int DIGITS>
__device__ __forceinline__ int pick_digit(const int* hist, int& need, int& holds) {
    constexpr int PER = DIGITS / 64;
    const int lane = threadIdx.x & 63;
    int c[PER], tot = 0;                           // lane l owns the digits from DIGITS - 1 - PER l downwards
#pragma unroll
    for (int j = 0; j < PER; ++j) { c[j] = hist[padded(DIGITS - 1 - PER * lane - j)]; tot += c[j]; }
    const int incl = wave_scan_i(tot), excl = incl - tot;
    int digit = 0, left = 0, here = 0;
    if (excl < need && need <= incl) {
        int above = excl;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (here == 0 && need <= above + c[j]) { digit = DIGITS - 1 - PER * lane - j; here = c[j]; left = need - above; }
            above += c[j];
        }
    }
    const int src = __ffsll(static_cast<long long>(__ballot(here > 0))) - 1;
    need = __builtin_amdgcn_readlane(left, src);
    holds = __builtin_amdgcn_readlane(here, src);
    return __builtin_amdgcn_readlane(digit, src);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_step(unsigned long long& v) {
    const int lo = dpp_shift<CTRL, ROWS>(static_cast<int>(v), 0), hi = dpp_shift<CTRL, ROWS>(static_cast<int>(v >> 32), 0);
    v += (static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) | static_cast<unsigned>(lo);
}

// x, x^2, ... up to the grid's largest draft count, the products that ipow takes, of every item: g(slot) at each draft count of the grid.
template <int N, class G>
__device__ __forceinline__ void powers(const GridParams& gp, const double (&x)[N], double (&pw)[N], G g) {
    unsigned long long left = gp.nmask;            // bit n - 1: n is in the grid
#pragma unroll
    for (int i = 0; i < N; ++i) pw[i] = x[i];
#pragma unroll 1
    for (int slot = 0, more = 63 - __builtin_clzll(left);; --more) {
        if (left & 1ull) { g(slot); ++slot; }
        if (more == 0) break;
        left >>= 1;
#pragma unroll
        for (int i = 0; i < N; ++i) pw[i] = __dmul_rn(pw[i], x[i]);
    }
}

}  // namespace

__global__ __launch_bounds__(kNT) void grid_kernel(GridParams gp) {
    extern __shared__ __align__(16) unsigned char grid_lds[];
    GridLds& S = *reinterpret_cast<GridLds*>(grid_lds);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int V = gp.V, nk = gp.nk, nn = gp.nn, slots = __popcll(gp.nmask);
    const float* pr = gp.p + static_cast<size_t>(row) * V;
    const float* qr = gp.q + static_cast<size_t>(row) * V;
    Interval* stack = reinterpret_cast<Interval*>(gp.work + row * gp.work_stride);

    // sums, validity, positive entries of q by magnitude
    for (int c = tid; c < padded(kClasses); c += kNT) S.classes[c] = 0;
    if (tid == 0) { S.listed = 0; S.heavies = 0; }
    __syncthreads();
    double ps = 0.0, qs = 0.0;
    int bad = 0, positive = 0;
    each_token<true>(pr, qr, V, [&](float pv, float qv, int) {
        bad |= !(qv >= 0.f) | !(pv >= 0.f);
        ps += static_cast<double>(pv); qs += static_cast<double>(qv);
        if (qv > 0.f) { ++positive; count_one(S.classes, padded(min(__float_as_uint(qv) >> 19, kClasses - 1u))); }
    });
    const double ptot = block_sum<kNW>(ps, S.red), qtot = block_sum<kNW>(qs, S.red);
    bad = block_sum_i<kNW>(bad, S.red);
    positive = block_sum_i<kNW>(positive, S.red);
    if (bad || !(fabs(ptot - 1.0) <= 1e-3) || !(fabs(qtot - 1.0) <= 1e-3)) {
        for (int c = tid; c < nk * nn; c += kNT) gp.accept_prob[static_cast<size_t>(row) * nk * nn + c] = __uint_as_float(0x7fc00000u);
        if (tid == 0) gp.status[row] = GR_ROW_BAD;
        return;
    }

    // the smallest key (q, then the lower id) of each top-k size, by radix selection: the classes first, then eight bits at a time over the
    // keys of the classes that thresholds fall into, from LDS where they fit and from the row where not
    if (wv <= nk) {                                // the last of these waves: the classes above that of the first key that has no place at hand
        const int rank = wv < nk ? gp.ks[wv] : kMaxHeavy + 1;
        const bool there = wv < nk ? rank < positive : rank <= positive;   // a size of every token has no threshold
        int need = rank, holds = rank, digit = 0;
        if (there) digit = pick_digit<kClasses>(S.classes, need, holds);
        if (lane == 0) {
            if (wv < nk) { S.prefix[wv] = static_cast<unsigned long long>(digit) << 51; S.need[wv] = need; S.bucket[wv] = holds; }
            else S.heavy_class = there ? digit + 1 : 0;
        }
    }
    __syncthreads();
    unsigned open = 0u;                            // the sizes whose threshold is not found yet
    for (int a = 0; a < nk; ++a) if (S.bucket[a] != S.need[a]) open |= 1u << a;
    if (open) {
        int keys = 0;
        unsigned long long last = ~0ull;               // sizes rise, so equal classes are neighbours
        for (int a = 0; a < nk; ++a)
            if (open >> a & 1u) { const unsigned long long c = S.prefix[a]; if (c != last) keys += S.bucket[a]; last = c; }
        const bool listed = keys <= kList;
        unsigned long long thr[kSweepMaxK];
        if (listed) {
            for (int c = tid; c < padded(kClasses); c += kNT) S.classes[c] = 0;
            __syncthreads();
            if (tid < nk && (open >> tid & 1u)) S.classes[padded(static_cast<int>(S.prefix[tid] >> 51))] = 1;
            __syncthreads();
            each_token<false>(pr, qr, V, [&](float, float qv, int id) {
                if (S.classes[padded(min(__float_as_uint(qv) >> 19, kClasses - 1u))] && qv > 0.f) S.keys[atomicAdd(&S.listed, 1)] = make_key(qv, id);
            });
            __syncthreads();
        }
        for (int shift = 51; open && shift > 0;) {
            const int width = min(8, shift), above = shift;
            shift -= width;
            for (int c = tid; c < kSweepMaxK * padded(256); c += kNT) (&S.hist[0][0])[c] = 0;
            __syncthreads();
            // sizes whose thresholds agree so far (neighbours, as the sizes rise) share the counters of the first of them
            int lead = 0, my_lead = 0;
            unsigned long long last = ~0ull;
#pragma unroll
            for (int a = 0; a < kSweepMaxK; ++a) {
                thr[a] = ~0ull;
                if (a < nk && (open >> a & 1u)) {
                    const unsigned long long t = S.prefix[a] >> above;
                    if (t != last) { thr[a] = t; lead = a; last = t; }
                    if (a == wv) my_lead = lead;
                }
            }
            auto add = [&](unsigned long long key) {
                const int d = static_cast<int>(key >> shift) & 255 & ((1 << width) - 1);
#pragma unroll
                for (int a = 0; a < kSweepMaxK; ++a) if (key >> above == thr[a]) count_one(S.hist[a], padded(d));
            };
            if (listed) { for (int i = tid; i < keys; i += kNT) add(S.keys[i]); }
            else each_token<false>(pr, qr, V, [&](float, float qv, int id) { if (qv > 0.f) add(make_key(qv, id)); });
            __syncthreads();
            if (wv < nk && (open >> wv & 1u)) {
                int need = S.need[wv], holds = 0;
                const int d = pick_digit<256>(S.hist[my_lead], need, holds);
                if (lane == 0) { S.prefix[wv] |= static_cast<unsigned long long>(d) << shift; S.need[wv] = need; S.bucket[wv] = holds; }
            }
            __syncthreads();
            open = 0u;
            for (int a = 0; a < nk; ++a) if (S.bucket[a] != S.need[a]) open |= 1u << a;
        }
    }
    unsigned thr_q[kSweepMaxK], thr_id[kSweepMaxK];            // the same in every lane: scalar registers
#pragma unroll
    for (int a = 0; a < kSweepMaxK; ++a) {
        const unsigned long long t = a < nk ? S.prefix[a] : 0ull;
        thr_q[a] = __builtin_amdgcn_readfirstlane(static_cast<int>(t >> 32)); thr_id[a] = __builtin_amdgcn_readfirstlane(static_cast<int>(t));
    }
    // the smallest top-k size that holds a token; nk: none.  A size of all tokens has the threshold 0, and so have those that the grid does not use: no
    // positive entry is below it.
    auto class_of = [&](float qv, int id) {
        const unsigned b = __float_as_uint(qv);
        int cls = 0;
        bool ties = false;
        auto compare = [&](int from, int to) {
#pragma unroll
            for (int a = from; a < to; ++a) { cls += b < thr_q[a]; ties |= b == thr_q[a]; }
        };
        compare(0, 2);
        if (nk > 2) compare(2, 4);
        if (nk > 4) compare(4, kSweepMaxK);
        if (ties) {
            const unsigned low = 0xFFFFFFFFu - static_cast<unsigned>(id);
#pragma unroll
            for (int a = 0; a < kSweepMaxK; ++a) cls += b == thr_q[a] && low < thr_id[a];
        }
        return qv > 0.f ? cls : nk;
    };
    auto add = [&](int cls, int bin, float pv, float qv, int id) {
        const float odds = odds_of(id);
        atomicAdd(&S.sum[0][cls][bin], fixed62(pv, odds));
        atomicAdd(&S.sum[1][cls][bin], fixed62(qv, odds));
        atomicAdd(&S.count[cls][bin], 1);
    };
    for (int c = tid; c < kSweepMaxK * kSweepMaxN; c += kNT) (&S.best[0][0])[c] = 0.0;   // F(0) = 0: the empty prefix
    const double invp = 1.0 / ptot;
    const int heavy_class = S.heavy_class;
    constexpr double kUnit = 1.0 / 4611686018427387904.0;      // 2^-62

    int waiting = 0;                               // intervals on the stack, the one of smallest keys on top
    for (int taken = 0;; ) {                       // intervals of this round; 0: the first, over all keys
        const int log_per = taken ? kBinsLog - (31 - __clz(2 * taken - 1)) : kBinsLog;
        __syncthreads();
        static_assert((kBins + 2) % 2 == 0 && kBins % 4 == 0, "whole vectors");
        for (int c = tid; c < nk * (kBins + 2) / 2; c += kNT) {
            reinterpret_cast<ulonglong2*>(S.sum[0])[c] = make_ulonglong2(0ull, 0ull); reinterpret_cast<ulonglong2*>(S.sum[1])[c] = make_ulonglong2(0ull, 0ull);
        }
        for (int c = tid; c < nk * kBins / 4; c += kNT) reinterpret_cast<int4*>(S.count)[c] = make_int4(0, 0, 0, 0);
        if (tid < taken) {
            const unsigned long long width = S.open[tid].hi - S.open[tid].lo - 1ull;
            S.shift[tid] = max(0, (width ? 64 - __clzll(static_cast<long long>(width)) : 0) - log_per);
        }
        __syncthreads();
        if (!taken) {
            each_token<true>(pr, qr, V, [&](float pv, float qv, int id) {
                const int cls = class_of(qv, id);
                if (cls >= nk) return;
                int bin = quick_bin(qv, pv);
                if (bin < 0) bin = first_bin(ratio_key(qv, pv));
                add(cls, bin, pv, qv, id);
                if (static_cast<int>(__float_as_uint(qv) >> 19) >= heavy_class) S.heavy[min(atomicAdd(&S.heavies, 1), kMaxHeavy - 1)] = Element{pv, qv, id};   // they fit
            });
        } else {
            const unsigned long long from = S.open[0].lo, to = S.open[taken - 1].hi;
            // the open interval of a token's key, -1: none
            auto interval = [&](unsigned long long key) {
                if (key < from || key >= to) return -1;
                int i = 0;                         // the last one that begins at the key or before it
                for (int step = kMaxOpen / 2; step > 0; step >>= 1) if (i + step < taken && S.open[i + step].lo <= key) i += step;
                return key < S.open[i].hi ? i : -1;
            };
            auto put = [&](float pv, float qv, int id) {
                const int cls = class_of(qv, id);
                if (cls >= nk) return;
                const unsigned long long key = ratio_key(qv, pv);
                const int i = interval(key);
                if (i >= 0) add(cls, (i << log_per) + static_cast<int>((key - S.open[i].lo) >> S.shift[i]), pv, qv, id);
            };
            // Far from the thresholds a bin is wide, and one or two tokens of a large mass leave it open: those are at hand.  (One row of 256 needs
            // the round more often than not, and a pass over its row for it took a third of the launch again.)
            const int heavies = S.heavies;
            if (tid == 0) S.inside = 0;
            __syncthreads();
            for (int h = tid; h < heavies; h += kNT) {
                const Element e = S.heavy[h];
                if (class_of(e.q, e.id) < nk && interval(ratio_key(e.q, e.p)) >= 0) atomicAdd(&S.inside, 1);
            }
            __syncthreads();
            int tokens = 0;
            for (int i = lane; i < taken; i += 64) tokens += static_cast<int>(S.open[i].tokens);
            if (wave_sum_i(tokens) == S.inside) { for (int h = tid; h < heavies; h += kNT) { const Element e = S.heavy[h]; put(e.p, e.q, e.id); } }
            else each_token<true>(pr, qr, V, put);
        }
        __syncthreads();
        // every top-k size holds the tokens of the smaller ones: a thread adds up one bin's p or q
        {
            const int which = tid / kBins, j = tid % kBins;
            unsigned long long v[kSweepMaxK]; int c[kSweepMaxK];
#pragma unroll
            for (int a = 0; a < kSweepMaxK; ++a) { v[a] = a < nk ? S.sum[which][a][j] : 0ull; c[a] = which == 0 && a < nk ? S.count[a][j] : 0; }
#pragma unroll
            for (int a = 1; a < kSweepMaxK; ++a) {
                v[a] += v[a - 1]; c[a] += c[a - 1];
                if (a < nk) { S.sum[which][a][j] = v[a]; if (which == 0) S.count[a][j] = c[a]; }
            }
            if (which == 0) S.flag[j] = 0;
        }
        __syncthreads();
        // P and Q at every bin's last place: sums over the bins, a wave to a size and sum, from where the bin's interval begins
        if (wv < 2 * nk) {
            const int a = wv >> 1, which = wv & 1;
            unsigned long long carry = 0ull;
#pragma unroll 1
            for (int j = lane; j < kBins; j += 64) {
                unsigned long long v = S.sum[which][a][j];
                scan_step<0x111, 0xF>(v); scan_step<0x112, 0xF>(v); scan_step<0x114, 0xF>(v); scan_step<0x118, 0xF>(v);
                scan_step<0x142, 0xA>(v); scan_step<0x143, 0xC>(v);
                v += carry;
                carry = (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v >> 32), 63))) << 32) |
                        static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
                S.sum[which][a][j] = v;
            }
            if (!taken && which == 1) { const double m = static_cast<double>(carry) * kUnit; if (lane == 0) { S.mass[a] = m; S.inv_mass[a] = 1.0 / m; } }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
            const double scale = kUnit * (which == 0 ? invp : S.inv_mass[a]);
#pragma unroll 1
            for (int j = kBins - 64 + lane; j >= 0; j -= 64) {       // downwards: what lies before an interval is still a sum
                const int o = j >> log_per, from = o << log_per;
                unsigned long long v = S.sum[which][a][j];
                if (from > 0) v -= S.sum[which][a][from - 1];
                const double base = taken && o < taken ? (which == 0 ? S.open[o].P[a] : S.open[o].Q[a]) : 0.0;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier();
                S.at[which][a][j] = base + static_cast<double>(v) * scale;
            }
        }
        __syncthreads();
        // (P, Q) at the first place of a bin
        auto start = [&](int a, int j, double& p, double& q) {
            const int o = j >> log_per;
            if (j != o << log_per) { p = S.at[0][a][j - 1]; q = S.at[1][a][j - 1]; }
            else if (taken) { p = S.open[o].P[a]; q = S.open[o].Q[a]; }
            else { p = 0.0; q = 0.0; }
        };
        auto keys_of = [&](int j, unsigned long long& lo, unsigned long long& hi) {
            if (!taken) { const int u = kBins - 1 - j; lo = kInf + 1ull - first_edge(u + 1); hi = kInf + 1ull - first_edge(u); return; }
            const int i = j >> log_per;
            lo = S.open[i].lo + (static_cast<unsigned long long>(j & ((1 << log_per) - 1)) << S.shift[i]);
            hi = min(S.open[i].hi, lo + (1ull << S.shift[i]));
        };
        // F at the bins' last places, two waves to a top-k size: their lanes take four bins each, and a draft count's minimum goes over four lanes; all
        // others wait until the last count, as the loops over the counts are chains of one instruction's latency after the other (minima over the wave
        // and their limits read from LDS at every count: 1024 rows of 300 tokens, eight sizes and 16 counts 155 us, so 143; one row 39 and 37).
        if (wv < 2 * nk) {
            constexpr int PER = kBins / 128;
            double p[PER], x[PER], pw[PER];
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int j = 128 * i + 64 * (wv & 1) + lane;
                const bool in = (j >> log_per) < max(taken, 1);                // no interval behind the last one
                p[i] = in ? S.at[0][wv >> 1][j] : 1e300; x[i] = in ? S.at[1][wv >> 1][j] : 0.0;
            }
            powers(gp, x, pw, [&](int slot) {
                double m = p[0] - pw[0];
#pragma unroll
                for (int i = 1; i < PER; ++i) m = fmin(m, p[i] - pw[i]);
                m = fmin(m, dpp_move<kDppXor1>(m));
                m = fmin(m, dpp_move<kDppXor2>(m));
                if ((lane & 3) == 0) S.low[slot][wv][lane >> 2] = m;
            });
        }
        __syncthreads();
        {
            static_assert(kNT == 8 * kSweepMaxK * kSweepMaxN, "eight lanes to a size and draft count, four minima of the two waves' 32 to a lane");
            const int a = tid / (8 * kSweepMaxN), slot = tid / 8 % kSweepMaxN, part = tid % 8;
            const double* low = &S.low[slot][2 * a][0] + 4 * part;
            double m = fmin(fmin(low[0], low[1]), fmin(low[2], low[3]));
            m = fmin(m, dpp_move<kDppXor1>(m));
            m = fmin(m, dpp_move<kDppXor2>(m));
            m = fmin(m, dpp_move<kDppHalfMirror>(m));
            if (part == 0 && a < nk && slot < slots) {
                m = fmin(m, S.best[a][slot]);
                S.best[a][slot] = m;
                S.limit[a][slot] = m - (1e-13 * (1.0 + m) + 1e-16);   // what is not looked for is below 1e-13 of the acceptance
            }
        }
        __syncthreads();
        // bins that may hold less: a thread takes one bin of every other size
        {
            const int j = tid % kBins, odd = tid / kBins;
            unsigned long long lo = 0ull, hi = 0ull;
            if ((j >> log_per) < max(taken, 1)) keys_of(j, lo, hi);
            const double r0 = 1.0 / __longlong_as_double(static_cast<long long>(kInf - lo)), r1 = 1.0 / __longlong_as_double(static_cast<long long>(kInf + 1ull - hi));
            double px[kItems], qx[kItems], pw[kItems];
            bool some = false;
#pragma unroll
            for (int i = 0; i < kItems; ++i) {
                const int a = min(2 * i + odd, nk - 1);
                px[i] = 1e300; qx[i] = 0.0;
                if (hi - lo >= 2ull && S.count[a][j] >= 2) {
                    double p0, q0;
                    start(a, j, p0, q0);
                    const double scale = S.mass[a] * invp, s0 = scale * r0, s1 = scale * r1, dq = S.at[1][a][j] - q0, dp = S.at[0][a][j] - p0;
                    double x = s1 < 1e300 ? (s1 * dq - dp) / (s1 - s0) : dq;
                    x = fmin(fmax(x, 0.0), dq);
                    px[i] = p0 + s0 * x; qx[i] = q0 + x;
                    some = true;
                }
            }
            static_assert(kItems * kSweepMaxN == 64, "a wave's limits, one to a lane");
            const double limit = S.limit[min(2 * (lane / kSweepMaxN) + odd, nk - 1)][lane % kSweepMaxN];
            bool less = false;
            if (__any(some))
                powers(gp, qx, pw, [&](int slot) {
#pragma unroll
                    for (int i = 0; i < kItems; ++i) less |= px[i] - pw[i] < read_lane(limit, i * kSweepMaxN + slot);
                });
            if (less) S.flag[j] = 1;
        }
        __syncthreads();
        // onto the stack, in falling order of their keys
        const bool push = tid < kBins && S.flag[tid];
        const unsigned long long mask = __ballot(push);
        if (lane == 0) S.wcount[wv] = __popcll(mask);
        __syncthreads();
        int before = 0, all = 0;
        for (int w = 0; w < kBins / 64; ++w) { if (w < wv) before += S.wcount[w]; all += S.wcount[w]; }
        if (push) {
            Interval& t = stack[waiting + all - 1 - (before + __popcll(mask & ((1ull << lane) - 1ull)))];
            keys_of(tid, t.lo, t.hi);
            t.tokens = S.count[nk - 1][tid];
            for (int a = 0; a < nk; ++a) start(a, tid, t.P[a], t.Q[a]);
        }
        waiting += all;
        __syncthreads();
        if (waiting == 0) break;
        taken = min(waiting, kMaxOpen);
        constexpr int kWords = sizeof(Interval) / 8;
        for (int c = tid; c < taken * kWords; c += kNT) {
            const int i = c / kWords, w = c % kWords;
            reinterpret_cast<unsigned long long*>(&S.open[i])[w] = reinterpret_cast<const unsigned long long*>(&stack[waiting - 1 - i])[w];
        }
        waiting -= taken;
    }
    for (int c = tid; c < nk * kSweepMaxN; c += kNT) {
        const int a = c / kSweepMaxN, b = c % kSweepMaxN;
        if (b < nn) gp.accept_prob[(static_cast<size_t>(row) * nk + gp.kpos[a]) * nn + b] = static_cast<float>(1.0 + S.best[a][gp.slot[b]]);
    }
    if (tid == 0) gp.status[row] = GR_ROW_OK;
}

hipError_t grid_kernel_setup() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(grid_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(sizeof(GridLds)));
}

void launch_grid(const GridParams& gp, int B, hipStream_t stream) {
    hipLaunchKernelGGL(grid_kernel, dim3(B), dim3(kNT), sizeof(GridLds), stream, gp);
}

}  // namespace gr
