// Acceptance-only sweep: alpha*(k, n) = 1 + min_H psi(H) (Thm 3.1) for a grid of top-k sizes and numbers
// of i.i.d. drafts, per row, behind ONE streaming selection pass over p and q (with the largest k of
// the grid).  Sec. 5.1: the minimiser is a prefix of the order by decreasing q/p; for a smaller top-k
// the support is the first k tokens by decreasing q (App. "Top-k Sampling for the Relaxed OTLP") and
// its ratio order is the sub-sequence of the largest support's order, so one ordering serves the grid.
//
// One workgroup per row, everything in LDS: its 1024 threads share the comparisons of the ranks, then a wave takes each top-k size.
// Only the minimum of F(m) = P_m - Q_m^n is reported, to 1e-5, so the prefix sums here are parallel
// scans in float64 (no integer decision hangs on their rounding).
// Bound: latency, a row's chain of LDS reads, scans and barriers; 256 threads to a row left most of a compute unit idle
// (256 rows, six sizes up to 256, ten draft counts: 44 us; 1024 threads 25.7, and 16.9 with a wave to a size).
#include <hip/hip_runtime.h>

#include "gr_internal.h"

namespace gr {

namespace {

constexpr int kSweepThreads = 1024, kGroups = kSweepThreads / kThreads;
static_assert(kThreads == kMaxSupport, "a thread of a group to a rank");

struct SweepLds {
    unsigned long long keys[kSelCap];     // merged slice candidates
    unsigned long long ckey[kMaxSupport]; // the kmax largest, unordered
    double pv[kMaxSupport]; double qv[kMaxSupport];   // by slot
    unsigned long long ratio[kMaxSupport];            // by slot: the pattern of q/p, which rises with it
    double rp[kMaxSupport]; double rq[kMaxSupport];   // by ratio rank: p / sum p, raw q
    int rqr[kMaxSupport];                 // by ratio rank: the token's rank by decreasing q
    int ids[kMaxSupport];
    int rank[2][kMaxSupport];             // by slot: the ranks by decreasing q and by decreasing q/p
    double least[kSweepMaxK][kSweepMaxDrafts];   // per top-k size and draft count: the minimum of F
    int hist[256]; int pick[4]; int count;
};

// Inclusive sums of a over the lanes of a wave.
__device__ __forceinline__ double wave_scan(double a) {
    a += dpp_shift<0x111, 0xF>(a, 0.0);
    a += dpp_shift<0x112, 0xF>(a, 0.0);
    a += dpp_shift<0x114, 0xF>(a, 0.0);
    a += dpp_shift<0x118, 0xF>(a, 0.0);
    a += dpp_shift<0x142, 0xA>(a, 0.0);
    a += dpp_shift<0x143, 0xC>(a, 0.0);
    return a;
}
__global__ __launch_bounds__(kSweepThreads) void sweep_kernel(SweepParams sw) {
    constexpr int NT = kSweepThreads;
    __shared__ SweepLds L;
    const int tid = threadIdx.x, row = blockIdx.x, m = tid & (kThreads - 1), group = tid / kThreads;
    const int cells = sw.nk * sw.nn;
    float* out = sw.accept_prob + static_cast<size_t>(row) * cells;

    // ---- merge the slices (same per-slice records as the solve kernel reads)
    const SliceTotals found = slice_totals<false>(sw.cand_count, sw.part_bad, sw.part_psum, sw.part_qsum, nullptr, row, sw.splits, 0.0);
    const int total = found.total;
    const double ptot = found.ptot, qtot = found.qtot;
    if (found.bad || !(fabs(ptot - 1.0) <= 1e-3) || !(fabs(qtot - 1.0) <= 1e-3) || total <= 0 || total > kSelCap) {
        for (int c = tid; c < cells; c += NT) out[c] = __uint_as_float(0x7fc00000u);
        if (tid == 0) sw.status[row] = GR_ROW_BAD;
        return;
    }
    gather_keys<NT>(L.keys, sw.cand + static_cast<size_t>(row) * kSelCap, found, sw.splits);
    if (tid == 0) L.count = 0;
    if (tid < kMaxSupport) { L.rank[0][tid] = 0; L.rank[1][tid] = 0; }
    __syncthreads();
    unsigned long long theta = 0ull;
    if (total > sw.kmax) theta = block_kth_largest<NT>(L.keys, total, sw.kmax, L.hist, L.pick);
    const int kk = min(total, sw.kmax);                       // <= kMaxSupport = kThreads
    for (int i = tid; i < total; i += NT) {
        const unsigned long long key = L.keys[i];
        if (key >= theta) {
            const int slot = atomicAdd(&L.count, 1);
            if (slot < kMaxSupport) L.ckey[slot] = key;
        }
    }
    __syncthreads();
    // ---- per slot: token id, q, p; rank by decreasing q (keys are distinct: ties go to the lower id).  A group compares
    // with its share of the slots.
    const int each = (kk + kGroups - 1) / kGroups, j0 = group * each, j1 = min(kk, j0 + each);
    if (m < kk) {
        const unsigned long long mine = L.ckey[m];
        if (group == 0) {
            const int id = key_id(mine);
            L.ids[m] = id;
            const double q = static_cast<double>(key_q(mine)), p = static_cast<double>(sw.p[static_cast<size_t>(row) * sw.V + id]);
            L.qv[m] = q; L.pv[m] = p;
            L.ratio[m] = static_cast<unsigned long long>(__double_as_longlong(p > 0.0 ? q / p : __builtin_inf()));
        }
        int before = 0;
#pragma unroll 8
        for (int j = j0; j < j1; ++j) before += static_cast<int>(L.ckey[j] > mine);
        atomicAdd(&L.rank[0][m], before);
    }
    __syncthreads();
    // ---- rank by decreasing q/p, ties by id: the quotients of different float32 ratios differ by 2^-48 relative at least, so rounded to
    // float64 they keep the order of the exact cross products (which took two products more per pair)
    if (m < kk) {
        const unsigned long long mine = L.ratio[m];
        const int id = L.ids[m];
        int before = 0;
#pragma unroll 8
        for (int j = j0; j < j1; ++j) {
            const unsigned long long other = L.ratio[j];
            before += static_cast<int>(other > mine) | (static_cast<int>(other == mine) & static_cast<int>(L.ids[j] < id));
        }
        atomicAdd(&L.rank[1][m], before);
    }
    __syncthreads();
    if (tid < kk) {
        const int rank = L.rank[1][tid];
        L.rp[rank] = L.pv[tid] / ptot; L.rq[rank] = L.qv[tid]; L.rqr[rank] = L.rank[0][tid];
    }
    __syncthreads();
    // ---- the grid, a wave to a top-k size: masked prefix sums along the order, four ranks to a lane, and the best prefix for every draft count, by one
    // chain of powers.  (A rank to a thread of four groups, which took the sizes in turn, a power from scratch for every draft count: 25.7 us for 256
    // rows, six sizes up to 256 and ten draft counts, 16.9 now.)
    const int lane = tid & 63, a = tid >> 6;
    if (a < sw.nk) {
        constexpr int E = kMaxSupport / 64;
        const int top = sw.ks[a];
        double P[E], S[E], Q[E], pw[E], ps = 0.0, ss = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = E * lane + e;
            const bool on = r < kk && L.rqr[min(r, kMaxSupport - 1)] < top;
            ps += on ? L.rp[r] : 0.0; ss += on ? L.rq[r] : 0.0;
            P[e] = ps; S[e] = ss;
        }
        const double pi = wave_scan(ps), si = wave_scan(ss), total_s = read_lane(si, 63);   // positive: the largest q is
        // a rank outside this support, and one beyond the last, repeats the prefix before it
#pragma unroll
        for (int e = 0; e < E; ++e) { P[e] += pi - ps; Q[e] = (S[e] + (si - ss)) / total_s; pw[e] = Q[e]; }
        unsigned long long left = sw.nmask;
        for (int n = 1;; ++n) {
            if (left & 1ull) {
                const double low = wave_min(fmin(fmin(fmin(P[0] - pw[0], P[1] - pw[1]), fmin(P[2] - pw[2], P[3] - pw[3])), 0.0));   // F(0) = 0
                if (lane == 0) L.least[a][n - 1] = low;
            }
            left >>= 1;
            if (left == 0ull) break;
#pragma unroll
            for (int e = 0; e < E; ++e) pw[e] = __dmul_rn(pw[e], Q[e]);
        }
        static_assert(E == 4, "four ranks to a lane");
    }
    __syncthreads();
    for (int c = tid; c < cells; c += NT) out[c] = static_cast<float>(1.0 + L.least[c / sw.nn][sw.ns[c % sw.nn] - 1]);
    if (tid == 0) sw.status[row] = GR_ROW_OK;
}

}  // namespace

hipError_t launch_sweep(const SweepParams& sw, int B, hipStream_t stream) {
    hipLaunchKernelGGL(sweep_kernel, dim3(B), dim3(kSweepThreads), 0, stream, sw);
    return hipGetLastError();
}

}  // namespace gr
