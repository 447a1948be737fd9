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
// Sums are whole numbers of 2^-62 (p and q sum to 1.001 at most): exact, so the result does not depend on the order of the additions.
//
// One workgroup per row.  Bound: three passes over the row (20 bytes a token; q alone in the second) and the LDS additions of the third.
// Two radix sorts per row (by q/p and by q), gathers and masked prefix scans took 3856 us for 256 rows of 128256 tokens, six sizes and ten draft
// counts; this takes 311 us.  256 rows whose drafts are almost the target 3630 -> 639, of 8192 tokens 324 -> 55, one row of 128256 tokens
// 1758 -> 181, of 300 tokens and one size 38.8 -> 14.3 us (and as long as before, 42 us, with eight sizes and eight draft counts).
#include "gr_internal.h"

namespace gr {

namespace {

constexpr int kNT = 1024, kNW = kNT / 64;
constexpr int kBins = 512, kBinsLog = 9;
constexpr int kMaxOpen = 64;                       // intervals cut in one round: eight bins each at least
constexpr int kClasses = 2048;                     // of q: exponent and four bits of the mantissa
constexpr int kList = 8192;                        // keys that the search for the top-k thresholds holds in LDS
constexpr unsigned long long kInf = 0x7ff0000000000000ull;

// An interval of the order's keys that is still open: [lo, hi), and what lies before it of every top-k size.
struct Interval { unsigned long long lo, hi, P[kSweepMaxK], Q[kSweepMaxK]; };
static_assert(sizeof(Interval) == 144, "two tokens of the workspace's 96 bytes hold one");

struct GridLds {
    union {
        struct { unsigned long long P[kSweepMaxK][kBins + 1], Q[kSweepMaxK][kBins + 1]; int count[kSweepMaxK][kBins]; };
        struct { unsigned long long keys[kList]; int hist[kSweepMaxK][256]; int classes[kClasses]; };
    };
    Interval open[kMaxOpen];
    int shift[kMaxOpen];                           // bin of a key of open[i]: (key - lo) >> shift[i]
    unsigned long long prefix[kSweepMaxK];         // the search: the threshold's digits so far; then the thresholds
    int need[kSweepMaxK], bucket[kSweepMaxK];
    double best[kSweepMaxK][kSweepMaxN];
    double cell[kSweepMaxN][kNW];
    double mass[kSweepMaxK];
    double red[kNW];
    int flag[kBins];
    int wcount[kNW];
    int listed;
};

// The order's key of a token: rising keys are falling ratios; p = 0 gives +inf, which comes first.  The quotient is rounded correctly, so two
// different ratios of float32 values have different keys.
__device__ __forceinline__ unsigned long long ratio_key(float q, float p) {
    const double r = p > 0.f ? static_cast<double>(q) / static_cast<double>(p) : __builtin_inf();
    return kInf - static_cast<unsigned long long>(__double_as_longlong(r));
}
// v in units of 2^-62, v in [0, 2).
__device__ __forceinline__ unsigned long long fixed62(float v) {
    const unsigned b = __float_as_uint(v);
    const int e = static_cast<int>(b >> 23) & 255;
    const unsigned long long m = (b & 0x7FFFFFu) | (e ? 0x800000u : 0u);
    const int s = max(e, 1) - 88;                  // 2^(e - 150) to 2^-62
    return s >= 0 ? m << s : m >> min(-s, 31);
}
// Bins of the first round, by the ratio's exponent e: 32 to an octave for -5 <= e < 5, where thresholds lie (a token is taken up to a ratio
// of about 1 / n, in the support's own scale), 4 up to 21, one to four octaves beyond, and one for the ratios that are not finite.
__device__ __forceinline__ int first_bin(unsigned long long key) {
    const unsigned long long r = kInf - key;
    const int e = static_cast<int>(r >> 52) - 1023;
    const int top5 = static_cast<int>(r >> 47) & 31;
    int u;
    if (e >= -5 && e < 5) u = 96 + (e + 5) * 32 + top5;
    else if (e < -21) u = max(0, 32 + ((e + 21) >> 2));
    else if (e < -5) u = 32 + (e + 21) * 4 + (top5 >> 3);
    else if (e < 21) u = 416 + (e - 5) * 4 + (top5 >> 3);
    else u = e < 1024 ? min(510, 480 + ((e - 21) >> 2)) : 511;
    return kBins - 1 - u;
}
// The smallest pattern of a ratio in bin u (counted by rising ratios), 0..kBins.
__device__ __forceinline__ unsigned long long first_edge(int u) {
    auto at = [](int e, unsigned long long sub) { return (static_cast<unsigned long long>(e + 1023) << 52) | sub; };
    if (u <= 0) return 0ull;
    if (u < 32) return at(-21 + 4 * (u - 32), 0ull);
    if (u < 96) return at(-21 + (u - 32) / 4, static_cast<unsigned long long>((u - 32) & 3) << 50);
    if (u < 416) return at(-5 + (u - 96) / 32, static_cast<unsigned long long>((u - 96) & 31) << 47);
    if (u < 480) return at(5 + (u - 416) / 4, static_cast<unsigned long long>((u - 416) & 3) << 50);
    if (u < 511) return at(21 + 4 * (u - 480), 0ull);
    return u == 511 ? kInf : kInf + 1ull;
}

// Every token of a row, four to a thread and step: f(p, q, id).
template <bool P, class F>
__device__ __forceinline__ void each_token(const float* pr, const float* qr, int V, F f) {
    const int tid = threadIdx.x;
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

// One wave: the digit of `hist` (DIGITS of them) that holds the need-th largest key; returns it, with the keys still needed from it and
// how many it holds.
template <int DIGITS>
__device__ __forceinline__ int pick_digit(const int* hist, int& need, int& holds) {
    constexpr int PER = DIGITS / 64;
    const int lane = threadIdx.x & 63;
    int tot = 0;                                   // lane l owns the digits from DIGITS - 1 - PER l downwards
    for (int j = 0; j < PER; ++j) tot += hist[DIGITS - 1 - PER * lane - j];
    const int incl = wave_scan_i(tot), excl = incl - tot;
    int digit = 0, left = 0, here = 0;
    if (excl < need && need <= incl) {
        int above = excl;
        for (int j = 0; j < PER; ++j) {
            digit = DIGITS - 1 - PER * lane - j;
            here = hist[digit]; left = need - above;
            if (left <= here) break;
            above += here;
        }
    }
    const int src = __ffsll(static_cast<long long>(__ballot(here > 0))) - 1;
    need = __builtin_amdgcn_readlane(left, src);
    holds = __builtin_amdgcn_readlane(here, src);
    return __builtin_amdgcn_readlane(digit, src);
}

// x, x^2, ... to the grid's draft counts in rising order: g(b, x^ns[b]), the products that ipow takes.
template <class G>
__device__ __forceinline__ void powers(const GridParams& gp, double x, G g) {
    double pw = x;
    int e = 1;
#pragma unroll
    for (int b = 0; b < kSweepMaxN; ++b) {
        if (b < gp.nn) {
            for (; e < gp.ns[b]; ++e) pw = __dmul_rn(pw, x);
            g(b, pw);
        }
    }
}

}  // namespace

__global__ __launch_bounds__(kNT) void grid_kernel(GridParams gp) {
    extern __shared__ __align__(16) unsigned char grid_lds[];
    GridLds& S = *reinterpret_cast<GridLds*>(grid_lds);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int V = gp.V, nk = gp.nk, nn = gp.nn;
    const float* pr = gp.p + static_cast<size_t>(row) * V;
    const float* qr = gp.q + static_cast<size_t>(row) * V;
    Interval* stack = reinterpret_cast<Interval*>(gp.work + row * gp.work_stride);

    // sums, validity, positive entries of q by magnitude
    for (int c = tid; c < kClasses; c += kNT) S.classes[c] = 0;
    if (tid == 0) S.listed = 0;
    __syncthreads();
    double ps = 0.0, qs = 0.0;
    int bad = 0, positive = 0;
    each_token<true>(pr, qr, V, [&](float pv, float qv, int) {
        bad |= !(qv >= 0.f) | !(pv >= 0.f);
        ps += static_cast<double>(pv); qs += static_cast<double>(qv);
        if (qv > 0.f) { ++positive; atomicAdd(&S.classes[min(__float_as_uint(qv) >> 19, kClasses - 1u)], 1); }
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
    if (wv < nk) {
        int need = gp.ks[wv], holds = 0;
        unsigned long long prefix = 0ull;
        if (need < positive) prefix = static_cast<unsigned long long>(pick_digit<kClasses>(S.classes, need, holds)) << 51;
        if (lane == 0) { S.prefix[wv] = prefix; S.need[wv] = need; S.bucket[wv] = gp.ks[wv] < positive ? holds : need; }
    }
    __syncthreads();
    unsigned open = 0u;                            // the sizes whose threshold is not found yet
    for (int a = 0; a < nk; ++a) if (S.bucket[a] != S.need[a]) open |= 1u << a;
    if (open) {
        int keys = 0;
        for (int a = 0; a < nk; ++a) {
            bool first = open >> a & 1u;
            for (int o = 0; o < a; ++o) first = first && !((open >> o & 1u) && S.prefix[o] == S.prefix[a]);
            if (first) keys += S.bucket[a];
        }
        const bool listed = keys <= kList;
        unsigned long long thr[kSweepMaxK];
        if (listed) {
#pragma unroll
            for (int a = 0; a < kSweepMaxK; ++a) thr[a] = a < nk && (open >> a & 1u) ? S.prefix[a] >> 51 : ~0ull;
            each_token<false>(pr, qr, V, [&](float, float qv, int id) {
                const unsigned c = __float_as_uint(qv) >> 19;
                bool in = false;
#pragma unroll
                for (int a = 0; a < kSweepMaxK; ++a) in |= c == static_cast<unsigned>(thr[a]);
                if (in && qv > 0.f) S.keys[atomicAdd(&S.listed, 1)] = make_key(qv, id);
            });
            __syncthreads();
        }
        for (int shift = 51; open && shift > 0;) {
            const int width = min(8, shift), above = shift;
            shift -= width;
            for (int c = tid; c < kSweepMaxK * 256; c += kNT) (&S.hist[0][0])[c] = 0;
            __syncthreads();
#pragma unroll
            for (int a = 0; a < kSweepMaxK; ++a) thr[a] = a < nk && (open >> a & 1u) ? S.prefix[a] >> above : ~0ull;
            auto add = [&](unsigned long long key) {
                const int d = static_cast<int>(key >> shift) & 255 & ((1 << width) - 1);
#pragma unroll
                for (int a = 0; a < kSweepMaxK; ++a) if (key >> above == thr[a]) atomicAdd(&S.hist[a][d], 1);
            };
            if (listed) { for (int i = tid; i < keys; i += kNT) add(S.keys[i]); }
            else each_token<false>(pr, qr, V, [&](float, float qv, int id) { if (qv > 0.f) add(make_key(qv, id)); });
            __syncthreads();
            if (wv < nk && (open >> wv & 1u)) {
                int need = S.need[wv], holds = 0;
                const int d = pick_digit<256>(S.hist[wv], need, holds);
                if (lane == 0) { S.prefix[wv] |= static_cast<unsigned long long>(d) << shift; S.need[wv] = need; S.bucket[wv] = holds; }
            }
            __syncthreads();
            open = 0u;
            for (int a = 0; a < nk; ++a) if (S.bucket[a] != S.need[a]) open |= 1u << a;
        }
    }
    unsigned long long thr[kSweepMaxK];
#pragma unroll
    for (int a = 0; a < kSweepMaxK; ++a) thr[a] = a < nk ? S.prefix[a] : 0ull;
    for (int c = tid; c < kSweepMaxK * kSweepMaxN; c += kNT) (&S.best[0][0])[c] = 0.0;   // F(0) = 0: the empty prefix
    const double invp = 1.0 / ptot;
    constexpr double kUnit = 1.0 / 4611686018427387904.0;      // 2^-62

    int waiting = 0;                               // intervals on the stack, the one of smallest keys on top
    for (int taken = 0;; ) {                       // intervals of this round; 0: the first, over all keys
        const int log_per = taken ? kBinsLog - (31 - __clz(2 * taken - 1)) : kBinsLog;
        __syncthreads();
        for (int c = tid; c < nk * (kBins + 1); c += kNT) { (&S.P[0][0])[c] = 0ull; (&S.Q[0][0])[c] = 0ull; }
        for (int c = tid; c < nk * kBins; c += kNT) (&S.count[0][0])[c] = 0;
        if (tid < taken) {
            const unsigned long long width = S.open[tid].hi - S.open[tid].lo - 1ull;
            S.shift[tid] = max(0, (width ? 64 - __clzll(static_cast<long long>(width)) : 0) - log_per);
        }
        __syncthreads();
        const unsigned long long from = taken ? S.open[0].lo : 0ull, to = taken ? S.open[taken - 1].hi : ~0ull;
        each_token<true>(pr, qr, V, [&](float pv, float qv, int id) {
            const unsigned long long qkey = make_key(qv, id);
            if (!(qv > 0.f) || qkey < thr[nk - 1]) return;
            const unsigned long long key = ratio_key(qv, pv);
            int bin;
            if (!taken) bin = first_bin(key);
            else {
                if (key < from || key >= to) return;
                int i = 0;                         // the last interval that begins at the key or before it
                for (int step = kMaxOpen / 2; step > 0; step >>= 1) if (i + step < taken && S.open[i + step].lo <= key) i += step;
                if (key >= S.open[i].hi) return;
                bin = (i << log_per) + static_cast<int>((key - S.open[i].lo) >> S.shift[i]);
            }
            int cls = 0;
#pragma unroll
            for (int a = 0; a < kSweepMaxK; ++a) cls += a < nk && qkey < thr[a];
            atomicAdd(&S.P[cls][bin], fixed62(pv));
            atomicAdd(&S.Q[cls][bin], fixed62(qv));
            atomicAdd(&S.count[cls][bin], 1);
        });
        __syncthreads();
        // every top-k size holds the tokens of the smaller ones
        if (tid < kBins) {
            unsigned long long p = 0ull, q = 0ull; int c = 0;
            for (int a = 0; a < nk; ++a) {
                p += S.P[a][tid]; S.P[a][tid] = p;
                q += S.Q[a][tid]; S.Q[a][tid] = q;
                c += S.count[a][tid]; S.count[a][tid] = c;
            }
            S.flag[tid] = 0;
        }
        __syncthreads();
        // prefix sums over the bins: a wave to a size and sum
        if (wv < 2 * nk) {
            unsigned long long* x = (wv & 1) ? S.Q[wv >> 1] : S.P[wv >> 1];
            constexpr int PER = kBins / 64;
            unsigned long long v[PER], tot = 0ull;
#pragma unroll
            for (int j = 0; j < PER; ++j) { v[j] = x[PER * lane + j]; tot += v[j]; }
            unsigned long long incl = tot;
            for (int o = 1; o < 64; o <<= 1) { const unsigned long long up = __shfl_up(incl, o); if (lane >= o) incl += up; }
            unsigned long long at = incl - tot;
#pragma unroll
            for (int j = 0; j < PER; ++j) { x[PER * lane + j] = at; at += v[j]; }
            if (lane == 63) { x[kBins] = at; if (!taken && (wv & 1)) S.mass[wv >> 1] = static_cast<double>(at) * kUnit; }
        }
        __syncthreads();
        // A bin's ends: (Q, P) of its first and last place; false where it holds no token of size a.
        auto ends = [&](int a, int j, double& p0, double& q0, double& p1, double& q1) {
            if (S.count[a][j] == 0) return false;
            unsigned long long bp = 0ull, bq = 0ull;
            if (taken) { const int i = j >> log_per; bp = S.open[i].P[a] - S.P[a][i << log_per]; bq = S.open[i].Q[a] - S.Q[a][i << log_per]; }
            const double inv = 1.0 / S.mass[a];
            p0 = static_cast<double>(S.P[a][j] + bp) * kUnit * invp; q0 = static_cast<double>(S.Q[a][j] + bq) * kUnit * inv;
            p1 = static_cast<double>(S.P[a][j + 1] + bp) * kUnit * invp; q1 = static_cast<double>(S.Q[a][j + 1] + bq) * kUnit * inv;
            return true;
        };
        auto keys_of = [&](int j, unsigned long long& lo, unsigned long long& hi) {
            if (!taken) { const int u = kBins - 1 - j; lo = kInf + 1ull - first_edge(u + 1); hi = kInf + 1ull - first_edge(u); return; }
            const int i = j >> log_per;
            lo = S.open[i].lo + (static_cast<unsigned long long>(j & ((1 << log_per) - 1)) << S.shift[i]);
            hi = min(S.open[i].hi, lo + (1ull << S.shift[i]));
        };
        // F at the bins' last places: the eight waves of a size by turns
        for (int a0 = 0; a0 < nk; a0 += kNT / kBins) {
            const int a = a0 + tid / kBins, j = tid % kBins;
            double f[kSweepMaxN];
#pragma unroll
            for (int b = 0; b < kSweepMaxN; ++b) f[b] = 0.0;
            double p0, q0, p1, q1;
            if (a < nk && ends(a, j, p0, q0, p1, q1)) powers(gp, q1, [&](int b, double pw) { f[b] = fmin(0.0, p1 - pw); });
#pragma unroll
            for (int b = 0; b < kSweepMaxN; ++b) {
                if (b < nn) {
                    const double m = wave_min(f[b]);
                    if (lane == 0) S.cell[b][wv] = m;
                }
            }
            __syncthreads();
            if (tid < kNT / kBins * kSweepMaxN) {
                const int b = tid % kSweepMaxN, s = tid / kSweepMaxN;
                if (b < nn && a0 + s < nk) {
                    double m = S.best[a0 + s][b];
                    for (int w = 0; w < kBins / 64; ++w) m = fmin(m, S.cell[b][s * (kBins / 64) + w]);
                    S.best[a0 + s][b] = m;
                }
            }
            __syncthreads();
        }
        // bins that may hold less.  What is not looked for is below 1e-13 of the acceptance.
        for (int a0 = 0; a0 < nk; a0 += kNT / kBins) {
            const int a = a0 + tid / kBins, j = tid % kBins;
            double p0, q0, p1, q1;
            if (a >= nk || S.count[a < nk ? a : 0][j] < 2 || !ends(a, j, p0, q0, p1, q1)) continue;
            unsigned long long lo, hi;
            keys_of(j, lo, hi);
            if (hi - lo < 2ull) continue;
            const double scale = S.mass[a] * invp, rmax = __longlong_as_double(static_cast<long long>(kInf - lo)),
                         rmin = __longlong_as_double(static_cast<long long>(kInf + 1ull - hi));
            const double s0 = scale / rmax, s1 = scale / rmin, dq = q1 - q0;
            double x = s1 < 1e300 ? (s1 * dq - (p1 - p0)) / (s1 - s0) : dq;
            x = fmin(fmax(x, 0.0), dq);
            const double px = p0 + s0 * x;
            bool less = false;
            powers(gp, q0 + x, [&](int b, double pw) { const double m = S.best[a][b]; less |= px - pw < m - (1e-13 * (1.0 + m) + 1e-16); });
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
            const int i = tid >> log_per;
            for (int a = 0; a < nk; ++a) {
                t.P[a] = S.P[a][tid] + (taken ? S.open[i].P[a] - S.P[a][i << log_per] : 0ull);
                t.Q[a] = S.Q[a][tid] + (taken ? S.open[i].Q[a] - S.Q[a][i << log_per] : 0ull);
            }
        }
        waiting += all;
        __syncthreads();
        if (waiting == 0) break;
        taken = min(waiting, kMaxOpen);
        for (int c = tid; c < taken * (2 + 2 * kSweepMaxK); c += kNT) {
            const int i = c / (2 + 2 * kSweepMaxK), w = c % (2 + 2 * kSweepMaxK);
            reinterpret_cast<unsigned long long*>(&S.open[i])[w] = reinterpret_cast<const unsigned long long*>(&stack[waiting - 1 - i])[w];
        }
        waiting -= taken;
    }
    for (int c = tid; c < nk * kSweepMaxN; c += kNT) {
        const int a = c / kSweepMaxN, b = c % kSweepMaxN;
        if (b < nn) gp.accept_prob[(static_cast<size_t>(row) * nk + gp.kpos[a]) * nn + gp.npos[b]] = static_cast<float>(1.0 + S.best[a][b]);
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
