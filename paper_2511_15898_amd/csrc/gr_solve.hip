// Per-row solve: one workgroup per decode position, everything after the streaming
// selection lives in LDS.
//
//   merge the slices' candidates -> top-k support V_0       (App. "Top-k Sampling ...")
//   order by decreasing q/p, prefix psi, H*, alpha*         (Sec. 5.1, Thm 3.1)
//   suffix minima -> outer targets p_i and block boundaries (Thm 6.2, Lemma 6.3)
//   truncation sets T                                       (Alg. 1, Sec. 6.3)
//   softmax weights of Theta_T / Phi_T by Newton's iteration (Thm 6.5 / Thm 6.4)
//
// A second kernel (full_programs_kernel) runs the same programs for rows whose steps 1-2 were done in
// HBM because the support is the whole vocabulary.
//
// The gradient of Theta_T / Phi_T is (mass routed to token j) - target_j.  The routed mass is a sum
// over draft tuples; here it is evaluated in polynomial time from
//     1/x = int_0^inf e^{-xt} dt,
//     E[ prod_{i in set(tuple)} x_i ] = n! [z^n] e^{z ctx} prod_i (1 + x_i (e^{z q_i} - 1)),  x_i = e^{-t w_i},
// with power series in z truncated at degree n and the trapezoid rule in log t.  The product is taken
// through its logarithm: log(1 + x (e^u - 1)) = sum_k kappa_k(x) u^k / k! with the cumulants of a
// Bernoulli(x) variable, and only k <= n can reach the z^n coefficient, so n cumulant sums per
// quadrature node describe all tokens exactly; the series exponential is taken once per node.
#include <type_traits>

#include "gr_internal.h"
#include "gr_verify_row.h"

namespace gr {

// The workgroup's LDS (dynamic: its size is that of Lds<D>), named at file scope so that functions that are not
// inlined address it as LDS and not through generic pointers.
extern __shared__ __align__(16) unsigned char gr_lds_raw[];

namespace {

// Optional cycle accounting (builds with -DGR_PHASE_CLOCKS only): thread 0 adds the shader-clock cycles since
// its previous mark to one of 24 slots; the totals per row are written to RowInfo::clk.
#ifdef GR_PHASE_CLOCKS
#define GR_CLK(L, slot) do { if (threadIdx.x == 0) { const long long now_ = clock64(); (L).clk[slot] += now_ - (L).clk_last; (L).clk_last = now_; } } while (0)
#else
#define GR_CLK(L, slot) do {} while (0)
#endif

constexpr int KS = kMaxSupport;
constexpr int kScan = 32;            // operands that a sequential sum takes from LDS between two rounds of stores
__device__ __forceinline__ int padded(int count) { return (count + kScan - 1) / kScan * kScan; }
// Threads of the solve workgroup: eight waves (two per SIMD, 256 registers each) up to 8 drafts, so that one
// wave's dependent float64 chains and LDS waits are filled by the other; four waves (one per SIMD, all 512
// registers) for the longer series of 9 to 16 drafts.
template <int D> constexpr int kThreadsOf = D > 8 ? 256 : 512;
template <int D> constexpr int kWavesOf = D > 8 ? 1 : 2;
// With more rows than compute units, two workgroups of four waves share one up to 8 drafts: while one row's stepping wave or its prologue keeps the other waves
// waiting, the other row evaluates.  The call, one workgroup and two: 512 rows of 32000 tokens, n = 4, k = 64 217 and 178 us,
// 1024 rows of 1024, n = 4, k = 32 246 and 169, of 128256, n = 8, k = 128 611 and 507 (selection 210).  A row by itself is slower on four waves, and a handful of
// rows beyond the compute units begins behind the rows that end first, before the slowest one has.  So the line lies above their number, and higher for two and
// three drafts, whose rows take up to 19 evaluations among many of 4; with one there are none.  16 kinds of rows (k 32 to 256, V 400 to 60000), four seeds, one
// workgroup's time over two's, in the mean and the calls that lose more than 2 %: n = 2 and 3 304 rows 0.96 and 20 of 32, 400 1.01 and 11, 448 1.04 and 8, 512 1.11
// and 5; n = 4 to 8 264 rows 1.00 and half, 304 1.09 and 9 of 32, 352 1.13 and 3, 400 1.14 and 1, 512 1.23 and none; n = 1 264 rows 1.30 and none.
constexpr int kNarrow = 256;
static int most_rows(int n) { return n == 1 ? 256 : (n < 4 ? 448 : 320); }   // of a batch that have a compute unit each, or wait for one
// A program that asks for more than kPatience evaluations there, or for the fallback, leaves its row to a second launch, of one workgroup to a compute unit, in
// which it goes on from its best weights and the workgroups of all other rows end at once (2 us): of 43000 rows of 14 kinds one took 1005 evaluations, one 68 and
// all others 19 at most, and where there is such a row it is the call (1024 rows of 1000 tokens, n = 4, k = 32, 1005 evaluations: 9.9 ms in workgroups of eight
// waves, 13.1 of four, 9.6 so; of 50000, n = 2, k = 256, 68 of them: 0.80, 0.84 and 0.87).
constexpr int kPatience = 24;
template <int D, int ST> constexpr bool kDefers = D <= 8 && ST == kNarrow;
constexpr int kDeferred = -1;        // of a program; RowInfo::status of its row between the launches: -1 - the program's number
constexpr double kQuadStep = 0.45;   // trapezoid step in log t (discretisation error 5.6e-9 relative at most)
constexpr double kQuadLo = 0.1;      // t_lo * (slack + sum w)
// The nodes below t_lo, t_lo e^{-step k}, are not evaluated: the integrand over t, a sum of e^{-s t} with s (slack + sum w)^-1
// at most 1, is extrapolated from its value at 0 (kQuadZero) and at the first nodes (kQuadEnd, added to their weights in units of
// t_lo): the sums over k >= 1 of step e^{-step k} times the Lagrange polynomials on 0, 1, e^step .. e^{4 step}.  Largest relative
// error of 1/s over s: 6.1e-9, of which the trapezoid rule's own 5.6e-9; taking the integrand's value at 0 for all nodes below
// t_lo = 1e-4, as was done before, 7.1e-9 with 16 nodes more.
constexpr double kQuadZero = 0.307605450234338265;
constexpr double kQuadEnd[5] = {1.01966774875832561, -0.714299827412849101, 0.202748276556553684, -0.0250005611332631344, 0.00109723308425186904};
constexpr double kQuadPair = 1.198;  // weight of the first node of every other one for t^2: 1 + 1 / (e^{4 step} - 1)
constexpr double kQuadHi = 25.0;     // t_hi * (slowest decay rate)
constexpr int kStar = 8;             // tokens of a program whose couplings to every token are computed (the others meet in a hub)
constexpr double kClip = 3.0;        // longest step of a token in log weight.  Each token's own: one that saturates asks for steps without a bound, and with
                                     // all steps scaled to the longest it held up the others for good (rows at the cap after 1000 evaluations)
constexpr double kOddsFrom = 0.5;    // a target above this share of Pr[token drawn] aims at its log odds while its mass falls short
constexpr double kSecantBelow = 1e-2;   // stopping measure from which on a step is combined with the one before it ...
constexpr int kSecantAfter = 5;      // ... as it is after this many evaluations, which only a program with a slow mode needs
constexpr double kKeepBelow = 1e-3;  // stopping measure from which on the couplings stay as they are
constexpr int kTurn = 8;             // evaluations between two looks at whether the step should change (a power of two)
constexpr int kStall = 4;            // steps without a better point before fixed-point steps are mixed in
constexpr int kRetreats = 30;        // returns to the best point, each with half the step, before the program is left to the fallback
constexpr int kStarBudget = 120;     // the iteration gets kStarBudget + m evaluations before the fallback takes over
constexpr int kRowW = 12;            // floats of a token's row of couplings: kStar couplings, slack, hub, right-hand side, 1 / sum
constexpr int kNodes = kStar + 2;    // the reduced system's vertices: kStar tokens, slack, hub
constexpr double kMostCoupled = 1e30;   // a larger weight of a coupling is that of nodes where only tokens too light for the step are left,
                                     // and would overflow
constexpr float kLightest = 0x1p-100f;   // a row whose edges sum to less of the program's mass takes no part in the reduced system:
                                     // its reciprocal overflows below 2^-127, and from 2^-102 on its right-hand side lacks the digits for 1e-8
constexpr int kMaxHeavy = 3;         // tokens that keep their exact factor (only with more than 8 drafts)
constexpr double kHeavyShare = 0.3;  // ... those above this share of the program's draw mass

// Operands of one token / one quadrature node, packed so that they are a few 16-byte LDS reads.
template <int D> struct alignas(16) TokRec { double aw; double e[D]; double pad; };     // weight; e[k-1] = q^k / k! (0 for k > n)
template <int D> struct alignas(16) NodeRec { double t, qw; double Tr[D]; };            // abscissa, quadrature weight; Tr[k-1] = T_{n-k}

// The quadrature grid of one evaluation: nodes t_lo e^{kQuadStep j}, j = 0..N-1, and the weight of the integrand's value at 0.
struct Grid { double t_lo, tail; int N; };

// What the policy object holds of a rank beside its block and weight.  Where there is room it stays in LDS to the end of the row; two workgroups to a compute
// unit write it out before the programs, whose first barrier then waits for these stores (0.4 % of a call of 256 rows).
struct PolicyRows { int tok[KS]; double pn[KS]; double rho[KS]; };
struct Nothing {};

// D: the series degree of the kernel (>= n).
template <int D, int ST = kThreadsOf<D>>
struct Lds {
    static constexpr int kST = ST;
    static constexpr bool kKeeps = !kDefers<D, ST>;
    static constexpr int kSW = kST / 64;
    static constexpr int kNPW = D > 8 ? 16 : 4;               // quadrature nodes a wave owns within a chunk
    static constexpr int kChunk = kSW * kNPW;
    static constexpr int kSer = D < 4 ? 4 : D;                // floats of one series of hser ...
    static constexpr int kSerStride = kStar * kSer + 4;      // ... and of a node's kStar of them (padded: neighbouring nodes start four banks apart)
    // support, in ratio order
    std::conditional_t<kKeeps, PolicyRows, Nothing> kept;
    __device__ PolicyRows& rows() { if constexpr (kKeeps) return kept; else return early; }
    int blk[KS]; int inT[KS]; int ordq[KS]; int apos[kMaxT];
    int flag[KS + 2]; int blo[KS + 2]; int star[kStar];
    double qn[KS]; double tgt[KS]; double wgt[KS];
    double Q[KS + 1]; double F[KS + 2];
    // one convex program (the kStar tokens of largest target first, then by decreasing q)
    double aq[kMaxT]; double at[kMaxT]; double aal[kMaxT]; double aR[kMaxT];
    double aS[kMaxT]; double ag[kMaxT];   // with aR: what one evaluation hands to the step (see solve_program)
    double aR0, alc;                      // ... the slack mass and, with slack, log(slack mass / its target)
    double ared[2][3];                    // ... and the first two waves' sum of R, max and min of log(target / R)
    double apd[kMaxT];              // Pr[token drawn within the program] = atot^n - (atot - q)^n
    double af[kMaxT];
    // Newton fallback (its Jacobian lives in a per-row HBM scratch)
    double nR[kMaxT]; double nstep[kMaxT]; double nsave[kMaxT]; int nused[kMaxT]; int ncolof[kMaxT];
    // scans and counters of the prologue (dead once the first program starts) share their bytes with the
    // evaluator's records and per-wave partial sums
    union {
        struct {
            int cnt0[KS + 2]; int cnt1[KS + 2]; int ids[KS]; int byq[KS];
            double qd[KS]; double accb[KS]; std::conditional_t<kKeeps, Nothing, PolicyRows> early;
            union {
                unsigned long long keys[kSelCap];   // unsorted candidates (select merge), until ids and accb hold the support
                struct {
                    double dlt[KS]; double dval[KS];   // rows given as logits: draft minus target logit, draft logit
                    double P[KS + 2]; double S[KS + 2]; double G0[KS]; double G1[KS + 2]; double O0[KS]; double O1[KS + 2];
                };
            };
        };
        struct {
            double hpair[kSW][4];       // per wave: the couplings of the heavy tokens 0-1, 0-2, 1-2 (only with more than 8 drafts)
            double rpart[kSW][kMaxT];   // per wave: sum over its nodes of the integrand of each token
            double spart[kSW][kMaxT];   // the same weighted by t
            float cpart[kSW][kMaxT * kStar];   // per wave: the couplings of each token to the first kStar
            float hser[kSW][kNPW / 2 * kSerStride];   // per wave: the series of the first kStar tokens at every other node
            NodeRec<D> nrec[D > 8 ? kSW : 1][D > 8 ? kNPW : 1];
            TokRec<D> trec[kMaxT + 4];  // active tokens; every record beyond the last has aw = 1e300 (x = 0), e = 0
        };
    };
    double aBest[kMaxT]; double fBest[kMaxT]; double aPrev[kMaxT]; double fPrev[kMaxT];
    alignas(16) float W[kMaxT][kRowW];   // the tokens' rows of the reduced system
    alignas(16) float Am[16][20];        // the light tokens' share of it, as the matrix cores leave it
    Grid ctl_grid; int ctl_go, ctl_result, ctl_bestok, ctl_couple; double turn_err;   // handed from the stepping wave to all waves
    double e2tab[32];               // 2^(-j/32)
    int nheavy;                     // leading tokens that keep their exact factor
    int nfull;                      // leading tokens (the heavy ones included) that need all D cumulants; the rest need four
    double work;                    // sum over evaluator calls of nodes x active tokens (thread 0 only)
#ifdef GR_PHASE_CLOCKS
    long long clk[24]; long long clk_last; double errlog[24];
#endif
    double red[2][kSW][8]; double redn[kSW]; double r0part[kSW]; int pick[4]; int count; int hist[256];
};

// ---- workgroup reductions with one barrier: the waves' partial results alternate between two LDS
// strips (`par`), so the strip of the reduction before the previous one is free again.
enum { kOpSum = 0, kOpMax = 1, kOpMin = 2 };
__device__ __forceinline__ double combine(double a, double b, int op) {
    return op == kOpSum ? a + b : (op == kOpMax ? fmax(a, b) : fmin(a, b));
}
// Several reductions over the lanes of one wave at once (their butterfly steps interleave): every lane ends with
// the results.  All 64 lanes must be active.
template <int NV>
__device__ __forceinline__ void wave_reduce_many(double (&v)[NV], const int (&op)[NV]) {
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = combine(v[j], dpp_move<kDppXor1>(v[j]), op[j]);
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = combine(v[j], dpp_move<kDppXor2>(v[j]), op[j]);
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = combine(v[j], dpp_move<kDppHalfMirror>(v[j]), op[j]);
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = combine(v[j], dpp_move<kDppMirror>(v[j]), op[j]);
#pragma unroll
    for (int j = 0; j < NV; ++j)
        v[j] = combine(combine(read_lane(v[j], 0), read_lane(v[j], 16), op[j]), combine(read_lane(v[j], 32), read_lane(v[j], 48), op[j]), op[j]);
}

// v[j] holds this wave's partial result of operation op[j]; on return it holds the workgroup's.  After the
// barrier lane l reads the partial of wave l mod 4 or 16 (one LDS instruction per value and wave, not NW), and a
// butterfly over that many neighbouring lanes combines them: every lane ends with the same bits.
template <int NV, class LdsT>
__device__ __forceinline__ void wg_reduce(LdsT& L, int& par, double (&v)[NV], const int (&op)[NV]) {
    constexpr int NW = LdsT::kSW;
    static_assert(NW <= 16, "the butterfly below covers up to sixteen waves");
    constexpr int G = NW <= 4 ? 4 : 16;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int j = 0; j < NV; ++j) L.red[par][wv][j] = v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int w = lane & (G - 1);
        double r = L.red[par][min(w, NW - 1)][j];
        if (G != NW) r = w < NW ? r : (op[j] == kOpSum ? 0.0 : (op[j] == kOpMax ? -1e301 : 1e301));
        r = combine(r, dpp_move<kDppXor1>(r), op[j]);
        r = combine(r, dpp_move<kDppXor2>(r), op[j]);
        if (G == 16) { r = combine(r, dpp_move<kDppHalfMirror>(r), op[j]); r = combine(r, dpp_move<kDppMirror>(r), op[j]); }
        v[j] = r;
    }
    par ^= 1;
}
template <class LdsT> __device__ __forceinline__ double wg_sum(LdsT& L, int& par, double v) {
    double a[1] = {wave_sum(v)};
    wg_reduce<1>(L, par, a, {kOpSum});
    return a[0];
}
template <class LdsT> __device__ __forceinline__ double wg_max(LdsT& L, int& par, double v) {
    double a[1] = {wave_max(v)};
    wg_reduce<1>(L, par, a, {kOpMax});
    return a[0];
}

__device__ __forceinline__ unsigned wave_max_u(unsigned x) {
    int v = static_cast<int>(x);
    v = static_cast<int>(max(static_cast<unsigned>(v), static_cast<unsigned>(dpp_move<kDppXor1>(v))));
    v = static_cast<int>(max(static_cast<unsigned>(v), static_cast<unsigned>(dpp_move<kDppXor2>(v))));
    v = static_cast<int>(max(static_cast<unsigned>(v), static_cast<unsigned>(dpp_move<kDppHalfMirror>(v))));
    v = static_cast<int>(max(static_cast<unsigned>(v), static_cast<unsigned>(dpp_move<kDppMirror>(v))));
    return max(max(static_cast<unsigned>(__builtin_amdgcn_readlane(v, 0)), static_cast<unsigned>(__builtin_amdgcn_readlane(v, 16))),
               max(static_cast<unsigned>(__builtin_amdgcn_readlane(v, 32)), static_cast<unsigned>(__builtin_amdgcn_readlane(v, 48))));
}

// 1/x from the hardware estimate and two Newton steps (about 1e-16 relative; x = 0, infinite or NaN gives NaN or 0).
__device__ __forceinline__ double fast_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = r * fma(-x, r, 2.0);
    r = r * fma(-x, r, 2.0);
    return r;
}

// e^x for |x| <= 1000 (clamped beyond) with the table of exp_neg: x = -(k ln2/32 + r), k of either sign.
__device__ __forceinline__ double exp_signed(double x, const double* tab) {
    const double y = fmax(fmin(-x, 1000.0), -1000.0);
    const double kf = rint(y * 46.166241308446828);
    const int ki = static_cast<int>(kf);
    const double tv = tab[ki & 31];                            // k = 32 (k >> 5) + (k & 31), also for negative k
    double r = fma(kf, -(6.93147180369123816490e-01 / 32.0), y);
    r = -fma(kf, -(1.90821492927058770002e-10 / 32.0), r);
    double p = 8.33333333333333333333e-03;
    p = fma(p, r, 4.16666666666666666667e-02);
    p = fma(p, r, 1.66666666666666666667e-01);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p * tv, -(ki >> 5));
}

// log(x) to about 1e-16 relative for positive normal x: x = 2^e m with m in [sqrt(1/2), sqrt(2)),
// log m = 2 atanh(s) = 2 s (1 + s^2/3 + s^4/5 + ...), s = (m - 1) / (m + 1), |s| <= 0.172 (eleven terms).
// Anything else (zero, negative, denormal, infinite, NaN) goes to the library routine.
__device__ __forceinline__ double fast_log(double x) {
    if (!(x >= 2.3e-308 && x <= 1.7e308)) return log(x);
    int e;
    double m = frexp(x, &e);                                   // m in [1/2, 1)
    if (m < 0.70710678118654752) { m *= 2.0; e -= 1; }
    const double s = (m - 1.0) * fast_rcp(m + 1.0), z = s * s;
    double p = 1.0 / 21.0;
    p = fma(p, z, 1.0 / 19.0); p = fma(p, z, 1.0 / 17.0); p = fma(p, z, 1.0 / 15.0); p = fma(p, z, 1.0 / 13.0);
    p = fma(p, z, 1.0 / 11.0); p = fma(p, z, 1.0 / 9.0); p = fma(p, z, 1.0 / 7.0); p = fma(p, z, 1.0 / 5.0);
    p = fma(p, z, 1.0 / 3.0); p = fma(p, z, 1.0);
    const double ed = static_cast<double>(e);
    return fma(ed, 6.93147180369123816490e-01, fma(2.0 * s, p, ed * 1.90821492927058770002e-10));
}

// Cumulants of a Bernoulli(x) variable: kappa_1 = x, kappa_{k+1} = v g_k with v = x (1 - x),
// g_k = d kappa_k / dx = a_k(v) for odd k, s a_k(v) for even k, s = 1 - 2x (from kappa_{k+1} = x (1 - x) kappa_k').
// Row k: the coefficients of a_k in rising powers of v.
__device__ constexpr double kCumA[17][8] = {
    {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -6.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -12.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -30.0, 120.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -60.0, 360.0, 0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -126.0, 1680.0, -5040.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -252.0, 5040.0, -20160.0, 0.0, 0.0, 0.0, 0.0},
    {1.0, -510.0, 17640.0, -151200.0, 362880.0, 0.0, 0.0, 0.0},
    {1.0, -1020.0, 52920.0, -604800.0, 1814400.0, 0.0, 0.0, 0.0},
    {1.0, -2046.0, 168960.0, -3160080.0, 19958400.0, -39916800.0, 0.0, 0.0},
    {1.0, -4092.0, 506880.0, -12640320.0, 99792000.0, -239500800.0, 0.0, 0.0},
    {1.0, -8190.0, 1561560.0, -57657600.0, 726485760.0, -3632428800.0, 6227020800.0, 0.0},
    {1.0, -16380.0, 4684680.0, -230630400.0, 3632428800.0, -21794572800.0, 43589145600.0, 0.0},
    {1.0, -32766.0, 14217840.0, -988107120.0, 22313491200.0, -210680870400.0, 871782912000.0, -1307674368000.0},
    {1.0, -65532.0, 42653520.0, -3952428480.0, 111567456000.0, -1264085222400.0, 6102480384000.0, -10461394944000.0},
};

// g[k-1] = g_k(x) for k = 1..C.
template <int K, int C, class T>
__device__ __forceinline__ void cum_g_from(T v, T s, T (&g)[C]) {
    if constexpr (K <= C) {
        constexpr int deg = (K - 1) / 2;
        T r = static_cast<T>(kCumA[K][deg]);
#pragma unroll
        for (int j = deg - 1; j >= 0; --j) r = fma(r, v, static_cast<T>(kCumA[K][j]));
        g[K - 1] = (K % 2 == 0) ? r * s : r;
        cum_g_from<K + 1, C>(v, s, g);
    }
}

// A(z) <- A(z) * (1 + x (e^{zq} - 1)), e[a-1] = q^a / a!.
template <int D>
__device__ __forceinline__ void mul_factor(double (&A)[D + 1], double x, const double (&e)[D]) {
#pragma unroll
    for (int d = D; d >= 1; --d) {
        double acc = 0.0;
#pragma unroll
        for (int a = 1; a <= d; ++a) acc = fma(e[a - 1], A[d - a], acc);
        A[d] = fma(x, acc, A[d]);
    }
}

// [z^n] of  (e^{zq} - 1) * T(z) / (1 + x (e^{zq} - 1)): the leave-one-out coefficient of a token that
// keeps its exact factor, by series division (the quotient is only needed below degree n).
template <int D>
__device__ __forceinline__ double loo_coeff(const double (&T)[D + 1], double x, const double (&e)[D], int n) {
    double Bq[D + 1];
    Bq[0] = T[0];
    double cn = 0.0;
#pragma unroll
    for (int d = 1; d <= D; ++d) {
        double conv = 0.0;
#pragma unroll
        for (int a = 1; a <= d; ++a) conv = fma(e[a - 1], Bq[d - a], conv);
        Bq[d] = fma(-x, conv, T[d]);
        if (d == n) cn = conv;
    }
    return cn;
}

// rec.Tr[k-1] = T_{NN-k} (0 below degree 0); returns T_NN.
template <int D, int NN>
__device__ __forceinline__ double pick_series(NodeRec<D>& rec, const double (&T)[D + 1], int n) {
    if constexpr (NN >= 1) {
        if (n == NN) {
#pragma unroll
            for (int k = 1; k <= D; ++k) rec.Tr[k - 1] = (NN - k >= 0) ? T[(NN - k >= 0) ? NN - k : 0] : 0.0;
            return T[NN];
        }
        return pick_series<D, NN - 1>(rec, T, n);
    } else {
        return 0.0;
    }
}

// Phase 1, one token at one node: its cumulant terms into the node's sums, K[k-1] += kappa_k(x) q^k / k!
// for k <= C (C = D: exact; C = 4 for a token so small that its higher terms cannot reach the z^n
// coefficient within 1e-11).
template <int D, int C>
__device__ __forceinline__ void phase1_token(double (&K)[D], const TokRec<D>& r, double x) {
    const double v = fma(-x, x, x), s = fma(-2.0, x, 1.0);
    K[0] = fma(x, r.e[0], K[0]);
    if constexpr (C >= 2) {
        double g[C - 1];
        cum_g_from<1, C - 1>(v, s, g);
#pragma unroll
        for (int k = 2; k <= C; ++k) K[k - 1] = fma(v * g[k - 2], r.e[k - 1], K[k - 1]);
    }
}

// Tokens first + tsub, first + tsub + NS, ... below `last` at this lane's node, two records in flight.
template <int D, int C, int NS>
__device__ __forceinline__ void phase1_range(double (&K)[D], const TokRec<D>* trec, int first, int last, int pad, int tsub,
                                             double t, const double* tab) {
    if (first >= last) return;
    const int i0 = first + tsub;
    TokRec<D> cur = trec[i0 < last ? i0 : pad];
    for (int b = first; b < last; b += 2 * NS) {           // uniform trip count; the pad record has x = 0
        const int i1 = b + tsub + NS, i2 = b + tsub + 2 * NS;
        const TokRec<D> nxt = trec[i1 < last ? i1 : pad];
        double x0, x1;
        exp_neg2(t * cur.aw, t * nxt.aw, tab, x0, x1);
        phase1_token<D, C>(K, cur, x0);
        cur = trec[i2 < last ? i2 : pad];
        phase1_token<D, C>(K, nxt, x1);
    }
}

// Phase 3, one token at one node: (e^u - 1) / (1 + x (e^u - 1)) = sum_k g_k(x) u^k / k!, so the
// leave-one-out coefficient is sum_{k <= C} g_k(x) (q^k / k!) T_{n-k}.
template <int D, int C>
__device__ __forceinline__ void phase3_pair(const NodeRec<D>& c, const double (&e)[D], double x, double& acc, double& at) {
    const double v = fma(-x, x, x), s = fma(-2.0, x, 1.0);
    double g[C];
    cum_g_from<1, C>(v, s, g);
    double cn = e[0] * c.Tr[0];
#pragma unroll
    for (int k = 2; k <= C; ++k) cn = fma(e[k - 1] * g[k - 1], c.Tr[k - 1], cn);
    const double term = c.qw * x * cn;
    acc += term;
    at = fma(term, c.t, at);
}

// Tokens [first, last) against the npw nodes of this wave: lane = (token slot, node subset), the split that
// needs the fewest rounds; the sums go to this wave's rpart / spart.
template <int D, int C, class LdsT>
__device__ __forceinline__ void phase3_range(LdsT& L, int first, int last, int pad, int npw, int wv, int lane) {
    constexpr int NPW = LdsT::kNPW;
    const int cnt = last - first;
    if (cnt <= 0 || npw <= 0) return;
    // cost of a split in units of one (token, node) pair: per group of tokens the rounds over the node
    // subsets, one unit for loading the token and storing its sums, one per level of the butterfly
    int ts_log = 6, best = ((cnt + 63) >> 6) * (npw + 1);
#pragma unroll
    for (int tl = 5; tl >= 3; --tl) {
        const int nsub_ = 64 >> tl;
        if (nsub_ > NPW) break;
        const int c = ((cnt + (1 << tl) - 1) >> tl) * ((npw + nsub_ - 1) / nsub_ + 1 + (6 - tl));
        if (c < best) { best = c; ts_log = tl; }
    }
    const int TS = 1 << ts_log, nsub = 64 >> ts_log;
    const int tslot = lane & (TS - 1), ns = lane >> ts_log;
    const int rounds = (npw + nsub - 1) / nsub;
    for (int g0 = first; g0 < last; g0 += TS) {
        const int tok = g0 + tslot;
        const TokRec<D> tr = L.trec[tok < last ? tok : pad];
        double acc = 0.0, at = 0.0;
        NodeRec<D> cur = L.nrec[wv][ns];
        for (int r = 0; r < rounds; r += 2) {
            const int j1 = ns + (r + 1) * nsub, j2 = ns + (r + 2) * nsub;
            const NodeRec<D> nxt = L.nrec[wv][j1 < NPW ? j1 : ns];
            double x0, x1;
            exp_neg2(cur.t * tr.aw, nxt.t * tr.aw, L.e2tab, x0, x1);
            phase3_pair<D, C>(cur, tr.e, x0, acc, at);
            cur = L.nrec[wv][j2 < NPW ? j2 : ns];
            if (r + 1 < rounds) phase3_pair<D, C>(nxt, tr.e, x1, acc, at);
        }
        if (ts_log <= 5) { acc += __shfl_xor(acc, 32); at += __shfl_xor(at, 32); }
        if (ts_log <= 4) { acc += __shfl_xor(acc, 16); at += __shfl_xor(at, 16); }
        if (ts_log <= 3) { acc += __shfl_xor(acc, 8); at += __shfl_xor(at, 8); }
        if (ns == 0 && tok < last) { L.rpart[wv][tok] += acc; L.spart[wv][tok] += at; }
    }
}

// The evaluator for up to eight drafts takes phase 3 in two parts: the first CL terms, which every token needs, and
// the terms CL + 1 .. D of a token that needs them all.
// Phase 3: the sum of phase3_pair by Horner's rule in q = e[0], with Tp[k-1] = T_{n-k} / k!, so that only q is read:
//   cn = q (Tp_1 + q (g_2 Tp_2 + ... + q (g_CL Tp_CL + q top))),  top = g_{CL+1} Tp_{CL+1} + q (... + q g_D Tp_D)
// for a token that needs all terms, top = 0 otherwise.
template <int D, int CL>
__device__ __forceinline__ double loo_top(const double (&Tp)[D], double q, double v, double s) {
    if constexpr (D > CL) {
        double g[D];
        cum_g_from<CL + 1, D>(v, s, g);
        double h = g[D - 1] * Tp[D - 1];
#pragma unroll
        for (int k = D - 1; k > CL; --k) h = fma(q, h, g[k - 1] * Tp[k - 1]);
        return h;
    } else {
        return 0.0;
    }
}
template <int D, int CL>
__device__ __forceinline__ double loo_low(const double (&Tp)[D], double q, double v, double s, double top) {
    double h = top;
    if constexpr (CL >= 2) {
        double g[CL];
        cum_g_from<1, CL>(v, s, g);
#pragma unroll
        for (int k = CL; k >= 2; --k) h = fma(q, h, g[k - 1] * Tp[k - 1]);
    }
    h = fma(q, h, Tp[0]);
    return q * h;
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ Grid make_grid(int slack, double ctx, double wsum, double wmin) {
    Grid g;
    g.t_lo = kQuadLo * fast_rcp(slack + wsum);
    const double lowest = slack + ((slack == 0 || ctx == 0.0) ? wmin : 0.0);
    const double range = fast_log((kQuadHi / kQuadLo) * (slack + wsum) * fast_rcp(lowest));
    g.N = min(max(static_cast<int>(ceil(range / kQuadStep)) + 1, 1), 4096);
    g.tail = kQuadZero * g.t_lo;
    return g;
}
// The weight of node j, at t, without the slack's e^{-slack t}.
__device__ __forceinline__ double node_weight(int j, double t, double t_lo) {
    double e = 0.0;
#pragma unroll
    for (int k = 0; k < 5; ++k) e = j == k ? kQuadEnd[k] : e;
    return fma(e, t_lo, kQuadStep * t);
}

// The couplings C_ij = E[s_i s_j] (s_i = w_i / (slack + sum of the drawn tokens' w) for a drawn token, 0 otherwise) are
// the off-diagonal entries of -dR_i / dalpha_j; with phi_i(z) = x_i (e^{zq_i} - 1) / (1 + x_i (e^{zq_i} - 1)),
//     C_ij = w_i w_j n! int t e^{-slack t} [z^n] T phi_i phi_j dt.
// They only steer the step, so they are taken in float32 and at every other node of the grid (the trapezoid rule with twice
// the step is good to 1e-4), for the first kStar tokens j and every token i.  Two lanes share a node: that of the
// wave's even node takes the tokens 0..3 of the kStar, its partner (that of the odd neighbour) the tokens 4..7.
// star_series: u[k-1] = weight * t w_j [z^{n-k}] (T phi_j) / k!, k = 1 .. D - 1, of one of the kStar tokens at one node; the
// row of token i is then w_i n! sum over the nodes and k of x_i g_k(x_i) q_i^k u[k-1].  Tr[k-1] = T_{n-k}; e: the token's series.
template <int D>
__device__ __forceinline__ void star_series(const float (&Tr)[D], const double* e, double tw, double qw2, float x, float* out) {
    constexpr int M = D - 1;
    float g[M], phi[M];
    cum_g_from<1, M>(fmaf(-x, x, x), fmaf(-2.f, x, 1.f), g);
#pragma unroll
    for (int b = 1; b <= M; ++b) phi[b - 1] = x * g[b - 1] * static_cast<float>(e[b - 1]);
    float cw = static_cast<float>(fmin(qw2 * fmin(tw, 1000.0), kMostCoupled));   // beyond 1000 x = 0
    float u[Lds<D>::kSer];
#pragma unroll
    for (int k = 1; k <= Lds<D>::kSer; ++k) {
        float acc = 0.f;
#pragma unroll
        for (int b = 1; b <= D - k; ++b) acc = fmaf(phi[b - 1], Tr[k + b - 1], acc);
        cw *= 1.f / static_cast<float>(k);
        u[k - 1] = acc * cw;
    }
#pragma unroll
    for (int k = 0; k < Lds<D>::kSer; k += 4) *reinterpret_cast<float4*>(out + k) = make_float4(u[k], u[k + 1], u[k + 2], u[k + 3]);
}
// This lane's four series of a node (half = 0: tokens 0..3, 1: tokens 4..7).
template <int D>
__device__ __forceinline__ void star_load(float (&U)[4][Lds<D>::kSer], const float* node, int half) {
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int k = 0; k < Lds<D>::kSer; k += 4) {
            const float4 v = *reinterpret_cast<const float4*>(node + (4 * half + h) * Lds<D>::kSer + k);
            U[h][k] = v.x; U[h][k + 1] = v.y; U[h][k + 2] = v.z; U[h][k + 3] = v.w;
        }
}
// One token's terms at one node for four of the kStar tokens, its orders up to C.
template <int D, int C>
__device__ __forceinline__ void star_row(const float (&U)[4][Lds<D>::kSer], float q, float x, float (&acc)[4]) {
    float y[C];
    y[0] = x * q;
    if constexpr (C >= 2) {
        float g[C], xq = y[0];
        cum_g_from<1, C>(fmaf(-x, x, x), fmaf(-2.f, x, 1.f), g);
#pragma unroll
        for (int k = 2; k <= C; ++k) { xq *= q; y[k - 1] = xq * g[k - 1]; }
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        acc[h] = y[0] * U[h][0];
#pragma unroll
        for (int k = 2; k <= C; ++k) acc[h] = fmaf(y[k - 1], U[h][k - 1], acc[h]);
    }
}
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) { return __int_as_float(dpp_move<CTRL>(__float_as_int(v))); }
// Keeps one of two values and adds the partner lane's copy of it: the first step of a sum that also parts the values.
template <int CTRL> __device__ __forceinline__ float part_add(float a, float b, bool second) {
    const float keep = second ? b : a, send = second ? a : b;
    return keep + dpp_f<CTRL>(send);
}

// The same for a token that keeps its exact factor (more than 8 drafts): its cumulants cancel, so T phi = (T / (1 + x (e^u - 1)))
// x (e^u - 1) is taken by series division in float64.
template <int D, int NN>
__device__ __forceinline__ void pick_star(float (&u)[D], const double (&V)[D], int n) {
    if constexpr (NN >= 1) {
        if (n == NN) {
#pragma unroll
            for (int k = 1; k <= D; ++k) u[k - 1] = (NN - k >= 1) ? static_cast<float>(V[(NN - k >= 1) ? NN - k : 0]) : 0.f;
            return;
        }
        pick_star<D, NN - 1>(u, V, n);
    }
}
// B = T / (1 + x (e^u - 1)) up to degree D - 1.
template <int D>
__device__ __forceinline__ void divide_factor(double (&B)[D], double x, const double* e) {
#pragma unroll
    for (int d = 1; d < D; ++d) {
        double conv = 0.0;
#pragma unroll
        for (int a = 1; a <= d; ++a) conv = fma(e[a - 1], B[d - a], conv);
        B[d] = fma(-x, conv, B[d]);
    }
}
template <int D>
__device__ __forceinline__ void star_series_exact(const double (&T)[D + 1], const double* e, double tw, double qw2, double x, int n, float* out) {
    double B[D], V[D];
#pragma unroll
    for (int d = 0; d < D; ++d) B[d] = T[d];
    divide_factor<D>(B, x, e);
    const double cx = fmin(qw2 * fmin(tw, 1000.0), kMostCoupled) * x;
    V[0] = 0.0;
#pragma unroll
    for (int d = 1; d < D; ++d) {
        double conv = 0.0;
#pragma unroll
        for (int a = 1; a <= d; ++a) conv = fma(e[a - 1], B[d - a], conv);
        V[d] = cx * conv;
    }
    float u[D], inv = 1.f;
    pick_star<D, D>(u, V, n);
#pragma unroll
    for (int k = 1; k <= D; ++k) { inv *= 1.f / static_cast<float>(k); u[k - 1] *= inv; }
#pragma unroll
    for (int k = 0; k < D; k += 4) *reinterpret_cast<float4*>(out + k) = make_float4(u[k], u[k + 1], u[k + 2], u[k + 3]);
}
// [z^n] T phi_a phi_b of two such tokens.
template <int D>
__device__ __forceinline__ double heavy_pair(const double (&T)[D + 1], const double* ea, const double* eb, double xa, double xb, int n) {
    double B[D];
#pragma unroll
    for (int d = 0; d < D; ++d) B[d] = T[d];
    divide_factor<D>(B, xa, ea);
    divide_factor<D>(B, xb, eb);
    double V[D];
    V[0] = 0.0;
#pragma unroll
    for (int d = 1; d < D; ++d) {
        double conv = 0.0;
#pragma unroll
        for (int a = 1; a <= d; ++a) conv = fma(ea[a - 1], B[d - a], conv);
        V[d] = conv;
    }
    double out = 0.0;
#pragma unroll
    for (int d = 1; d < D; ++d) out = fma(d < n ? V[d] : 0.0, eb[n - d > 0 ? n - d - 1 : 0], out);
    return xa * xb * out;
}
// Phase 4 of an evaluation: the rows of all tokens from the series that the wave has left in hser.  t: abscissa of the
// lane's node.  The sixteen tokens that come first (the kStar, then the largest q) take all orders, the others the first (the first
// two with more than 8 drafts): with all orders for all of them the step is no better, as their q is small.
// `more`: the wave has been through a chunk of nodes before.
template <int D, int ST>
__device__ __forceinline__ void star_phase(Lds<D, ST>& L, int lane, int wv, int m, double t, bool more) {
    constexpr int NPW = Lds<D, ST>::kNPW, NS = 64 / NPW, CC = D > 8 ? 2 : 1;
    static_assert(NPW == 4 || NPW == 16, "the sums over a subset's node lanes below");
    const int j = lane & (NPW - 1), tsub = lane / NPW;
    const bool b0 = j & 1, b1 = j & 2, b2 = j & 4;
    const bool upper = NPW == 4 ? b0 : j >= 8;
    const double tm = dpp_move<NPW == 4 ? kDppXor1 : kDppMirror>(t);
    const double te = upper ? tm : t;                          // the pair's even node
    wave_lds_sync();
    float U[4][Lds<D, ST>::kSer];
    star_load<D>(U, &L.hser[wv][(NPW == 4 ? j >> 1 : (upper ? 15 - j : j)) * Lds<D, ST>::kSerStride], upper);
    float* out = &L.cpart[wv][tsub * kStar + (upper ? 4 : 0) + (NPW == 4 ? (b1 ? 2 : 0) : (b2 ? 2 : 0) + (b0 ? 1 : 0))];
    auto row = [&](int i, auto all) {
        const TokRec<D>& rec = L.trec[NS * i + tsub];          // records beyond the last token: x = 0
        const float x = __expf(-static_cast<float>(fmin(te * rec.aw, 1000.0))), q = static_cast<float>(rec.e[0]);
        float acc[4];
        star_row<D, decltype(all)::value>(U, q, x, acc);
        float* const at = out + i * NS * kStar;
        if constexpr (NPW == 4) {
            const float c0 = part_add<kDppXor2>(acc[0], acc[2], b1), c1 = part_add<kDppXor2>(acc[1], acc[3], b1);
            float2* const p = reinterpret_cast<float2*>(at);
            const float2 old = more ? *p : make_float2(0.f, 0.f);
            *p = make_float2(old.x + c0, old.y + c1);
        } else {
            const float r0 = part_add<kDppHalfMirror>(acc[0], acc[2], b2), r1 = part_add<kDppHalfMirror>(acc[1], acc[3], b2);
            float c = part_add<kDppXor1>(r0, r1, b0);
            c += dpp_f<kDppXor2>(c);
            if (!b1) *at = more ? *at + c : c;
        }
    };
    const int rows = (m + NS - 1) / NS;
    int i = 0;
    for (; i < min(rows, 16 / NS); ++i) row(i, std::integral_constant<int, D - 1>());
#pragma unroll 2
    for (; i < rows; ++i) row(i, std::integral_constant<int, CC>());
}

// Routed mass of every active token, and the mass left to the slack term.
//
// Tokens are held in decreasing q: first the (at most three, only with more than 8 drafts) heavy ones that keep
// their exact factor, then up to L.nfull tokens with all D cumulants, then the tokens that need four.  A chunk
// of up to 64 quadrature nodes is dealt to the waves (wave w owns the pairs of nodes w, w + NW, ...), and a wave takes
// its nodes through all three phases without a workgroup barrier:
//   phase 1  lane = (node, token subset): the cumulant sums of its tokens at its node, then a butterfly over
//            the subsets;
//   phase 2  per node: T = exp(z ctx + cumulant series) (times the exact factors of the heavy tokens), the
//            slack integrand, and the node record {t, weight, T_{n-1..n-D}} -> LDS;
//   phase 3  lane = (token, node subset): the leave-one-out coefficient of its token at each of the wave's
//            nodes; the waves' partial sums meet in LDS at the end;
//   phase 4  lane = (node pair and half of the first kStar tokens, token subset): the couplings (star_phase).
// In: L.trec[] (weights and series terms), L.apd / L.nheavy / L.nfull (set up by solve_program), the grid.
// Out: every wave's partial sums in L.rpart / L.spart / L.r0part, and in L.cpart where `couple` is set.  All waves call it
// behind a barrier that made the weights visible; it contains no workgroup barrier itself.
template <int D, int ST>
__device__ __forceinline__ void eval_core_nodes(Lds<D, ST>& L, const Grid& gr, int m, int n, double ctx, int slack, bool couple) {
    constexpr int kSW = Lds<D, ST>::kSW, NPW = Lds<D, ST>::kNPW, NS = 64 / NPW;
    constexpr int CL = D < 4 ? D : 4;                          // cumulants of a light token
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int nheavy = (D > 8) ? L.nheavy : 0;
    const int nfull = (D > 4) ? L.nfull : nheavy;              // up to four drafts four cumulants are all there are
    const double t_lo = gr.t_lo;
    const int N = gr.N;
    static_assert(NPW == 16 && NS == 4, "phase 4 pairs the sixteen node lanes of a subset by a row mirror");
    for (int i = lane; i < m; i += 64) { L.rpart[wv][i] = 0.0; L.spart[wv][i] = 0.0; }
    double r0 = 0.0;                                       // slack integrand, lanes of token subset 0
    double hacc[kMaxHeavy] = {0.0, 0.0, 0.0}, hacct[kMaxHeavy] = {0.0, 0.0, 0.0};
    const int j = lane & (NPW - 1), tsub = lane / NPW;
    GR_CLK(L, 6);

    for (int c0 = 0; c0 < N; c0 += 64) {
        const int nn = min(64, N - c0);
        // pairs of neighbouring nodes are dealt to the waves; the wave's node j sits at place `at` of its nodes in rising order
        const int pairs = (nn + 1) >> 1, mine = (pairs - wv + kSW - 1) / kSW;
        const int npw = 2 * mine - ((nn & 1) && (pairs - 1) % kSW == wv ? 1 : 0);
        const int at = j < 8 ? 2 * j : 2 * (15 - j) + 1;
        const int node = c0 + 2 * wv + 2 * kSW * (at >> 1) + (at & 1);
        const double t = t_lo * exp(kQuadStep * static_cast<double>(node));
        const double es = at < npw ? exp_neg(slack * t, L.e2tab) : 0.0, qw = node_weight(node, t, t_lo) * es;
        // ---- phase 1: cumulant sums at node j of the tokens of subset tsub
        double K[D];
#pragma unroll
        for (int k = 0; k < D; ++k) K[k] = 0.0;
        if (npw > 0) {
            if constexpr (D > 4) phase1_range<D, D, NS>(K, L.trec, nheavy, nfull, m, tsub, t, L.e2tab);
            phase1_range<D, CL, NS>(K, L.trec, nfull, m, m, tsub, t, L.e2tab);
        }
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (NS >= 8) K[k] += __shfl_xor(K[k], 8);
            K[k] += __shfl_xor(K[k], 16);
            K[k] += __shfl_xor(K[k], 32);
        }
        GR_CLK(L, 7);
        // ---- phase 2: the node's series T = exp(z ctx + sum_k K_k z^k), every lane of the node alike
        K[0] += ctx;
        double T[D + 1];
        T[0] = 1.0;
        {
            double kK[D];
#pragma unroll
            for (int k = 1; k <= D; ++k) kK[k - 1] = static_cast<double>(k) * K[k - 1];
#pragma unroll
            for (int d = 1; d <= D; ++d) {
                double acc = kK[0] * T[d - 1];
#pragma unroll
                for (int k = 2; k <= d; ++k) acc = fma(kK[k - 1], T[d - k], acc);
                T[d] = acc * (1.0 / d);
            }
        }
        if constexpr (D > 8) {
            // the heavy tokens' exact factors, then each one's leave-one-out coefficient by series division
            double xh[kMaxHeavy];
            for (int hv = 0; hv < nheavy; ++hv) {
                double e[D];
#pragma unroll
                for (int a = 0; a < D; ++a) e[a] = L.trec[hv].e[a];
                xh[hv] = exp_neg(t * L.trec[hv].aw, L.e2tab);
                mul_factor<D>(T, xh[hv], e);
            }
            for (int hv = 0; hv < nheavy; ++hv) {
                double e[D];
#pragma unroll
                for (int a = 0; a < D; ++a) e[a] = L.trec[hv].e[a];
                const double term = (tsub == 0 ? qw : 0.0) * xh[hv] * loo_coeff<D>(T, xh[hv], e, n);
                hacc[hv] += term;
                hacct[hv] = fma(term, t, hacct[hv]);
            }
        }
        {
            NodeRec<D> rec;
            rec.t = t; rec.qw = qw;
            const double tn = pick_series<D, D>(rec, T, n);
            if (tsub == 0) { r0 = fma(qw, tn, r0); L.nrec[wv][at] = rec; }
            if (couple) {
            // the even nodes' series of the first kStar tokens: lane (k, tsub) takes token tsub at the k-th of them, its
            // mirror token 4 + tsub
            const bool upper = j >= 8;
            const int k = upper ? 15 - j : j, a = tsub + (upper ? 4 : 0);
            float Tr[D];
#pragma unroll
            for (int b = 0; b < D; ++b) {
                const float v = static_cast<float>(rec.Tr[b]), w = dpp_f<kDppMirror>(v);
                Tr[b] = upper ? w : v;
            }
            const double tq = 2.0 * kQuadStep * (node == 0 ? kQuadPair : 1.0) * t * es;
            const double tm = dpp_move<kDppMirror>(t), qm = dpp_move<kDppMirror>(tq);       // not inside the selection: every lane must be active
            const double te = upper ? tm : t, qe = upper ? qm : tq;
            const double tw = te * L.trec[a].aw;
            float* const out = &L.hser[wv][k * Lds<D, ST>::kSerStride + a * Lds<D, ST>::kSer];
            if (a >= nheavy) star_series<D>(Tr, L.trec[a].e, tw, qe, __expf(-static_cast<float>(fmin(tw, 1000.0))), out);
            else star_series_exact<D>(T, L.trec[a].e, tw, qe, exp_neg(tw, L.e2tab), n, out);
            // the heavy tokens' couplings among themselves: one pair per token subset
            if (nheavy >= 2) {
                const int pa = tsub == 2 ? 1 : 0, pb = tsub == 0 ? 1 : 2;
                double c = 0.0;
                if (tsub < 3 && pb < nheavy)
                    c = qw * t * heavy_pair<D>(T, L.trec[pa].e, L.trec[pb].e, exp_neg(t * L.trec[pa].aw, L.e2tab), exp_neg(t * L.trec[pb].aw, L.e2tab), n);
                c += dpp_move<kDppXor1>(c); c += dpp_move<kDppXor2>(c); c += dpp_move<kDppHalfMirror>(c); c += dpp_move<kDppMirror>(c);
                if (j == 0 && tsub < 3) L.hpair[wv][tsub] = c0 > 0 ? L.hpair[wv][tsub] + c : c;
            }
            }
        }
        wave_lds_sync();
        GR_CLK(L, 8);
        // ---- phase 3
        if constexpr (D > 4) phase3_range<D, D>(L, nheavy, nfull, m, npw, wv, lane);
        phase3_range<D, CL>(L, nfull, m, m, npw, wv, lane);
        // ---- phase 4
        if (couple) star_phase<D>(L, lane, wv, m, t, c0 > 0);
        wave_lds_sync();                                   // this wave's node records are rewritten by its next chunk
        GR_CLK(L, 9);
    }
    if constexpr (D > 8) {
        for (int hv = 0; hv < nheavy; ++hv) {
            const double a = wave_sum(hacc[hv]), b = wave_sum(hacct[hv]);
            if (lane == 0) { L.rpart[wv][hv] = a; L.spart[wv][hv] = b; }
        }
    }
    {
        const double r0w = wave_sum(r0);
        if (lane == 0) L.r0part[wv] = r0w;
    }
    if (tid == 0) L.work += static_cast<double>(N) * m;
}

// The same evaluation for up to eight drafts (no heavy tokens there), both phases in ONE lane layout: lane = (node j
// of the wave, token subset tsub), token row i of a lane = token NS i + tsub.  The factor x = e^{-t w} of a (node,
// token) pair is computed once, in phase 1, and stays in a register until phase 3 uses it again (NT = kMaxT / NS rows
// per lane; the row loops are unrolled so that the array is indexed by constants).  Phase 3 then needs the node's
// series, which this lane already holds, and the token's q; it ends with a sum over the NPW neighbouring lanes that
// hold the nodes of a subset.  No node records in LDS and no exchange between the phases.
// Rows whose first token is below L.nfull take all D cumulants, the others four.
// A wave owns four neighbouring nodes of a chunk of 32: most grids have 27 to 50 nodes, and the chunk behind the first is taken
// by as many waves as it has nodes for.  Eight nodes a wave and chunks of 64 left no wave out and took 217 us where this takes 210
// for a call of 256 rows of 128256 tokens (n = 8, k = 128), 660 and 634 for 1024 of them; 77 and 78 for 64 rows of 1024 (n = 4).
// The first row's lanes hold the factors of the first kStar tokens: lane (node, tsub) takes the series of token tsub.
template <int D, int ST>
__device__ __forceinline__ void eval_core_rows(Lds<D, ST>& L, const Grid& gr, int m_, int n_, double ctx, int slack_, bool couple) {
    constexpr int NPW = Lds<D, ST>::kNPW, NS = 64 / NPW, NT = kMaxT / NS;
    constexpr int CL = D < 4 ? D : 4;
    static_assert(D <= 8 && NPW == 4 && NS >= kStar, "four node lanes per subset; the first row holds the kStar");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // the sizes are the same in every lane; said so, the row guards below are scalar branches, not lane masks
    const int m = __builtin_amdgcn_readfirstlane(m_), n = __builtin_amdgcn_readfirstlane(n_);
    const int slack = __builtin_amdgcn_readfirstlane(slack_);
    const int nfull = (D > 4) ? __builtin_amdgcn_readfirstlane(L.nfull) : 0;
    const double t_lo = gr.t_lo;
    const int N = __builtin_amdgcn_readfirstlane(gr.N);
    const int j = lane & (NPW - 1), tsub = lane / NPW;
    const bool odd = j & 1;
    double r0 = 0.0;                                       // slack integrand, lanes of token subset 0
    GR_CLK(L, 6);

    if (NPW * wv >= N) {                                   // no node for this wave: its sums are 0
        for (int i = lane; i < m; i += 64) { L.rpart[wv][i] = 0.0; L.spart[wv][i] = 0.0; }
        if (couple) for (int i = lane; i < m * (kStar / 4); i += 64) *reinterpret_cast<float4*>(&L.cpart[wv][4 * i]) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int c0 = NPW * wv; c0 < N; c0 += Lds<D, ST>::kChunk) {  // this wave's first node of the chunk
        const bool more = c0 >= Lds<D, ST>::kChunk;             // its sums go on
        const int node = c0 + j;
        const double t = t_lo * exp(kQuadStep * static_cast<double>(node));
        const double es = node < N ? exp_neg(slack * t, L.e2tab) : 0.0, qw = node_weight(node, t, t_lo) * es;
        // ---- phase 1: cumulant sums at this lane's node over the tokens of its subset
        double K[D], xs[NT];
#pragma unroll
        for (int k = 0; k < D; ++k) K[k] = 0.0;
        // the weight of a row is requested one row ahead: it heads the longest chain (the exponential)
        double aw = L.trec[tsub].aw;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            xs[i] = 0.0;
            if (NS * i < m) {
                const TokRec<D>& rec = L.trec[NS * i + tsub];  // the records behind the last token have x = 0
                const double y = t * aw;
                if (i + 1 < NT) aw = L.trec[NS * (i + 1) + tsub].aw;
                const double x = exp_neg(y, L.e2tab);
                if (D > 4 && NS * i < nfull) phase1_token<D, D>(K, rec, x);
                else phase1_token<D, CL>(K, rec, x);
                xs[i] = x;
            }
        }
        // over the subsets: rotations within a row of sixteen lanes, then the four rows
#pragma unroll
        for (int k = 0; k < D; ++k) {
            K[k] += dpp_move<kDppRor8>(K[k]);
            K[k] += dpp_move<kDppRor4>(K[k]);
            K[k] += __shfl_xor(K[k], 16);
            K[k] += __shfl_xor(K[k], 32);
        }
        GR_CLK(L, 7);
        // ---- phase 2: the node's series T = exp(z ctx + sum_k K_k z^k), every lane of the node alike
        K[0] += ctx;
        double T[D + 1];
        T[0] = 1.0;
        {
            double kK[D];
#pragma unroll
            for (int k = 1; k <= D; ++k) kK[k - 1] = static_cast<double>(k) * K[k - 1];
#pragma unroll
            for (int d = 1; d <= D; ++d) {
                double acc = kK[0] * T[d - 1];
#pragma unroll
                for (int k = 2; k <= d; ++k) acc = fma(kK[k - 1], T[d - k], acc);
                T[d] = acc * (1.0 / d);
            }
        }
        double Tp[D];                                      // quadrature weight x T_{n-k} / k!
        {
            NodeRec<D> rec;
            const double tn = pick_series<D, D>(rec, T, n);
            if (tsub == 0) r0 = fma(qw, tn, r0);
            if (couple) {
                float Tr[D];
#pragma unroll
                for (int k = 0; k < D; ++k) Tr[k] = static_cast<float>(rec.Tr[k]);
                if (!odd && tsub < kStar)
                    star_series<D>(Tr, L.trec[tsub].e, t * L.trec[tsub].aw, 2.0 * kQuadStep * (node == 0 ? kQuadPair : 1.0) * t * es,
                                   static_cast<float>(xs[0]), &L.hser[wv][(j >> 1) * Lds<D, ST>::kSerStride + tsub * Lds<D, ST>::kSer]);
            }
            double invf = qw;
#pragma unroll
            for (int k = 1; k <= D; ++k) { invf *= 1.0 / k; Tp[k - 1] = rec.Tr[k - 1] * invf; }
        }
        GR_CLK(L, 8);
        // ---- phase 3: the leave-one-out coefficient of every pair, summed over the nodes of the wave.  The sums over
        // the four node lanes of a subset: the first step (lane k with lane k ^ 1) also parts the two sums, R to
        // the even lanes and its t-weighted companion S to the odd ones, so that the other step moves one value, not two.
        double qn = L.trec[tsub].e[0];
        double* const part = odd ? &L.spart[wv][0] : &L.rpart[wv][0];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            if (NS * i < m) {
                const int a = NS * i + tsub;                        // a <= kMaxT - 1: the sums of places past the last token are 0
                double old = 0.0;
                if (more && j < 2) old = part[a];
                const double q = qn;
                if (i + 1 < NT) qn = L.trec[a + NS].e[0];
                const double x = xs[i], v = fma(-x, x, x), s = fma(-2.0, x, 1.0);
                double top = 0.0;
                if (D > CL && NS * i < nfull) top = loo_top<D, CL>(Tp, q, v, s);
                const double r_ = x * loo_low<D, CL>(Tp, q, v, s, top), s_ = r_ * t;
                double k = odd ? s_ : r_;
                k += dpp_move<kDppXor1>(odd ? r_ : s_);
                k += dpp_move<kDppXor2>(k);
                if (j < 2) part[a] = old + k;
            }
        }
        // ---- phase 4
        if (couple) star_phase<D>(L, lane, wv, m, t, more);
        wave_lds_sync();                                   // the series are rewritten by the wave's next chunk
        GR_CLK(L, 9);
    }
    {
        const double r0w = wave_sum(r0);
        if (lane == 0) L.r0part[wv] = r0w;
    }
    if (tid == 0) L.work += static_cast<double>(N) * m;
}

template <int D, int ST>
__device__ __forceinline__ void eval_core(Lds<D, ST>& L, const Grid& gr, int m, int n, double ctx, int slack, bool couple) {
    if constexpr (D <= 8) eval_core_rows<D>(L, gr, m, n, ctx, slack, couple); else eval_core_nodes<D>(L, gr, m, n, ctx, slack, couple);
}

// The routed mass R of token `tok`, its t-weighted companion S (the share that the token loses to itself) and, with slack,
// its coupling to the slack vertex, from the waves' partial sums (behind the barrier that follows eval_core).
struct TokenSums { double R, S, b; };
template <int D, int ST>
__device__ __forceinline__ TokenSums token_sums(const Lds<D, ST>& L, const Grid& gr, int tok, double fact) {
    constexpr int kSW = Lds<D, ST>::kSW;
    const double rfact = fast_rcp(fact);
    double r = L.apd[tok] * gr.tail * rfact, sq = 0.0;           // the integrand of S is 0 at t = 0
#pragma unroll
    for (int w2 = 0; w2 < kSW; ++w2) {
        r += L.rpart[w2][tok]; sq += L.spart[w2][tok];
    }
    const double w = L.trec[tok].aw;
    TokenSums o;
    o.R = r * w * fact;
    o.b = sq * w * fact;
    o.S = o.b * w;
    return o;
}
template <int D, int ST>
__device__ __forceinline__ double slack_mass(const Lds<D, ST>& L, const Grid& gr, int n, double atot, double fact, int slack) {
    constexpr int kSW = Lds<D, ST>::kSW;
    double r0all = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < kSW; ++w2) r0all += L.r0part[w2];
    return (r0all * fact + ipow(atot, n) * gr.tail) * slack;
}
// The couplings of token `tok` to four of the kStar tokens (half: 0 or 1), times `scale`, into its row; none to itself.
template <int D, int ST>
__device__ __forceinline__ void token_couplings(Lds<D, ST>& L, const Grid& gr, int tok, int half, double scale) {
    constexpr int kSW = Lds<D, ST>::kSW;
    float c[4] = {0.f, 0.f, 0.f, 0.f};
    if (D > 8 && tok < L.nheavy) {
        // the other token's row, or the heavy pair's own sum
        for (int h = 0; h < 4; ++h) {
            const int o = 4 * half + h;
            double v = 0.0;
            if (o < L.nheavy) { if (o != tok) for (int w2 = 0; w2 < kSW; ++w2) v += L.hpair[w2][o + tok - 1]; }
            else for (int w2 = 0; w2 < kSW; ++w2) v += static_cast<double>(L.cpart[w2][o * kStar + tok]);
            v = o < L.nheavy ? v * L.trec[tok].aw * L.trec[o].aw * scale : v * L.trec[o].aw * scale;
            L.W[tok][o] = L.trec[o].aw < 1e300 && v > 0.0 ? static_cast<float>(v) : 0.f;
        }
        return;
    }
#pragma unroll
    for (int w2 = 0; w2 < kSW; ++w2) {
        const float4 v = *reinterpret_cast<const float4*>(&L.cpart[w2][tok * kStar + 4 * half]);
        c[0] += v.x; c[1] += v.y; c[2] += v.z; c[3] += v.w;
    }
    const double f = L.trec[tok].aw * scale;
#pragma unroll
    for (int h = 0; h < 4; ++h) c[h] = tok == 4 * half + h ? 0.f : fmaxf(static_cast<float>(static_cast<double>(c[h]) * f), 0.f);
    *reinterpret_cast<float4*>(&L.W[tok][4 * half]) = make_float4(c[0], c[1], c[2], c[3]);
}

// Workgroup-wide evaluation (the Newton fallback's): every thread passes the log weight of its own token and gets
// that token's routed mass back (also left in L.aR); returns the slack mass.  All threads call it.
struct Routed { double R0, R, S; };
template <int D, int ST>
__device__ __forceinline__ Routed routed_eval(Lds<D, ST>& L, int& par, int m, int n, double ctx, int slack, double qsum, double fact, double alpha) {
    const int tid = threadIdx.x;
    double w = 0.0;
    if (tid < m) { w = exp(alpha); L.trec[tid].aw = w; }
    double a[2] = {wave_sum(tid < m ? w : 0.0), wave_min(tid < m ? w : 1e300)};
    wg_reduce<2>(L, par, a, {kOpSum, kOpMin});              // its barrier also publishes the weights
    const Grid gr = make_grid(slack, ctx, a[0], a[1]);
    eval_core<D>(L, gr, m, n, ctx, slack, false);
    __syncthreads();
    Routed out;
    out.R = 0.0; out.S = 0.0;
    if (tid < m) { const TokenSums ts = token_sums<D>(L, gr, tid, fact); out.R = ts.R; out.S = ts.S; L.aR[tid] = out.R; }
    out.R0 = slack_mass<D>(L, gr, n, ctx + qsum, fact, slack);
    GR_CLK(L, 10);
    return out;
}

// One evaluation and the stopping measure: max_i | log(target_i / routed_i) - common term |, where the
// common term is log(slack_target / slack mass) with slack, log(sum target / sum routed) without
// (the latter is zero in exact arithmetic and removes the common quadrature error).  Per-token quantities are
// those of the calling thread's token: alpha and target in, f = log(target / routed) - common term, R and S out.
struct Defect { double err, f, R, S, rsum, R0; };
template <int D, int ST>
__device__ __forceinline__ Defect defect_eval(Lds<D, ST>& L, int& par, int m, int n, double ctx, int slack, double slack_target, double qsum,
                                              double tsum, double fact, double alpha, double target) {
    const int tid = threadIdx.x;
    Defect d;
    {
        const Routed r = routed_eval<D>(L, par, m, n, ctx, slack, qsum, fact, alpha);
        d.R0 = r.R0; d.R = r.R; d.S = r.S;
    }
    double g = 0.0;
    if (tid < m) { g = fast_log(target / d.R); if (!(g == g)) g = 1e301; }
    double a[3] = {wave_sum(tid < m ? d.R : 0.0), wave_max(tid < m ? g : -1e300), wave_min(tid < m ? g : 1e300)};
    wg_reduce<3>(L, par, a, {kOpSum, kOpMax, kOpMin});
    d.rsum = a[0];
    const double gmax = a[1], gmin = a[2];
    const double lc = fast_log(slack ? d.R0 / slack_target : d.rsum / tsum);
    d.f = tid < m ? g + lc : 0.0;
    double worst = fmax(fabs(gmax + lc), fabs(gmin + lc));
    if (!(worst == worst)) worst = 1e301;                  // NaN: treated as "no finite point"
    if (!(gmax < 1e300) || !(gmin > -1e300)) worst = 1e301;
    d.err = worst;
    GR_CLK(L, 11);
    return d;
}

// Damped Newton iteration on routed(alpha) = target with a finite-difference Jacobian (the Hessian of
// Theta_T / Phi_T in alpha), for programs on which the iteration of newton_step is slow (a target that
// nearly exhausts the tuples containing its token).  One step costs one evaluation per variable, so
// it only takes over when the iteration of newton_step has used up its budget.  Without slack the last weight
// is pinned (the system is singular along the common shift).  Starts from L.aal.
// J: this row's scratch in HBM, kMaxT rows of kMaxT + 1 doubles (the last column is the right-hand side).
// The cap counts the evaluations of this program only (`evals0` = the row's count when the program began).
template <int D, int ST>
__device__ int newton_program(Lds<D, ST>& L, int& par, double* J, int m, int n, double ctx, int slack, double slack_target, double qsum,
                              double tsum, double fact, double rel_tol, int max_evals, int* evals, int evals0) {
    constexpr int kSW = Lds<D, ST>::kSW;
    const int tid = threadIdx.x;
    const int nfree = slack ? m : m - 1;
    constexpr int LD = kMaxT + 1;
    constexpr double kFd = 1e-6;
    const double target = tid < m ? L.at[tid] : 0.0;
    Defect dd = defect_eval<D>(L, par, m, n, ctx, slack, slack_target, qsum, tsum, fact, tid < m ? L.aal[tid] : 0.0, target);
    double err = dd.err, rsum = dd.rsum, R0 = dd.R0, f = dd.f;
    *evals += 1;
    while (err > rel_tol && *evals - evals0 < max_evals && err < 1e300) {
        if (tid < m) { L.nR[tid] = L.aR[tid]; L.af[tid] = f; }
        // common ratio routed/target over all vertices, the slack vertex included: Newton aims at
        // routed_j = ratio * target_j, which is what the stopping measure asks for
        const double ratio = slack ? (rsum + R0) / (tsum + slack_target) : rsum / tsum;
        __syncthreads();
        for (int k = 0; k < nfree; ++k) {
            if (tid == k) L.aal[k] += kFd;
            __syncthreads();
            const Routed rk = routed_eval<D>(L, par, m, n, ctx, slack, qsum, fact, tid < m ? L.aal[tid] : 0.0);
            if (tid < nfree) J[tid * LD + k] = (rk.R - L.nR[tid]) / kFd;
            if (tid == k) L.aal[k] -= kFd;
            __syncthreads();
        }
        *evals += nfree;
        if (tid < nfree) { J[tid * LD + kMaxT] = L.at[tid] * ratio - L.nR[tid]; L.nused[tid] = 0; L.ncolof[tid] = -1; L.nstep[tid] = 0.0; }
        __syncthreads();
        // Gauss-Jordan with partial pivoting: thread r owns row r
        for (int c = 0; c < nfree; ++c) {
            const double mag = (tid < nfree && !L.nused[tid]) ? fabs(J[tid * LD + c]) : -1.0;
            const double best = block_max<kSW>(mag, L.redn);
            if (!(best > 0.0)) continue;                   // no pivot left in this column: its step stays 0
            const int who = static_cast<int>(block_min<kSW>(mag == best ? static_cast<double>(tid) : 1e9, L.redn));
            const double piv = J[who * LD + c];
            if (tid < nfree && tid != who) {
                const double fct = J[tid * LD + c] / piv;
                for (int jc = c; jc < nfree; ++jc) J[tid * LD + jc] -= fct * J[who * LD + jc];
                J[tid * LD + kMaxT] -= fct * J[who * LD + kMaxT];
            }
            if (tid == who) { L.nused[tid] = 1; L.ncolof[tid] = c; }
            __syncthreads();
        }
        if (tid < nfree && L.ncolof[tid] >= 0) {
            const int my_col = L.ncolof[tid];
            const double dg = J[tid * LD + my_col];
            L.nstep[my_col] = dg != 0.0 ? J[tid * LD + kMaxT] / dg : 0.0;
        }
        __syncthreads();
        const double smax = block_max<kSW>(tid < nfree ? fabs(L.nstep[tid]) : 0.0, L.redn);
        if (!(smax < 1e300)) break;
        const double clip = smax > 2.0 ? 2.0 / smax : 1.0;
        // slope of the objective along the step: grad . d with grad_j = routed_j - ratio * target_j
        double slope0 = block_sum<kSW>(tid < nfree ? (L.nR[tid] - L.at[tid] * ratio) * clip * L.nstep[tid] : 0.0, L.redn);
        if (!(slope0 < 0.0)) {
            // not a descent direction (noise in the difference quotients): take the plain
            // fixed-point step instead, which always is one
            if (tid < nfree) L.nstep[tid] = L.af[tid] / clip;
            __syncthreads();
            slope0 = block_sum<kSW>(tid < nfree ? (L.nR[tid] - L.at[tid] * ratio) * L.af[tid] : 0.0, L.redn);
        }
        if (tid < m) L.nsave[tid] = L.aal[tid];
        __syncthreads();
        // Backtracking on the slope: the objective is convex, so it decreases along the step as long
        // as the slope stays negative; accept the first lam whose slope is below half of |slope0|.
        double lam = 1.0, err2 = err;
        bool ok = false;
        for (int ls = 0; ls < 20 && !ok; ++ls) {
            if (tid < nfree) L.aal[tid] = L.nsave[tid] + lam * clip * L.nstep[tid];
            __syncthreads();
            dd = defect_eval<D>(L, par, m, n, ctx, slack, slack_target, qsum, tsum, fact, tid < m ? L.aal[tid] : 0.0, target);
            err2 = dd.err; rsum = dd.rsum; R0 = dd.R0; f = dd.f;
            *evals += 1;
            const double ratio2 = slack ? (rsum + R0) / (tsum + slack_target) : rsum / tsum;
            const double slope = block_sum<kSW>(tid < nfree ? (L.aR[tid] - L.at[tid] * ratio2) * clip * L.nstep[tid] : 0.0, L.redn);
            ok = (err2 < 1e300) && (slope <= 0.5 * fabs(slope0) || err2 < err);
            if (!ok) lam *= 0.5;
        }
        if (!ok) {                                 // no acceptable point along the direction: stop here
            if (tid < m) L.aal[tid] = L.nsave[tid];
            __syncthreads();
            break;
        }
        err = err2;
    }
    __syncthreads();
    return err <= rel_tol ? 0 : 1;
}

// One step of the iteration, by wave 0 alone behind the barrier that follows the evaluation: Newton's step on the program
// with a reduced Hessian.  The Hessian of Theta_T / Phi_T in the log weights, -dR_i / dalpha_j, is the Laplacian of the
// graph whose edges are the couplings C_ij (star_series), with the slack term as one more vertex (its edges S_i / w_i come
// with the masses): R_i is the sum of row i, S_i included.  The edges of the kStar tokens of largest target are known, and so is
// what is left of every other row; the light tokens' edges among themselves are taken to be in proportion to what is left of
// both rows, which is a star around one more vertex, the hub.  Light tokens then touch only the kStar, the slack and the hub: they
// are eliminated one by one, sum over i of W_i W_i^T / d_i on the matrix cores, and ten vertices remain.  Those are eliminated
// with every diagonal taken as the sum of its row's edges, so nothing is subtracted and float32 gives the step to 1e-5
// relative whatever the edges' sizes; the token of largest target is held, so its equation, the one whose rounding would
// hide the slack's, is the one left out; a token whose row is too light for float32 takes the fixed-point step, which is exact to first
// order there.  Rows of 40 to 512 tokens with one to three tokens that the draft favours and the target excludes by up to e^-800 (7577
// rows, n = 2..16) take 5.6 evaluations on average and 31 at most; the fixed-point iteration with Anderson mixing that stood here
// 10.1 and 90.
// Bound: the serial chain of the stepping wave (about 9 k cycles for up to 64 tokens) between two evaluations.  Against that iteration, both
// timed in turn, a call of 256 rows of 32000 tokens, n = 4, k = 64: 251 -> 150 us (its slowest row decides: 1.4 to 1.9 times on other
// rows); 64 rows of 1024, n = 4, k = 32: 119 -> 77; 256 rows of 128256, n = 8, k = 128: 264 -> 221.  Single rows: 1.25 times on average over 60,
// three of them slower (0.80 to 0.97), where both take the same three to five evaluations and a series of degree 16 makes the couplings dear.
// Compiled as a function of its own (not inlined) so that its values do not compete for registers with the evaluator's series.
// The uniform solver state travels in StepState; per-token values live in LDS (see solve_program).
// held: the token of largest target (0 up to eight drafts), and kPlainly where the fixed-point step has its turn.
struct StepState { int since, retreats, havePrev, held; double best_err; };
constexpr int kPlainly = 16;
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int D, int ST>
__device__ __attribute__((noinline)) StepState newton_step(StepState st, int m, int n, int slack, double ctx, double slack_target, double tsum,
                                                           double rel_tol, int evals, int evals0) {
    Lds<D, ST>& L = *reinterpret_cast<Lds<D, ST>*>(gr_lds_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const bool two = m > 64;                               // uniform: lane l holds tokens l and l + 64
    const int tk[2] = {lane, lane + 64};
    const bool on[2] = {tk[0] < m, tk[1] < m};
    double R[2] = {0.0, 0.0}, S[2] = {0.0, 0.0}, g[2] = {0.0, 0.0}, al[2] = {0.0, 0.0}, f[2] = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 2; ++u) if (on[u]) {
        R[u] = L.aR[tk[u]]; S[u] = L.aS[tk[u]]; g[u] = L.ag[tk[u]];
        al[u] = L.aal[tk[u]];
    }
    GR_CLK(L, 18);
    // stopping measure: max_i | log(target_i / routed_i) - common term |, the common term log(slack_target / slack
    // mass) with slack, log(sum target / sum routed) without (zero in exact arithmetic: it removes the common
    // quadrature error)
    const double rsum = L.ared[0][0] + L.ared[1][0], gmax = fmax(L.ared[0][1], L.ared[1][1]), gmin = fmin(L.ared[0][2], L.ared[1][2]);
    const double lc = slack ? L.alc : fast_log(rsum * fast_rcp(tsum));
    double err = fmax(fabs(gmax + lc), fabs(gmin + lc));
    if (!(err == err) || !(gmax < 1e300) || !(gmin > -1e300)) err = 1e301;      // NaN or infinite: "no finite point"
#ifdef GR_PHASE_CLOCKS
    if (tid == 0 && evals <= 24) L.errlog[evals - 1] = err;
#endif
    GR_CLK(L, 11);
    const bool astray = !(err < 1e300) || err > 100.0 * st.best_err;
    if (err <= rel_tol || (astray && (!(st.best_err < 1e300) || st.retreats >= kRetreats))) {
        if (lane == 0) { L.ctl_go = 0; L.ctl_bestok = st.best_err < 1e300 ? 1 : 0; if (err <= rel_tol) L.ctl_result = 0; }
        return st;
    }
    const bool better = err < st.best_err;
    if (astray) {
        // back to the best point, with half the step that was last taken from it
        ++st.retreats; st.havePrev = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) if (on[u]) { al[u] = L.aBest[tk[u]]; f[u] = 0.5 * L.fBest[tk[u]]; L.fBest[tk[u]] = f[u]; }
    } else {
        st.since = better ? 0 : st.since + 1;
        const double R0 = L.aR0, total = rsum + R0, mass = tsum + slack_target;
        const double inv = fast_rcp(mass), over = (total - mass) * inv, rho = 1.0 + over, share = fast_rcp(total);
        const double lrho = over * (1.0 - 0.5 * over);         // the masses sum to the tuples' mass, up to the quadrature's error
        // What a token's mass lacks, in a form that is nearly linear in its log weight: target - R below the target (there R
        // grows at most in proportion to the weight), R log(target / R) above it.  A target that takes more than half of
        // P = Pr[token drawn] saturates: R / (P - R) is what its weight moves (the single-draft rule), so its log odds set the
        // aim while that is the longer way.
        double rhs[2] = {0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 2; ++u) if (on[u]) {
            const double tr = L.at[tk[u]] * rho, lg = g[u] + lrho, P = L.apd[tk[u]];
            rhs[u] = lg > 0.0 ? tr - R[u] : R[u] * lg;
            const double room = P - R[u];
            if (u == 0 && lg > 0.0 && tr > kOddsFrom * P && room > 0.0)      // such a token is among the first
                rhs[u] = fmax(rhs[u], R[u] * room * fast_rcp(P) * (lg + fast_log(room * fast_rcp(fmax(P - tr, 1e-5 * P)))));
        }
        double rhs0 = 0.0;
        if (slack) { const double t0 = slack_target * rho, l0 = lrho - L.alc; rhs0 = l0 > 0.0 ? t0 - R0 : R0 * l0; }
        const double lack = (wave_sum(rhs[0] + rhs[1]) + rhs0) * share;       // the sum of a Laplacian's right-hand side is 0
        rhs0 = (rhs0 - lack * R0) * inv;
        // the tokens' rows: couplings to the kStar (in place), to the slack, what is left (light tokens), right-hand side, 1 / sum
        float wr[2][kRowW];
        bool alone[2] = {false, false};                        // tokens too light for the reduced system: they take the fixed-point step
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (u == 1 && !two) continue;
#pragma unroll
            for (int c = 0; c < kRowW; ++c) wr[u][c] = 0.f;
            if (on[u]) {
                rhs[u] = (rhs[u] - lack * R[u]) * inv;
                const float4 c0 = *reinterpret_cast<const float4*>(&L.W[tk[u]][0]), c1 = *reinterpret_cast<const float4*>(&L.W[tk[u]][4]);
                wr[u][0] = c0.x; wr[u][1] = c0.y; wr[u][2] = c0.z; wr[u][3] = c0.w;
                wr[u][4] = c1.x; wr[u][5] = c1.y; wr[u][6] = c1.z; wr[u][7] = c1.w;
                wr[u][8] = L.W[tk[u]][8];
                const float known = ((c0.x + c0.y) + (c0.z + c0.w)) + ((c1.x + c1.y) + (c1.z + c1.w)) + wr[u][8];
                wr[u][10] = static_cast<float>(rhs[u]);
                const float rest = fmaxf(static_cast<float>((R[u] - S[u]) * inv) - known, 0.f), d = known + rest;
                alone[u] = !(d >= kLightest);
                if (tk[u] >= kStar) { wr[u][9] = rest; wr[u][11] = alone[u] ? 0.f : __builtin_amdgcn_rcpf(d); }
            }
            if (tk[u] < max(m, kStar)) {
#pragma unroll
                for (int c = 0; c < kRowW; c += 4) *reinterpret_cast<float4*>(&L.W[tk[u]][c]) = make_float4(wr[u][c], wr[u][c + 1], wr[u][c + 2], wr[u][c + 3]);
            }
        }
        wave_lds_sync();
        GR_CLK(L, 16);
        // sum over the light tokens of W_i W_i^T / d_i, and of W_i rhs_i / d_i in column 10: lane = (vertex, token of a group of four)
        {
            const int c = lane & 15, g4 = lane >> 4, cc = c < kRowW ? c : kRowW - 1;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            for (int t0 = kStar; t0 < m; t0 += 32) {            // eight groups of four: their loads first, they are all that takes time
                float w[8], d[8];
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int t = min(t0 + 4 * r + g4, kMaxT - 1);
                    w[r] = L.W[t][cc]; d[r] = L.W[t][kRowW - 1];
                }
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const bool in = t0 + 4 * r + g4 < m;
                    acc[r & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(in && c < kNodes ? w[r] : 0.f, in && c <= kNodes ? w[r] * d[r] : 0.f, acc[r & 1], 0, 0, 0);
                }
            }
            *reinterpret_cast<float4*>(&L.Am[c][4 * g4]) = make_float4(acc[0][0] + acc[1][0], acc[0][1] + acc[1][1], acc[0][2] + acc[1][2], acc[0][3] + acc[1][3]);
        }
        wave_lds_sync();
        GR_CLK(L, 17);
        // lane i < 10 holds row i of the remaining vertices: their own edges and what the light tokens left
        float dl[kNodes];
        const int held = D > 8 ? __builtin_amdgcn_readfirstlane(st.held) & (kStar - 1) : 0;
        {
            const int i = min(lane, kNodes - 1);
            float a[kNodes], r1 = L.Am[kNodes][i];
#pragma unroll
            for (int k = 0; k < kNodes; ++k) a[k] = L.Am[i][k];
            if (lane < kStar) {
#pragma unroll
                for (int k = 0; k <= kStar; ++k) a[k] += wr[0][k];
                r1 += wr[0][10];
            } else if (lane == kStar) {
#pragma unroll
                for (int k = 0; k < kStar; ++k) a[k] += L.W[k][kStar];
                r1 += static_cast<float>(rhs0);
            }
            // Where heavy tokens stand first, the held one takes the place of vertex 0.  With a light one held the others' sum, which its equation hides, is rounding
            // over its own edges (six tokens, two drafts, the first one's target 1e-35: 68 evaluations).
            if (D > 8 && held != 0) {
                const int swapped = lane == 0 ? held : (lane == held ? 0 : lane);
                float other = 0.f;
#pragma unroll
                for (int k = 1; k < kStar; ++k) { other = k == held ? a[k] : other; a[k] = k == held ? a[0] : a[k]; }
                a[0] = other;
#pragma unroll
                for (int k = 0; k < kNodes; ++k) a[k] = __shfl(a[k], swapped);
                r1 = __shfl(r1, swapped);
            }
            float e[kNodes][kNodes], c[kNodes];
#pragma unroll
            for (int k = kNodes - 1; k >= 1; --k) {
                float ak[kNodes], s = 0.f;
#pragma unroll
                for (int x = 0; x < k; ++x) { ak[x] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a[x]), k)); s += ak[x]; }
                const float rk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r1), k));
                const float is = s >= kLightest ? __builtin_amdgcn_rcpf(s) : 0.f, fac = a[k] * is;
                c[k] = rk * is;
                r1 = fmaf(fac, rk, r1);
#pragma unroll
                for (int x = 0; x < k; ++x) { e[k][x] = ak[x] * is; a[x] = fmaf(fac, ak[x], a[x]); }
            }
            dl[0] = 0.f;
#pragma unroll
            for (int k = 1; k < kNodes; ++k) {
                float v = c[k];
#pragma unroll
                for (int x = 1; x < k; ++x) v = fmaf(e[k][x], dl[x], v);
                dl[k] = v;
            }
            if (D > 8 && held != 0) {
#pragma unroll
                for (int k = 1; k < kStar; ++k) { dl[0] = k == held ? dl[k] : dl[0]; dl[k] = k == held ? 0.f : dl[k]; }
            }
        }
        GR_CLK(L, 20);
        const float base = slack ? dl[kStar] : 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) if (on[u]) {
            float v = wr[u][10];
#pragma unroll
            for (int c = 0; c < kNodes; ++c) v = fmaf(wr[u][c], dl[c], v);
            v *= wr[u][11];
            if (u == 0) {
#pragma unroll
                for (int c = 0; c < kStar; ++c) v = lane == c ? dl[c] : v;
            }
            f[u] = alone[u] ? g[u] + lc : static_cast<double>(v - base);
        }
        // Where the couplings mislead (light tokens that meet only one another, tokens that saturate together, an acceptance near 0) the
        // measure stands still: after kTurn evaluations that did not take it to a tenth the fixed-point step and Newton's change turns, each
        // with its secant pair.  (Rows that ended at the cap: 31 to 52 evaluations; targets 1e-12 of the slack's 44 to 168: 17 to 33.)
        if (((evals - evals0) & (kTurn - 1)) == 0) {
            if (!(st.best_err < 0.1 * L.turn_err)) { st.held ^= kPlainly; st.havePrev = 0; }
            if (lane == 0) L.turn_err = st.best_err;
        }
        if (st.held & kPlainly) {
#pragma unroll
            for (int u = 0; u < 2; ++u) f[u] = on[u] ? g[u] + lc : 0.0;
        }
        const double plain[2] = {f[0], f[1]};                  // what the best point keeps: half of a secant step gone astray would still be one
        // A few programs are left with a linear rate by what the hub stands for: near the end a step is combined with the one
        // before it (one secant pair).
        if (err < kSecantBelow || evals - evals0 > kSecantAfter) {
            if (st.havePrev) {
                double df[2] = {0.0, 0.0}, da[2] = {0.0, 0.0};
#pragma unroll
                for (int u = 0; u < 2; ++u) if (on[u]) { df[u] = f[u] - L.fPrev[tk[u]]; da[u] = al[u] - L.aPrev[tk[u]]; }
                double v[2] = {df[0] * f[0] + df[1] * f[1], df[0] * df[0] + df[1] * df[1]};
                wave_reduce_many<2>(v, {kOpSum, kOpSum});
                const double gam = v[1] > 0.0 ? v[0] * fast_rcp(v[1]) : 0.0;
#pragma unroll
                for (int u = 0; u < 2; ++u) if (on[u]) { L.aPrev[tk[u]] = al[u]; L.fPrev[tk[u]] = f[u]; f[u] -= (da[u] + df[u]) * gam; }
            } else {
#pragma unroll
                for (int u = 0; u < 2; ++u) if (on[u]) { L.aPrev[tk[u]] = al[u]; L.fPrev[tk[u]] = f[u]; }
                st.havePrev = 1;
            }
        }
        const bool broken = __any(!(fabs(f[0]) < 1e300) || !(fabs(f[1]) < 1e300));   // a clipped NaN would pass for a step
        const bool fixed = st.since >= kStall || broken;
        if (fixed) {                 // the fixed-point step, which lowers the objective whatever the point
#pragma unroll
            for (int u = 0; u < 2; ++u) f[u] = on[u] ? g[u] + lc : 0.0;
            st.since = 0; st.havePrev = 0;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            f[u] = fmin(fmax(f[u], -kClip), kClip);
            if (better && on[u]) { L.aBest[tk[u]] = al[u]; L.fBest[tk[u]] = fixed ? f[u] : fmin(fmax(plain[u], -kClip), kClip); }
        }
        if (better) st.best_err = err;
    }
    double ws = 0.0, wm = 1e300, amax = -1e300;
#pragma unroll
    for (int u = 0; u < 2; ++u) if (on[u]) { al[u] += f[u]; amax = fmax(amax, al[u]); }
    if (!slack) amax = wave_max(amax); else amax = 0.0;   // without slack only differences of log weights matter
#pragma unroll
    for (int u = 0; u < 2; ++u) if (on[u]) {
        al[u] -= amax;
        const double w = exp_signed(al[u], L.e2tab);
        L.aal[tk[u]] = al[u]; L.trec[tk[u]].aw = w; ws += w; wm = fmin(wm, w);
    }
    ws = wave_sum(ws); wm = wave_min(wm);
    if (lane == 0) {
        L.ctl_grid = make_grid(slack, ctx, ws, wm); L.ctl_bestok = st.best_err < 1e300 ? 1 : 0;
        L.ctl_couple = err < kKeepBelow ? 0 : 1;
    }
    GR_CLK(L, 12);
    return st;
}

// Solve one program by Newton's iteration with a reduced Hessian (newton_step).  Returns 0 when converged.
// In: L.aq (decreasing), L.at (targets, already scaled to the tuple mass), L.aal (start log weights) and L.apos, the first three
// written by the thread of their token; qsum = sum aq, tsum = sum at.
// Out: L.aal, L.apos, in the program's own order of tokens.  Returns 0, 1 (not converged) or kDeferred.  `evals` counts evaluator calls (summed over the row's programs;
// max_iter caps this program's).
template <int D, int ST>
__device__ __forceinline__ int solve_program(Lds<D, ST>& L, int& par, double* newton_ws, int m, int n, double ctx, int slack, double slack_target,
                             double qsum, double tsum, double rel_tol, int max_iter, int* evals) {
    constexpr int kST = Lds<D, ST>::kST;
    const int tid = threadIdx.x;
    const int evals0 = *evals;
    if (n == 1) {
        // One draft: a tuple is a single token, so the routed mass of token i is q_i w_i / (1 + w_i)
        // with the slack term (the single-draft rule, w_i = t_i / (q_i - t_i) in closed form) and q_i
        // whatever the weights without it.
        // A scaled target at or above its token's draw probability has no finite weight: the program
        // is reported as not converged, like an iteration that ran into its cap.
        int stuck = 0;
        if (slack && tid < m) {
            const double d = L.aq[tid] - L.at[tid];
            stuck = !(d > 0.0);
            L.aal[tid] = stuck ? 690.0 : log(L.at[tid] / d);
        }
        return wg_sum(L, par, static_cast<double>(stuck)) > 0.0 ? 1 : 0;
    }
    const double atot = ctx + qsum;
    const int wvi = tid >> 6, lane = tid & 63;
    double q = 0.0;
    int me = tid, heavy = 0;
    if (tid < m) {
        q = L.aq[tid];
        // With more than 8 drafts the cumulant series of a token that dominates the draw mass loses digits to
        // cancellation: the (at most three) tokens above kHeavyShare keep their exact factor instead.
        heavy = (D > 8 && q > kHeavyShare * atot) ? 1 : 0;
    }
    if (m > kStar) {
        // the heavy tokens, then those of largest target, to the front: the kStar tokens whose couplings the steps know
        double t = 0.0, al = 0.0;
        int pos = 0;
        if (tid < m) { t = L.at[tid]; al = L.aal[tid]; pos = L.apos[tid]; L.nused[tid] = static_cast<int>(heavy ? 0x7F800000u - tid : (__float_as_uint(static_cast<float>(t)) & ~127u) | (127u - tid)); }
        __syncthreads();
        if (wvi == 0) {
            unsigned k0 = lane < m ? static_cast<unsigned>(L.nused[lane]) : 0u, k1 = lane + 64 < m ? static_cast<unsigned>(L.nused[lane + 64]) : 0u;
#pragma unroll
            for (int r = 0; r < kStar; ++r) {
                const unsigned top = wave_max_u(max(k0, k1));
                const unsigned long long h0 = __ballot(k0 == top), h1 = __ballot(k1 == top);
                const int at = h0 ? __ffsll(static_cast<long long>(h0)) - 1 : 63 + __ffsll(static_cast<long long>(h1));
                if (lane == 0) L.star[r] = at;
                if (at == lane) k0 = 0u;
                if (at == lane + 64) k1 = 0u;
            }
        }
        __syncthreads();
        if (tid < m) {
            int before = 0, place = -1;
#pragma unroll
            for (int r = 0; r < kStar; ++r) { const int x = L.star[r]; before += x < tid; if (x == tid) place = r; }
            me = place >= 0 ? place : tid + kStar - before;
            L.aq[me] = q; L.at[me] = t; L.aal[me] = al; L.apos[me] = pos;
        }
    }
    else if (D <= 8 && wvi == 0) {
        // the token of largest target to the front, where the step holds it; with more drafts heavy tokens may stand there
        const double t = tid < m ? L.at[tid] : 0.0, al = tid < m ? L.aal[tid] : 0.0;
        const int pos = tid < m ? L.apos[tid] : 0;
        const int big = (kStar - 1) - static_cast<int>(wave_max_u(tid < m ? (__float_as_uint(static_cast<float>(t)) & ~(kStar - 1u)) | (kStar - 1u - tid) : 0u) & (kStar - 1u));
        me = tid == 0 ? big : (tid == big ? 0 : tid);
        wave_lds_sync();
        if (tid < m) { L.aq[me] = q; L.at[me] = t; L.aal[me] = al; L.apos[me] = pos; }
    }
    int full = 0;
    if (tid < m) {
        // per-token series of e^{zq}: q^k / k! for k <= n (terms beyond z^n never reach the z^n coefficient)
        double e = 1.0;
#pragma unroll
        for (int a = 1; a <= D; ++a) {
            e = e * q * (1.0 / a);
            L.trec[me].e[a - 1] = a <= n ? e : 0.0;
        }
        L.trec[me].pad = 0.0;
        L.apd[me] = pow_diff(atot, q, n);
        // A token needs only four cumulants when the u^5 and later terms of its factor cannot change the z^n
        // coefficient by more than 1e-11 relative: C(n-1, 4) (q/atot)^4 / 5 < 1e-11 (always, up to four drafts).
        const double r = q / atot;
        double binom = 1.0;
        for (int c = 1; c <= 4; ++c) binom = binom * (n - c) / c;         // C(n-1, 4)
        full = (D > 4 && !(binom * r * r * r * r / 5.0 < 1e-11)) ? 1 : 0;
    }
    if (tid < 32) L.e2tab[tid] = exp2(-static_cast<double>(tid) / 32.0);
    if (tid >= m && tid < kMaxT + 4) {                     // every record behind the last token: x = 0, no mass
        TokRec<D>& z = L.trec[tid];
        z.aw = 1e300; z.pad = 0.0;
#pragma unroll
        for (int a = 0; a < D; ++a) z.e[a] = 0.0;
    }
    if (D > 4) {
        // the heavy tokens are the first nh; behind the kStar tokens come the others in decreasing q, those with all cumulants first
        double a[3] = {wave_sum(static_cast<double>(heavy)), wave_sum(static_cast<double>(full)), wave_sum(static_cast<double>(full && me >= kStar))};
        wg_reduce<3>(L, par, a, {kOpSum, kOpSum, kOpSum});
        const int nh = static_cast<int>(a[0]), nf = static_cast<int>(a[1]), rest = static_cast<int>(a[2]);
        if (tid == 0) { L.nheavy = nh < kMaxHeavy ? nh : kMaxHeavy; L.nfull = nf == 0 ? L.nheavy : min(m, kStar) + rest; }
    }
    __syncthreads();
    GR_CLK(L, 5);
    double fact = 1.0;
    for (int i = 2; i <= n; ++i) fact *= i;
    const int full_iters = (max_iter > kStarBudget + m) ? kStarBudget + m : max_iter;
    const int step_iters = kDefers<D, ST> ? min(full_iters, kPatience) : full_iters;
    // The iteration is steered by wave 0 alone (lane l holds tokens l and l + 64, so every reduction over the
    // tokens is a wave reduction and the step needs no workgroup exchange); all waves evaluate.  Per
    // iteration: barrier, evaluation by all waves, barrier, the waves' sums, barrier, the step by wave 0 (the others wait at the next
    // barrier).  Wave 0 hands over through L.ctl_*: whether to go on, and the quadrature grid of the new weights.
    // Wave-0 state: uniform scalars in registers, per-token values in LDS (L.aal, L.at, the best point and the last one, each with
    // its step).
    StepState st;
    st.since = 0; st.retreats = 0; st.havePrev = 0; st.held = 0; st.best_err = 1e300;
    if (wvi == 0) {
        if (D > 8) st.held = (kStar - 1) - static_cast<int>(wave_max_u(lane < min(m, kStar) ? (__float_as_uint(static_cast<float>(L.at[lane])) & ~(kStar - 1u)) | (kStar - 1u - lane) : 0u) & (kStar - 1u));
        const int tk[2] = {lane, lane + 64};
        const bool on[2] = {tk[0] < m, tk[1] < m};
        double ws = 0.0, wm = 1e300, amax = -1e300;
        if (!slack) {
#pragma unroll
            for (int u = 0; u < 2; ++u) if (on[u]) amax = fmax(amax, L.aal[tk[u]]);
            amax = wave_max(amax);
        } else amax = 0.0;
#pragma unroll
        for (int u = 0; u < 2; ++u) if (on[u]) {
            const double al = L.aal[tk[u]] - amax;
            const double w = exp_signed(al, L.e2tab);
            L.aal[tk[u]] = al; L.trec[tk[u]].aw = w; ws += w; wm = fmin(wm, w);
        }
        ws = wave_sum(ws); wm = wave_min(wm);
        if (lane == 0) { L.turn_err = 1.0; L.ctl_go = 1; L.ctl_result = 1; L.ctl_bestok = 0; L.ctl_couple = 1; L.ctl_grid = make_grid(slack, ctx, ws, wm); }
    }
    const double inv_mass = fast_rcp(tsum + slack_target);
    for (int it = 1; it <= step_iters; ++it) {
        __syncthreads();                                   // the weights and L.ctl of this iteration are in place
        if (!L.ctl_go) break;
        const Grid gr = L.ctl_grid;
        const bool couple = L.ctl_couple != 0;
        eval_core<D>(L, gr, m, n, ctx, slack, couple);
        *evals += 1;
        __syncthreads();                                   // every wave's partial sums are in place
        GR_CLK(L, 10);
        // one token per thread: the first two waves its routed mass R, the companion S and log(target / R), the next ones its
        // couplings, one thread the slack mass.  Done here side by side, not by the stepping wave for two tokens per lane.
        if (tid < kMaxT) {                                 // the first two waves, whole
            double R = 0.0, g = 0.0;
            if (tid < m) {
                const TokenSums ts = token_sums<D>(L, gr, tid, fact);
                R = ts.R;
                g = fast_log(L.at[tid] * fast_rcp(R));
                if (!(g == g)) g = 1e301;
                L.aR[tid] = R; L.aS[tid] = ts.S; L.ag[tid] = g;
                L.W[tid][kStar] = slack ? static_cast<float>(ts.b * inv_mass) : 0.f;
            }
            double a3[3] = {tid < m ? R : 0.0, tid < m ? g : -1e300, tid < m ? g : 1e300};
            wave_reduce_many<3>(a3, {kOpSum, kOpMax, kOpMin});
            if (lane == 0) { L.ared[wvi][0] = a3[0]; L.ared[wvi][1] = a3[1]; L.ared[wvi][2] = a3[2]; }
        } else {
            const int tok = tid & (kMaxT - 1), part = tid / kMaxT - 1;   // 256 threads: both halves by one of them
            if (couple && tok < m && part < 2) {
                token_couplings<D>(L, gr, tok, part, fact * inv_mass);
                if (kST == 2 * kMaxT) token_couplings<D>(L, gr, tok, 1, fact * inv_mass);
            }
            if (tid == kST - 1) {
                const double R0 = slack_mass<D>(L, gr, n, atot, fact, slack);
                L.aR0 = R0;
                if (slack) L.alc = fast_log(R0 * fast_rcp(slack_target));
            }
        }
        __syncthreads();
        if (wvi != 0) continue;
        st = newton_step<D, ST>(st, m, n, slack, ctx, slack_target, tsum, rel_tol, *evals, evals0);
    }
    __syncthreads();
    int result = L.ctl_result;
    const bool bestok = L.ctl_bestok != 0;
    GR_CLK(L, 12);
    if constexpr (kDefers<D, ST>) {
        if (result == 0 || !((L.ctl_go && step_iters < full_iters) || (full_iters < max_iter && bestok))) return result;
        if (bestok && tid < m) L.aal[tid] = L.aBest[tid];
        return kDeferred;
    }
    if (result != 0 && step_iters < max_iter && bestok) {
        if (tid < m) L.aal[tid] = L.aBest[tid];
        __syncthreads();
        result = newton_program<D>(L, par, newton_ws, m, n, ctx, slack, slack_target, qsum, tsum, fact, rel_tol, max_iter, evals, evals0);
        GR_CLK(L, 13);
    }
    return result;
}

// Build the active list of one program: the support positions in [lo, hi) that belong to T and have
// a positive target, in decreasing q (L.ordq lists the positions of H* and of the rest in that
// order).  Returns m (possibly > kMaxT, in which case nothing was written beyond kMaxT).
template <class LdsT>
__device__ int compact_active(LdsT& L, int lo, int hi, int kk) {
    constexpr int kSW = LdsT::kSW;
    const int tid = threadIdx.x;
    const int j = tid < kk ? L.ordq[tid] : -1;           // kk <= KS <= kST
    const int on = (j >= lo && j < hi && L.inT[j] && L.tgt[j] > 0.0) ? 1 : 0;
    // inclusive scan of `on` over the workgroup
    const int incl = wave_scan_i(on);
    int* wtot = reinterpret_cast<int*>(L.redn);
    if ((tid & 63) == 63) wtot[tid >> 6] = incl;
    __syncthreads();
    int base = 0, total = 0;
    for (int w = 0; w < kSW; ++w) { if (w < (tid >> 6)) base += wtot[w]; total += wtot[w]; }
    const int slot = base + incl - 1;
    if (on && slot < kMaxT) L.apos[slot] = j;
    __syncthreads();
    return total;
}

}  // namespace

// AGAIN: the launch for the rows that the one before has left (kernels of their own: the others stay as short as they were).
template <int D, int ST, bool AGAIN>
__global__ __launch_bounds__(ST, kWavesOf<D>) void solve_kernel(SolveParams sp) {
    constexpr int kST = Lds<D, ST>::kST, kSW = Lds<D, ST>::kSW;
    Lds<D, ST>& L = *reinterpret_cast<Lds<D, ST>*>(gr_lds_raw);
    const int tid = threadIdx.x;
    const int row = blockIdx.x;
    if (AGAIN && sp.info[row].status >= 0) return;
    const int n = sp.row_n ? sp.row_n[row] : sp.n, V = sp.V;
    const float* const prow = sp.p + (sp.row_at ? static_cast<size_t>(sp.row_at[row]) : static_cast<size_t>(row) * V);
    RowInfo info;
    info.support = 0; info.h = 0; info.status = GR_ROW_OK; info.iterations = 0;
    info.alpha_star = 0.0; info.res_total = 0.0; info.p_total = 0.0; info.q_total = 0.0; info.node_tokens = 0.0; info.p_ref = 0.0; info.inv_temp = 0.0; info.q_ref = 0.0;

    // ---- merge the slices
    SliceTotals found;
    int bad = 0;
    double p_ref = 0.0, inv_temp = 0.0, inv_temp_q = 0.0;
    if (sp.logits) {
        // rows given as logits: the slices' softmax sums are brought to the row's largest reference; q needs no
        // normaliser (it is renormalised over the support)
        const float T = sp.temperature[row];
        inv_temp = 1.0 / static_cast<double>(T);
        const float Td = sp.draft_temperature ? sp.draft_temperature[row] : T;
        inv_temp_q = 1.0 / static_cast<double>(Td);
        if (!(Td > 0.f) || !(Td <= 3.0e38f)) bad = 1;
        found = slice_totals<true>(sp.cand_count, sp.part_bad, sp.part_psum, sp.part_qsum, sp.part_pref, row, sp.splits, inv_temp);
        p_ref = static_cast<double>(found.ref); found.qtot = 1.0;
        if (!(found.ptot > 0.0) || !(found.ptot < 1e300) || !(found.ref > -3.0e38f)) bad = 1;
    } else {
        found = slice_totals<false>(sp.cand_count, sp.part_bad, sp.part_psum, sp.part_qsum, nullptr, row, sp.splits, 0.0);
        if (!(fabs(found.ptot - 1.0) <= 1e-3) || !(fabs(found.qtot - 1.0) <= 1e-3)) bad = 1;
    }
    bad |= found.bad;
    const int total = found.total;
    const double ptot = found.ptot, qtot = found.qtot;
    info.p_total = ptot; info.q_total = qtot; info.p_ref = p_ref; info.inv_temp = sp.logits ? inv_temp : 0.0;
    if (bad || total <= 0 || total > kSelCap) {
        if (tid == 0) {
            info.status = GR_ROW_BAD;
            info.alpha_star = __longlong_as_double(0x7ff8000000000000ll);
            sp.info[row] = info;
            sp.accept_prob[row] = __uint_as_float(0x7fc00000u);
            sp.status[row] = GR_ROW_BAD;
            if (sp.v_drafts) { sp.v_token[row] = -1; sp.v_accepted[row] = 0; }
        }
        return;
    }
    gather_keys<kST>(L.keys, sp.cand + static_cast<size_t>(row) * kSelCap, found, sp.splits);
    if (tid == 0) { L.count = 0; L.work = AGAIN ? sp.info[row].node_tokens : 0.0; }
#ifdef GR_PHASE_CLOCKS
    if (tid == 0) { for (int i = 0; i < 24; ++i) L.clk[i] = 0; L.clk_last = clock64(); }
#endif
    __syncthreads();
    unsigned long long theta = 0ull;
    if (total > sp.k) theta = block_kth_largest<kST>(L.keys, total, sp.k, L.hist, L.pick);
    int kk = min(total, sp.k);
    for (int i = tid; i < total; i += kST) {
        const unsigned long long key = L.keys[i];
        if (key >= theta) {
            const int slot = atomicAdd(&L.count, 1);
            if (slot < KS) { L.ids[slot] = key_id(key); L.accb[slot] = static_cast<double>(sp.logits ? key_logit(key) : key_q(key)); }
        }
    }
    __syncthreads();
    if (sp.tail_mass > 0.0 && !sp.logits) {
        // Nucleus cut of the draft (Sec. 5.1: top-p/k sampling of the draft restricts the domain): the candidates by
        // decreasing q (ties by token id), their running sum added one after the other, and the support ends with the
        // first token at which it reaches (1 - tail_mass) of the row's q mass.
        int qr_ = 0;
        if (tid < kk) {
            const double qa = L.accb[tid]; const int ta = L.ids[tid];
            for (int j = 0; j < kk; ++j) { const double qj = L.accb[j]; qr_ += static_cast<int>(qj > qa) | (static_cast<int>(qj == qa) & static_cast<int>(L.ids[j] < ta)); }
            L.qd[qr_] = qa;
        } else if (tid < padded(kk)) L.qd[tid] = 0.0;
        __syncthreads();
        {
#pragma clang fp contract(off)
            if ((tid >> 6) == 0) wave_sequential_scan_padded<kScan>(L.qd, L.S, kk, 0.0);
        }
        __syncthreads();
        const double need = (1.0 - sp.tail_mass) * qtot;
        const double first = block_min<kSW>((tid < kk && L.S[tid + 1] >= need) ? static_cast<double>(tid + 1) : static_cast<double>(kk), L.redn);
        const int keep = static_cast<int>(first);             // ranks 0 .. keep - 1 by q stay
        const bool stay = tid < kk && qr_ < keep;
        const int myid = tid < kk ? L.ids[tid] : 0; const double myq = tid < kk ? L.accb[tid] : 0.0;
        __syncthreads();
        if (stay) { L.ids[qr_] = myid; L.accb[qr_] = myq; }    // any order serves: the ranks are counted again below
        kk = keep;
        __syncthreads();
    }
    // unsorted: token ids in ids, q in accb (exact float values), p gathered into G0
    if (sp.logits) {
        // p = exp((t - p_ref) / T) (divided by the row's sum with the other p below), q = exp((d - largest d) / T),
        // and the two keys every order is decided on: d - t for the ratio (q/p is proportional to
        // exp((d - t) / T); exact for float32 logits) and d itself for q
        const double d = tid < kk ? L.accb[tid] : -1e300;
        const double dmax = block_max<kSW>(d, L.redn);
        if (tid < kk) {
            const double t = static_cast<double>(prow[L.ids[tid]]);
            L.G0[tid] = exp((t - p_ref) * inv_temp);
            L.dlt[tid] = logit_ratio_key(d, t, inv_temp_q, inv_temp); L.dval[tid] = d;
            L.accb[tid] = exp((d - dmax) * inv_temp_q);
        }
    } else if (tid < kk) L.G0[tid] = static_cast<double>(prow[L.ids[tid]]);
    if (tid < kk) { L.cnt0[tid] = 0; L.cnt1[tid] = 0; }
    __syncthreads();
    GR_CLK(L, 0);
    // ---- two orders from one pass of rank counting (`parts` threads share a token, each counts over a stretch
    // of the others): by decreasing q/p -- exact cross products (float x float fits a double), ties by id --
    // and by decreasing q, ties by id (the order in which truncation sets grow).
    {
        const int parts = kk <= kST / 4 ? 4 : (kk <= kST / 2 ? 2 : 1);
        const int per = kST / parts;                       // tokens a part can hold
        const int me = tid % per, part = tid / per;
        if (me < kk) {
            const int ta = L.ids[me];
            const int j0 = (kk * part) / parts, j1 = (kk * (part + 1)) / parts;
            int rank = 0, qrank = 0;
            if (sp.logits) {
                const double ka = L.dlt[me], da = L.dval[me];
#pragma unroll 4
                for (int j = j0; j < j1; ++j) {
                    const double kj = L.dlt[j], dj = L.dval[j];
                    const int lower = static_cast<int>(L.ids[j] < ta);
                    rank += static_cast<int>(kj > ka) | (static_cast<int>(kj == ka) & lower);
                    qrank += static_cast<int>(dj > da) | (static_cast<int>(dj == da) & lower);
                }
            } else {
                const double qa = L.accb[me], pa = L.G0[me];
#pragma unroll 4
                for (int j = j0; j < j1; ++j) {
                    const double qj = L.accb[j];
                    const double lhs = qj * pa, rhs = qa * L.G0[j];   // j before me?
                    const int lower = static_cast<int>(L.ids[j] < ta);
                    rank += static_cast<int>(lhs > rhs) | (static_cast<int>(lhs == rhs) & lower);
                    qrank += static_cast<int>(qj > qa) | (static_cast<int>(qj == qa) & lower);
                }
            }
            if (parts > 1) { atomicAdd(&L.cnt0[me], rank); atomicAdd(&L.cnt1[me], qrank); }
            else { L.cnt0[me] = rank; L.cnt1[me] = qrank; }
        }
        __syncthreads();
        if (tid < kk) {
            const int rank = L.cnt0[tid];
            L.rows().tok[rank] = L.ids[tid]; L.qd[rank] = L.accb[tid]; L.rows().pn[rank] = L.G0[tid] / ptot;
            L.byq[L.cnt1[tid]] = rank;                    // the token of q rank j sits at ratio rank byq[j]
        } else if (tid < padded(kk)) { L.rows().pn[tid] = 0.0; L.qd[tid] = 0.0; }
        __syncthreads();
    }
    GR_CLK(L, 1);
    // ---- prefix sums in the order, sequentially (bit-reproducible), then F(m) = P_m - Q_m^n
    {
#pragma clang fp contract(off)
        if ((tid >> 6) == 0) wave_sequential_scan_padded<kScan>(L.rows().pn, L.P, kk, 0.0);
        if ((tid >> 6) == 1) wave_sequential_scan_padded<kScan>(L.qd, L.S, kk, 0.0);
        __syncthreads();
        const double stot = L.S[kk];
        for (int m = tid; m <= kk; m += kST) {
            const double Qm = L.S[m] / stot;
            L.Q[m] = Qm;
            L.F[m] = (m == 0) ? 0.0 : L.P[m] - ipow(Qm, n);
            if (m < kk) L.qn[m] = L.qd[m] / stot;
        }
        __syncthreads();
    }
    // ---- one wave, no barriers: H* (the smallest minimising prefix), the suffix minima G of F, residuals,
    // targets and records (F(m) <= G(m+1) for m >= h; m = kk always), the block of every token, and the
    // order by decreasing q split into H* and the rest.  Lane l holds ranks 5 (63 - l) .. + 4 (kk + 1 <= 257): the suffix minima
    // are then a scan over the lanes.
    if ((tid >> 6) == 0) {
        constexpr int E = (KS + 1 + 63) / 64;
        const int lane = tid, m0 = (63 - lane) * E;
        double Fv[E];
#pragma unroll
        for (int e = 0; e < E; ++e) Fv[e] = (m0 + e <= kk) ? L.F[m0 + e] : 1e300;
        double lmin = Fv[0];
#pragma unroll
        for (int e = 1; e < E; ++e) lmin = fmin(lmin, Fv[e]);
        const double Fmin = wave_min(lmin);
        int lidx = 1 << 20;
#pragma unroll
        for (int e = E - 1; e >= 0; --e) if (Fv[e] == Fmin) lidx = m0 + e;
        const int hh = static_cast<int>(wave_min(static_cast<double>(lidx)));
        double sfx[E];
        sfx[E - 1] = Fv[E - 1];
#pragma unroll
        for (int e = E - 2; e >= 0; --e) sfx[e] = fmin(Fv[e], sfx[e + 1]);
        const double later = wave_scan_min(sfx[0]);        // min of F over this lane's ranks and all later ones
        double after = __shfl_up(later, 1);                // ... over the later ranks' lanes only
        if (lane == 0) after = 1e300;
        int fl[E], run = 0, cl[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int m = m0 + e;
            fl[e] = 0;
            if (m <= kk) {
                const double g = fmin(sfx[e], after);                                   // G(m)
                const double gn = (e < E - 1) ? fmin(sfx[e + 1], after) : after;         // G(m + 1), unused at m = kk
                fl[e] = (m >= hh && (m == kk || Fv[e] <= gn)) ? 1 : 0;
                L.flag[m] = fl[e];
                if (m < kk) {
                    const double r = (m >= hh) ? gn - g : 0.0;
                    L.rows().rho[m] = r; L.tgt[m] = L.rows().pn[m] - r;
                }
            }
            run += fl[e]; cl[e] = run;
        }
        const int from_here = wave_scan_i(run);            // records of this lane's ranks and all later ones
        const int nrec_ = __builtin_amdgcn_readlane(from_here, 63);
        const int base = nrec_ - from_here;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int m = m0 + e;
            if (m <= kk) {
                const int c = base + cl[e];
                if (fl[e]) L.blo[c] = m;                     // record number c (1-based) sits at rank m
                if (m < kk) L.blk[m] = (m >= hh) ? c : 0;    // token m (rank m+1) lies after record c
            }
        }
        // ordq: ratio ranks listed by decreasing q, the tokens of H* first (a stable split of the q order)
        constexpr int E4 = KS / 64;
        const int j0 = lane * E4;
        int rk[E4], in[E4], cin = 0, ci[E4];
#pragma unroll
        for (int e = 0; e < E4; ++e) {
            const int j = j0 + e;
            rk[e] = j < kk ? L.byq[j] : 0;
            in[e] = (j < kk && rk[e] < hh) ? 1 : 0;
            ci[e] = cin;                                   // members of H* among this lane's earlier entries
            cin += in[e];
        }
        const int base_in = wave_scan_i(cin) - cin;
#pragma unroll
        for (int e = 0; e < E4; ++e) {
            const int j = j0 + e;
            if (j < kk) {
                const int before_in = base_in + ci[e];
                L.ordq[in[e] ? before_in : hh + (j - before_in)] = rk[e];
            }
        }
        if (lane == 0) { L.pick[0] = hh; L.pick[1] = nrec_; }
    }
    __syncthreads();
    const int h = L.pick[0];
    const int nrec = L.pick[1];
    const int nblk = nrec - 1;
    GR_CLK(L, 2);
    // ---- truncation sets: fewest tokens by decreasing q with gamma_T <= tau / epsilon_T <= tau
    const double Qh = L.Q[h];
    {
#pragma clang fp contract(off)
        // running q mass in decreasing-q order: G0 <- q of H* in that order, G1 <- its sequential prefix sums; O0, O1: of the rest
        if (tid < kk) { const double q = L.qn[L.ordq[tid]]; if (tid < h) L.G0[tid] = q; else L.O0[tid - h] = q; }
        if (tid >= h && tid < padded(h)) L.G0[tid] = 0.0;
        if (tid >= kk - h && tid < padded(kk - h)) L.O0[tid] = 0.0;
        __syncthreads();
        if ((tid >> 6) == 0) wave_sequential_scan_padded<kScan>(L.G0, L.G1, h, 0.0);
        if ((tid >> 6) == 1) wave_sequential_scan_padded<kScan>(L.O0, L.O1, kk - h, Qh);
        __syncthreads();
        // the token at position t of that order has the mass G1[t] or O1[t - h] before it
        if (tid < kk) {
            const int j = L.ordq[tid];
            const double a = tid < h ? L.G1[tid] : L.O1[tid - h];
            const double an = (a > 0.0) ? ipow(a, n) : 0.0;
            L.inT[j] = (j < h) ? ((ipow(Qh, n) - an) > sp.tau) : ((1.0 - an) > sp.tau);
        }
    }
    // ---- start weights: target / Pr[token drawn within its system], inner ones in the slack's gauge
    if (tid < kk) {
        const int hi = (tid < h) ? h : L.blo[L.blk[tid] + 1];
        const double top = L.Q[hi];
        const double gauge = (tid < h) ? ipow(top, n) / (-L.F[h]) : 1.0;
        const double t = L.tgt[tid];
        L.wgt[tid] = AGAIN ? sp.weight[static_cast<size_t>(row) * KS + tid] : ((t > 0.0) ? gauge * t / pow_diff(top, L.qn[tid], n) : 0.0);
    }
    __syncthreads();

    GR_CLK(L, 3);
    // ---- policy object, but for the weights
    auto write_rows = [&]() {
        const size_t at = static_cast<size_t>(row) * KS + tid;
        if (tid < kk) { sp.order[at] = L.rows().tok[tid]; sp.block[at] = L.blk[tid]; sp.rho[at] = L.rows().rho[tid]; sp.pnorm[at] = L.rows().pn[tid]; }
    };
    if constexpr (!Lds<D, ST>::kKeeps) write_rows();

    // ---- the convex programs: program 0 = inner system, then every outer block of two or more tokens
    int status = GR_ROW_OK, evals = AGAIN ? sp.info[row].iterations : 0, par = 0;
    for (int b = (h > 0 ? 0 : 1); b <= nblk && status != GR_ROW_TRUNC_CAP; ++b) {
        const int lo = (b == 0) ? 0 : L.blo[b];
        const int hi = (b == 0) ? h : L.blo[b + 1];
        if (b > 0 && hi - lo < 2) continue;
        const int m = compact_active(L, lo, hi, kk);
        if (m > sp.max_T) { status = GR_ROW_TRUNC_CAP; break; }
        if (m == 0 || (b > 0 && m < 2)) continue;
        double w0 = 0.0, q0 = 0.0, t0 = 0.0;
        if (tid < m) {
            const int j = L.apos[tid];
            w0 = L.wgt[j]; q0 = L.qn[j]; t0 = L.tgt[j];
            L.aq[tid] = q0; L.aal[tid] = fast_log(w0);
        }
        // one exchange: the draw mass and the targets of the active tokens, their start weights, and (inner
        // system) the context = tokens of T with target 0 (weight 0): they fill tuples but take no mass
        double ex[4] = {wave_sum(q0), wave_sum(t0), wave_sum(w0),
                        wave_sum((b == 0 && tid < h && L.inT[tid] && !(L.tgt[tid] > 0.0)) ? L.qn[tid] : 0.0)};
        wg_reduce<4>(L, par, ex, {kOpSum, kOpSum, kOpSum, kOpSum});
        const double qa = ex[0], ta = ex[1], w0sum = ex[2];
        double ctx, scale, slack_target = 0.0;
        if (b == 0) {
            ctx = ex[3];
            const double mass = ipow(ctx + qa, n);
            scale = mass / (ta - L.F[h]);
            slack_target = -L.F[h] * scale;
        } else {
            ctx = L.Q[lo];
            scale = pow_diff(ctx + qa, qa, n) / ta;
        }
        if (tid < m) L.at[tid] = t0 * scale;
        GR_CLK(L, 4);
        const int rc = solve_program<D>(L, par, sp.newton_ws + static_cast<size_t>(row) * kMaxT * (kMaxT + 1), m, n, ctx, b == 0, slack_target,
                                        qa, ta * scale, sp.rel_tol, sp.max_iter - (AGAIN && sp.info[row].status == -1 - b ? kPatience : 0), &evals);
        if (rc != 0 && status == GR_ROW_OK) status = GR_ROW_ITER_CAP;
        const double wv = (tid < m) ? exp(L.aal[tid]) : 0.0;
        const double wsum = (b == 0) ? 1.0 : wg_sum(L, par, wv);
        if (tid < m && (!kDefers<D, ST> || rc >= 0 || L.ctl_bestok)) L.wgt[L.apos[tid]] = (b == 0) ? wv : wv * (w0sum / wsum);
        __syncthreads();
        if (kDefers<D, ST> && rc < 0) {
            if (tid < kk) sp.weight[static_cast<size_t>(row) * KS + tid] = L.wgt[tid];
            if (tid == 0) { RowInfo& left = sp.info[row]; left.status = -1 - b; left.iterations = evals; left.node_tokens = L.work; }
            return;
        }
    }

    if constexpr (Lds<D, ST>::kKeeps) write_rows();
    if (tid < kk) sp.weight[static_cast<size_t>(row) * KS + tid] = L.wgt[tid];
    info.support = kk; info.h = h; info.status = status; info.iterations = evals;
    info.alpha_star = 1.0 + L.F[h];
    info.res_total = -L.F[h];
    info.node_tokens = L.work;
    if (tid == 0) {
#ifdef GR_PHASE_CLOCKS
        { const long long now_ = clock64(); L.clk[14] += now_ - L.clk_last; for (int i = 0; i < 24; ++i) { info.clk[i] = L.clk[i]; info.errlog[i] = i < evals ? L.errlog[i] : 0.0; } }
#endif
        sp.info[row] = info;
        sp.accept_prob[row] = static_cast<float>(1.0 + L.F[h]);
        sp.status[row] = status;
    }
    // ---- the row's verification, when the drafts came with the call: the same routine as verify_kernel, run by the
    // first kThreads threads on the policy this workgroup has just written (visible to it behind the barrier).  The
    // other waves end here; a workgroup barrier waits for the waves that are still alive only.
    if (sp.v_drafts) {
        __syncthreads();
        if (tid >= kThreads) __builtin_amdgcn_endpgm();
        RowPolicy rp;
        const size_t at = static_cast<size_t>(row) * KS;
        rp.o = sp.order + at; rp.bl = sp.block + at; rp.wt = sp.weight + at; rp.rh = sp.rho + at; rp.rk = nullptr; rp.rid = nullptr;
        rp.pieces = sp.piece_psum ? sp.piece_psum + static_cast<size_t>(row) * sp.piece_stride : nullptr;
        rp.prefs = sp.piece_pref ? sp.piece_pref + static_cast<size_t>(row) * sp.piece_stride : nullptr;
        static_assert(sizeof(VerifyLds) <= sizeof(Lds<D, ST>), "the verification reuses the solve's LDS");
        verify_row(*reinterpret_cast<VerifyLds*>(gr_lds_raw), prow, V, n, rp, info,
                   sp.v_drafts + static_cast<size_t>(row) * sp.v_stride, sp.v_uniforms[row], sp.v_token + row, sp.v_accepted + row);
    }
}

// ---- full-vocabulary policies: the convex programs of a row whose steps 1-2 were done in HBM: the
// inner program over T inside H* and one outer program per block that holds two or more active
// tokens of T -- the same programs, in the same arithmetic, as the LDS-resident path.
template <int D, int ST, bool AGAIN>
__global__ __launch_bounds__(ST, kWavesOf<D>) void full_programs_kernel(FullParams fp) {
    constexpr int kST = Lds<D, ST>::kST, kSW = Lds<D, ST>::kSW;
    Lds<D, ST>& L = *reinterpret_cast<Lds<D, ST>*>(gr_lds_raw);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = blockIdx.x;
    const int n = fp.n, V = fp.V;
    const size_t vs = static_cast<size_t>(V) + 2;
    if (AGAIN && fp.info[row].status >= 0) return;
    RowInfo info = fp.info[row];
    if (!AGAIN && info.status != GR_ROW_OK) return;   // bad, or above the cap on |T|: sampled from p
    auto leave = [&](int b, int evals) { if (tid == 0) { RowInfo& left = fp.info[row]; left.status = -1 - b; left.iterations = evals; left.node_tokens = L.work; } };
    const int kk = info.support, h = info.h;
    const RowValues val(fp, info, row);
    const int* byq = fp.byq + row * vs;
    const float2* by_rank = fp.pairs + row * vs;
    const double* Q = fp.Q + row * vs; const double* rho = fp.rho + row * vs;
    const int* blo = fp.blo + row * vs; const int* bcount = fp.bcount + row * vs;
    double* weight = fp.weight + row * vs;
    const double Fh = -info.res_total, stot = Q[kk];
    auto qn = [&](int r) { return val.q(by_rank[r].y) / stot; };
    auto target = [&](int r) { return val.p(by_rank[r].x) - rho[r]; };
    if (tid == 0) L.work = AGAIN ? info.node_tokens : 0.0;
    __syncthreads();

    int status = GR_ROW_OK, evals = AGAIN ? info.iterations : 0, par = 0;
    // ---- inner program: T inside H* is the first tcount[0] entries of byq, already by decreasing q
    if (h > 0) {
        const int c_in = fp.tcount[3 * row];
        int m = 0;
        double ctx_part = 0.0;
        for (int base = 0; base < c_in; base += kST) {
            const int i = base + tid;
            const int r = i < c_in ? byq[i] : -1;
            const double t = r >= 0 ? target(r) : 0.0;
            const bool on = r >= 0 && t > 0.0;
            if (r >= 0 && !on) ctx_part += qn(r);
            const unsigned long long mask = __ballot(on);
            if (lane == 0) L.hist[wv] = __popcll(mask);
            __syncthreads();
            int slot = m + __popcll(mask & ((1ull << lane) - 1ull));
            int tile_total = 0;
            for (int w = 0; w < kSW; ++w) { if (w < wv) slot += L.hist[w]; tile_total += L.hist[w]; }
            if (on && slot < kMaxT) { L.apos[slot] = r; L.aq[slot] = qn(r); L.at[slot] = t; L.aal[slot] = log(weight[r]); }
            m += tile_total;
            __syncthreads();
        }
        const double ctx = block_sum<kSW>(ctx_part, L.redn);
        if (m > 0 && m <= kMaxT) {
            const double qa = block_sum<kSW>(tid < m ? L.aq[tid] : 0.0, L.redn);
            const double ta = block_sum<kSW>(tid < m ? L.at[tid] : 0.0, L.redn);
            const double mass = ipow(ctx + qa, n);
            const double scale = mass / (ta - Fh);
            const double slack_target = -Fh * scale;
            if (tid < m) L.at[tid] *= scale;
            __syncthreads();
            const int rc = solve_program<D>(L, par, fp.newton_ws + static_cast<size_t>(row) * kMaxT * (kMaxT + 1), m, n, ctx, 1, slack_target,
                                            qa, ta * scale, fp.rel_tol, fp.max_iter - (AGAIN && fp.info[row].status == -1 ? kPatience : 0), &evals);
            if (rc != 0) status = GR_ROW_ITER_CAP;
            if (tid < m && (!kDefers<D, ST> || rc >= 0 || L.ctl_bestok)) weight[L.apos[tid]] = exp(L.aal[tid]);
            if (kDefers<D, ST> && rc < 0) { leave(0, evals); return; }
            __syncthreads();
        }
    }
    // ---- outer programs: those blocks with two or more active tokens of T
    const int nblk = fp.nblk[row], c_out = fp.tcount[3 * row + 1], at_out = fp.tcount[3 * row + 2];
    for (int b0 = 1; b0 <= nblk; b0 += KS) {               // windows of KS blocks: L.flag lists the window's programs
        const int bme = b0 + tid;
        const bool need = tid < KS && bme <= nblk && bcount[bme] >= 2;
        const unsigned long long nmask = __ballot(need);
        if (lane == 0) L.hist[wv] = __popcll(nmask);
        __syncthreads();
        int pslot = __popcll(nmask & ((1ull << lane) - 1ull));
        int nprog = 0;
        for (int w = 0; w < kSW; ++w) { if (w < wv) pslot += L.hist[w]; nprog += L.hist[w]; }
        if (need) L.flag[pslot] = bme;                      // nprog <= KS
        __syncthreads();
        for (int pi = 0; pi < nprog; ++pi) {
            const int b = L.flag[pi];
            const int lo = blo[b], hi = blo[b + 1];
            // its active tokens, by decreasing q as T lists them
            int m = 0;
            for (int base = 0; base < c_out; base += kST) {
                const int i = base + tid, r = i < c_out ? byq[at_out + i] : -1;
                const double t = r >= lo && r < hi ? target(r) : 0.0;
                const bool on = t > 0.0;
                const unsigned long long mask = __ballot(on);
                if (lane == 0) L.hist[wv] = __popcll(mask);
                __syncthreads();
                int slot = m + __popcll(mask & ((1ull << lane) - 1ull));
                int tile_total = 0;
                for (int w = 0; w < kSW; ++w) { if (w < wv) slot += L.hist[w]; tile_total += L.hist[w]; }
                if (on && slot < kMaxT) { L.apos[slot] = r; L.aq[slot] = qn(r); L.at[slot] = t; L.aal[slot] = log(weight[r]); }
                m += tile_total;
                __syncthreads();
            }
            if (m < 2 || m > kMaxT) continue;               // cannot happen for a row with status OK
            const double qa = block_sum<kSW>(tid < m ? L.aq[tid] : 0.0, L.redn);
            const double ta = block_sum<kSW>(tid < m ? L.at[tid] : 0.0, L.redn);
            const double ctx = Q[lo] / stot;
            const double scale = pow_diff(ctx + qa, qa, n) / ta;
            const double w0sum = block_sum<kSW>(tid < m ? exp(L.aal[tid]) : 0.0, L.redn);
            if (tid < m) L.at[tid] *= scale;
            __syncthreads();
            const int rc = solve_program<D>(L, par, fp.newton_ws + static_cast<size_t>(row) * kMaxT * (kMaxT + 1), m, n, ctx, 0, 0.0,
                                            qa, ta * scale, fp.rel_tol, fp.max_iter - (AGAIN && fp.info[row].status == -1 - b ? kPatience : 0), &evals);
            if (rc != 0 && status == GR_ROW_OK) status = GR_ROW_ITER_CAP;
            const double wvv = (tid < m) ? exp(L.aal[tid]) : 0.0;
            const double wsum = block_sum<kSW>(wvv, L.redn);
            if (tid < m && (!kDefers<D, ST> || rc >= 0 || L.ctl_bestok)) weight[L.apos[tid]] = wvv * (w0sum / wsum);
            if (kDefers<D, ST> && rc < 0) { leave(b, evals); return; }
            __syncthreads();
        }
        __syncthreads();
    }
    if (tid == 0) {
        info.status = status; info.iterations = evals; info.node_tokens = L.work;
        fp.info[row] = info;
        fp.status[row] = status;
    }
}

// The kernel of the series degree D >= n (2, 4, 8, 16), so that each keeps its series in registers, and of the workgroup that suits the batch.
enum { kSolve, kPrograms };
enum { kWide, kSmall, kAgain };      // a workgroup to a compute unit, two, and one for the rows that those leave
struct Chosen { const void* kernel; int threads, lds; };
template <int D, int ST, bool AGAIN = false> Chosen chosen(int which) {
    return Chosen{which == kSolve ? reinterpret_cast<const void*>(solve_kernel<D, ST, AGAIN>) : reinterpret_cast<const void*>(full_programs_kernel<D, ST, AGAIN>),
                  ST, static_cast<int>(sizeof(Lds<D, ST>))};
}
template <int D> Chosen chosen_of(int which, int how) {
    return how == kSmall ? chosen<D, kNarrow>(which) : (how == kAgain ? chosen<D, kThreadsOf<D>, true>(which) : chosen<D, kThreadsOf<D>>(which));
}
static Chosen choose(int which, int n, int how) {
    if (n <= 2) return chosen_of<2>(which, how);
    if (n <= 4) return chosen_of<4>(which, how);
    if (n <= 8) return chosen_of<8>(which, how);
    return chosen<16, kThreadsOf<16>>(which);
}

// A batch on the workgroups that suit it.
template <class Params>
static hipError_t launch_rows(int which, Params params, hipStream_t stream) {
    const bool small = params.n <= 8 && params.B > most_rows(params.n);
    void* args[] = {&params};
    for (int how = small ? kSmall : kWide;; how = kAgain) {
        const Chosen c = choose(which, params.n, how);
        (void)hipLaunchKernel(c.kernel, dim3(params.B), dim3(c.threads), args, c.lds, stream);
        const hipError_t e = hipGetLastError();                  // which clears it: the next call asks again
        if (e != hipSuccess || how != kSmall) return e;
    }
}

hipError_t launch_full_programs(const FullParams& fp, hipStream_t stream) { return launch_rows(kPrograms, fp, stream); }

static_assert(sizeof(Lds<16>) + 20 * 1024 <= 160 * 1024,
              "the solve workgroup's state and one streaming workgroup of the next batch must fit the CU's LDS together");
static_assert(sizeof(Lds<8, kNarrow>) <= 80 * 1024 && sizeof(Lds<4, kNarrow>) <= 80 * 1024 && sizeof(Lds<2, kNarrow>) <= 80 * 1024, "two to a compute unit");

// The kernels that a handle of up to max_n drafts and max_B rows can launch; hbm: those of supports above kMaxSupport too.  (A handle for one row,
// its inputs and its drafts: 353 us with eight kernels, 407 with two more, in every gr_create.)
hipError_t solve_kernel_setup(int max_n, int max_B, bool hbm) {
    for (int which = kSolve; which <= (hbm ? kPrograms : kSolve); ++which)
        for (int how = kWide; how <= kAgain; ++how)
            for (int n = 2; n <= GR_MAX_N && (n == 2 || n < 2 * max_n); n *= 2) {   // n: the series degrees that serve up to max_n
                if (how != kWide && (n > 8 || max_B <= most_rows(n == 2 ? 1 : n))) continue;   // the lowest line of the draft counts that it serves
                const Chosen c = choose(which, n, how);
                const hipError_t e = hipFuncSetAttribute(c.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, c.lds);
                if (e != hipSuccess) return e;
            }
    return hipSuccess;
}

hipError_t launch_solve(const SolveParams& sp, hipStream_t stream) { return launch_rows(kSolve, sp, stream); }

}  // namespace gr
