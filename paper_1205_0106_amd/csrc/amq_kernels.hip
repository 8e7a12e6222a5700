// amq_kernels.hip — gfx950 kernels for quasi-Monte Carlo American option
// valuation (Cvetanoska & Stojanovski; method in Sections III.D, III.E, V).
//
//   gen_kernel:   Sobol point -> Moro inverse normal -> Brownian bridge ->
//                 GBM value, stored path-contiguous as S[date][path].
//   paper_kernel: the paper's own per-path estimator.
// The backward-induction kernels live in amq_sweep.h (instantiated per
// precision and basis kind in amq_sweep_*.hip); this file dispatches to them.
//
// Compiled for gfx950 only.
#include "amq_math.h"
#include "amq_sync.h"

#include <math.h>

#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

namespace amq {

// a schedule node through the scalar cache
using GenNodeC = const __attribute__((address_space(4))) GenNode;

// ---------------------------------------------------------------------------
// Moro's inverse cumulative normal (Section III.D names it; coefficients from
// Moro 1995, "The full Monte", Risk 8(2)).  Central region |u - 1/2| < 0.42:
// Beasley–Springer rational function; tails: polynomial in log(-log q) where
// q is the tail probability, taken from the exact integer complement.
// ---------------------------------------------------------------------------
#define AMQ_A0 2.50662823884
#define AMQ_A1 -18.61500062529
#define AMQ_A2 41.39119773534
#define AMQ_A3 -25.44106049637
#define AMQ_B0 -8.47351093090
#define AMQ_B1 23.08336743743
#define AMQ_B2 -21.06224101826
#define AMQ_B3 3.13082909833
#define AMQ_C0 0.3374754822726147
#define AMQ_C1 0.9761690190917186
#define AMQ_C2 0.1607979714918209
#define AMQ_C3 0.0276438810333863
#define AMQ_C4 0.0038405729373609
#define AMQ_C5 0.0003951896511919
#define AMQ_C6 0.0000321767881768
#define AMQ_C7 0.0000002888167364
#define AMQ_C8 0.0000003960315187

// log(v) in binary64 for finite v > 0 (normal) by Tang's table method (P. T.
// P. Tang, "Table-driven implementation of the logarithm function in IEEE
// floating-point arithmetic", ACM TOMS 16(4), 1990): v = m 2^e with m in
// [1/2, 1); F = 1/2 + j/128 + 1/256 from the top 6 fraction bits j of m, so
// f = m - F is exact and |u| = |f / F| <= 2^-7; log v = e ln 2 + log F +
// log1p(u), log1p by its Taylor series to degree 7 (truncation below 2e-18).
// kLogTab[j] = log F rounded to nearest from a 60-digit decimal evaluation.
// About 1 ulp for the tail's arguments (results of magnitude 0.9 and more).
__constant__ double kLogTab[64] = {
    -0x1.5ee82aa241920p-1, -0x1.5707a26bb8c66p-1, -0x1.4f45a835a4e19p-1, -0x1.47a1527e8a2d3p-1,
    -0x1.4019c2125ca93p-1, -0x1.38ae2171976e7p-1, -0x1.315da4434068bp-1, -0x1.2a2786d0ec107p-1,
    -0x1.230b0d8bebc98p-1, -0x1.1c07849ae6007p-1, -0x1.151c3f6f29612p-1, -0x1.0e4898611cce1p-1,
    -0x1.078bf0533c568p-1, -0x1.00e5ae5b207abp-1, -0x1.f4aa7ee03192dp-2, -0x1.e7b42c3ddad73p-2,
    -0x1.dae75484c9616p-2, -0x1.ce42f18064743p-2, -0x1.c1c60693fa39ep-2, -0x1.b56fa04462909p-2,
    -0x1.a93ed3c8ad9e3p-2, -0x1.9d32bea15ed3bp-2, -0x1.914a8635bf68ap-2, -0x1.85855776dcbfbp-2,
    -0x1.79e26687cfb3ep-2, -0x1.6e60ee6af1972p-2, -0x1.630030b3aac49p-2, -0x1.57bf753c8d1fbp-2,
    -0x1.4c9e09e172c3cp-2, -0x1.419b423d5e8c7p-2, -0x1.36b6776be1117p-2, -0x1.2bef07cdc9354p-2,
    -0x1.214456d0eb8d4p-2, -0x1.16b5ccbacfb73p-2, -0x1.0c42d676162e3p-2, -0x1.01eae5626c691p-2,
    -0x1.ef5ade4dcffe6p-3, -0x1.db13db0d48940p-3, -0x1.c6ffbc6f00f71p-3, -0x1.b31d8575bce3dp-3,
    -0x1.9f6c407089664p-3, -0x1.8beafeb38fe8cp-3, -0x1.7898d85444c73p-3, -0x1.6574ebe8c133ap-3,
    -0x1.527e5e4a1b58dp-3, -0x1.3fb45a59928ccp-3, -0x1.2d1610c86813ap-3, -0x1.1aa2b7e23f72ap-3,
    -0x1.08598b59e3a07p-3, -0x1.ec739830a1120p-4, -0x1.c885801bc4b23p-4, -0x1.a4e7640b1bc38p-4,
    -0x1.8197e2f40e3f0p-4, -0x1.5e95a4d9791cbp-4, -0x1.3bdf5a7d1ee64p-4, -0x1.1973bd1465567p-4,
    -0x1.eea31c006b87cp-5, -0x1.aaef2d0fb10fcp-5, -0x1.67c94f2d4bb58p-5, -0x1.252f32f8d183fp-5,
    -0x1.c63d2ec14aaf2p-6, -0x1.432a925980cc1p-6, -0x1.82448a388a2aap-7, -0x1.0080559588b35p-8,
};

// exp(x) in binary64 by Tang's table method (P. T. P. Tang, "Table-driven
// implementation of the exponential function in IEEE floating-point
// arithmetic", ACM TOMS 15(2), 1989): n = rint(64 x / ln 2), g = x - n ln 2 / 64
// (Cody-Waite: ln 2 / 64 split into a 53-bit head and its tail, each product
// taken exactly inside an fma), |g| <= ln 2 / 128; exp(x) = 2^(n div 64)
// 2^((n mod 64) / 64) e^g, with e^g - 1 by its Taylor series to degree 5
// (truncation below 0.0055^6 / 6! < 4e-17 relative) and the table value
// added last.  kExpTab[j] = 2^(j / 64) rounded to nearest from a 60-digit
// decimal evaluation.  tab(j) reads the table (the path generator's LDS
// copy).  For the log-prices the generator produces (|x| < 700).
__constant__ double kExpTab[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};

// WIDE: any x (2^(n div 64) by ldexp, the table plain), brought into
// [-kWideExp, kWideExp] first: the value is 0 or infinite at either end, and n
// stays an integer that the sum's low word holds (from |x| = 2.3e7 it would
// wrap: a path whose drift takes it far below 0 came out infinite).  A NaN
// stays one.  Otherwise for |x| < 700: the table's entries come less j 2^46 in
// their bits (exp_tab_entry), and adding n 2^46 gives 2^(n / 64) whole.  The
// same values.
constexpr double kWideExp = 2000.0;
template <bool WIDE>
__device__ __forceinline__ double exp_tab_entry(uint32_t j)
{
    const uint64_t b = (uint64_t)__double_as_longlong(kExpTab[j]);
    return __longlong_as_double((long long)(WIDE ? b : b - ((uint64_t)j << 46)));
}

template <bool WIDE, typename Tab>
__device__ __forceinline__ double exp_tab(double x, Tab tab)
{
    if (WIDE) x = x < -kWideExp ? -kWideExp : x > kWideExp ? kWideExp : x;
    // n = rint(64 x / ln 2) by adding 1.5 2^52: the integer is in the sum's low
    // word (two's complement), no rounding and conversion instructions
    const double r = fma3s(x, 92.332482616893658, 0x1.8p52);  // 64 / ln 2
    const double n = r - 0x1.8p52;
    const uint32_t ni = (uint32_t)(uint64_t)__double_as_longlong(r);
    const double g = fma(-n, 3.6235106466348431e-19, fma(-n, 0.010830424696249145, x));
    double p = fma3s(1.0 / 120.0, g, kInvFact4);                // 1/4! (see exp_poly)
    p = fma3s(p, g, 1.0 / 6.0);
    p = fma(p, g, 0.5);
    p = fma(p, g, 1.0);
    double t = tab(ni & 63u);
    if (WIDE) return ldexp(fma(t, p * g, t), (int)ni >> 6);
    t = __hiloint2double((int)((uint32_t)__double2hiint(t) + (ni << 14)), __double2loint(t));
    return fma(t, p * g, t);
}

// F of interval j.
__device__ __forceinline__ double log_tab_centre(uint32_t j) { return fma((double)j, 0x1p-7, 0.5 + 0x1p-8); }

// log(m 2^e), m in [1/2, 1).  tab(j): {1 / F, log F} (the path generator's LDS
// table, 1 / F by the reciprocal's Newton refinement).  F itself is m with
// the bits below the interval's replaced by its midpoint's.
struct LogEntry { double rcp, log; };
template <typename Tab>
__device__ __forceinline__ double log_tab(double m, int e, Tab tab)
{
    const uint32_t hi = (uint32_t)((uint64_t)__double_as_longlong(m) >> 32);
    const LogEntry t = tab((hi >> 14) & 63u);
    const double F = __longlong_as_double((long long)((uint64_t)((hi & 0xFFFFC000u) | 0x2000u) << 32));
    const double u = (m - F) * t.rcp;
    double p = fma3s(1.0 / 7.0, u, -1.0 / 6.0);
    p = fma3s(p, u, 0.2);
    p = fma3s(p, u, -0.25);
    p = fma3s(p, u, 1.0 / 3.0);
    p = fma(p, u, -0.5);
    const double l1p = fma(p, u * u, u);
    const double de = (double)e;
    return fma(de, 0.69314718055994529, fma(de, 2.3190468138462996e-17, t.log + l1p));
}

// The inverse normal's two branches separately: which branch a point takes,
// the central rational function and the tail polynomial (its two logarithms
// by log_tab).  The path generator evaluates the tails packed.  MID: shifted
// (randomised) points sit at cell midpoints u = (x + 1/2) 2^-32, so a shifted
// integer 0 still maps to a finite normal.
template <bool MID> struct Moro {
    // Points come as xc = x ^ 2^31 (x - 2^31 as a signed integer).
    // d = x - 2^31 (+ 1/2) exactly; y = u - 1/2 = d 2^-32.  The branch test and the central
    // rational are taken on d with every constant scaled by a power of two,
    // which leaves each rounded intermediate scaled by the same power: the
    // values are bitwise those of the same steps on y (no under- or overflow
    // here).
    static __device__ __forceinline__ double centered(uint32_t xc)
    {
        const double d = (double)(int32_t)xc;
        return MID ? d + 0.5 : d;
    }
    static __device__ __forceinline__ bool tail(double d)
    {
        return !(fabs(d) < 0.42 * 0x1p32);   // |y| >= 0.42
    }
    static __device__ __forceinline__ double central(double d)
    {
        // y P(r) / Q(r), r = y^2 = D 2^-64: Horner in D with the k-th
        // coefficient of P scaled by 2^(-64k - 32) (the y factor's 2^-32
        // folded in) and of Q (beyond the constant 1) by 2^(-64(k + 1))
        const double D = d * d;
        const double num = d * fma3(fma3(fma3(AMQ_A3 * 0x1p-224, D, AMQ_A2 * 0x1p-160), D, AMQ_A1 * 0x1p-96),
                                    D, AMQ_A0 * 0x1p-32);
        const double den = fma(fma3(fma3(fma3(AMQ_B3 * 0x1p-256, D, AMQ_B2 * 0x1p-192), D, AMQ_B1 * 0x1p-128),
                                    D, AMQ_B0 * 0x1p-64),
                               D, 1.0);
        return num * rcp_f64(den);   // (a tail point's value is discarded)
    }
    template <typename Tab>
    static __device__ __forceinline__ double tail_value(uint32_t xc, Tab tab)
    {
        const uint32_t x = xc ^ 0x80000000u;
        // 2^32 q: the distance from the nearer end, an exact integer (+ 1/2);
        // the first logarithm takes the 2^-32 off the exponent
        const uint32_t k = min(x, MID ? ~x : 0u - x);
        double qd = (double)k;
        if (MID) qd += 0.5;
        const double l = -log_tab(__builtin_amdgcn_frexp_mant(qd), __builtin_amdgcn_frexp_exp(qd) - 32, tab);
        const double t = log_tab(__builtin_amdgcn_frexp_mant(l), __builtin_amdgcn_frexp_exp(l), tab);
        double v = fma3s(AMQ_C8, t, AMQ_C7);
        v = fma3s(v, t, AMQ_C6);
        v = fma3s(v, t, AMQ_C5);
        v = fma3s(v, t, AMQ_C4);
        v = fma3s(v, t, AMQ_C3);
        v = fma3s(v, t, AMQ_C2);
        v = fma3s(v, t, AMQ_C1);
        v = fma3s(v, t, AMQ_C0);
        // v > 0; the lower tail (x < 2^31) is its negative
        const uint64_t b = (uint64_t)__double_as_longlong(v);
        return __longlong_as_double((long long)(b ^ ((uint64_t)(~x & 0x80000000u) << 32)));
    }
};

// The bridge window: 16 binary64 values in v[96:127], the last registers of
// the generators' 128, so that a node's slots (run-time numbers, the same in
// every lane) index them in the instructions themselves (GPR index mode)
// rather than through two moves an access: 4 vector instructions a node where
// the compiler's indexing of an array took 9.
typedef double Window __attribute__((ext_vector_type(16)));
static_assert(kMaxSlots <= 16, "bridge window");

// xv = wl X[l] + wr X[r] + sd z, X[dst] = xv; slots: byte q twice the slot of
// l, r, dst (the index mode takes the low byte of its operand).
__device__ __forceinline__ double bridge_step(Window &X, uint32_t slots, double wl, double wr, double sd, double z)
{
    double t;
    const uint32_t sr = slots >> 8, sw = slots >> 16;
    asm("s_set_gpr_idx_on %[sr], 0x2\n\t"                      // second operand indexed
        "v_mul_f64 %[t], %[wr], v[96:97]\n\t"
        "s_set_gpr_idx_idx %[sl]\n\t"
        "v_fma_f64 %[t], %[wl], v[96:97], %[t]\n\t"
        "s_set_gpr_idx_off\n\t"
        "v_fma_f64 %[t], %[sd], %[z], %[t]\n\t"
        "s_set_gpr_idx_on %[sw], 0x8\n\t"                      // destination indexed
        "v_mov_b64 v[96:97], %[t]\n\t"
        "s_set_gpr_idx_off"
        : [t] "=&v"(t), "+{v[96:127]}"(X)
        : [sl] "s"(slots), [sr] "s"(sr), [sw] "s"(sw), [wl] "s"(wl), [wr] "s"(wr), [sd] "s"(sd), [z] "v"(z)
        : "m0");
    return t;
}

// ---------------------------------------------------------------------------
// Generation.  One wave owns 64 consecutive paths i = 64w + lane (Sobol index
// n = i + 1) and walks R such blocks.  Sobol (Gray-code order): for n = h + l
// with h a multiple of 64 and l < 64, gray(n) = gray(h) ^ gray(l), so
//   x_j(n) = X_j(h) ^ x_j^lo(l).
// X_j(h) is wave-uniform (kept per wave in LDS as the pair for h = 64w and
// h = 64(w+1), because lane 63 has n = 64(w+1)); x^lo comes from two 8-entry
// lane tables per dimension (bits 0-2 and 3-5 of gray(l)).  Moving to the
// next block: X(64(w+1)) = X(64w) ^ V[5] ^ V[6 + ctz(w+1)].  The tables are
// laid out in schedule order, so a chunk's reads are one running address and
// immediate offsets and wait for no node field.
//
// The bridge runs in depth-first order over a register window of ancestor
// values (slots chosen on the host), so a path never needs more than
// log2(M) + 2 live values; dimension order follows the breadth-first node
// numbering, which only changes the order the Sobol dimensions are read.
// ---------------------------------------------------------------------------
// One workgroup's share: `init` (the group holding the option's first block)
// writes the option's date constants and clears its barrier words; wave
// blocks [w0, w1) are generated.
template <typename T, int WHAT, bool MID, bool WIDE>
__device__ __forceinline__ void gen_body(const GenArgs &a, const uint32_t *__restrict__ V,
                                         const GenNode *__restrict__ sched, int len,
                                         const uint32_t *__restrict__ shift, bool init, int64_t w0,
                                         int64_t w1)
{
    extern __shared__ __align__(16) char lds[];
    const int M = a.M;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the wave's block range in scalar registers (it is the same in every
    // lane), so each store's row address is scalar and the lane's offset a
    // constant
    const auto uniform_i64 = [](int64_t v) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
    };
    w0 = uniform_i64(w0);
    w1 = uniform_i64(w1);
    double *etab = reinterpret_cast<double *>(lds);
    LogEntry *ltab = reinterpret_cast<LogEntry *>(lds + kLdsLog);
    // this wave's tail staging and the lane's spare word, as LDS addresses
    using LdsU32 = __attribute__((address_space(3))) uint32_t *;
    using LdsF64 = __attribute__((address_space(3))) double *;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)lds;
    const uint32_t stage = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + (uint32_t)kLdsTz + (uint32_t)wave * (kTailCap * 8u)));
    const uint32_t spare = lds0 + (uint32_t)kLdsSpare + (uint32_t)tid * 4u;
    uint32_t *ttab = reinterpret_cast<uint32_t *>(lds + kLdsNodes);              // [len][16]
    uint32_t *xw = ttab + (size_t)len * 16 + (size_t)wave * len * 2;             // [len][2]
    uint32_t *dims = ttab + (size_t)len * (16 + kWaves * 2);                     // [len]
    for (int j = tid; j < 64; j += kWG) {
        etab[j] = exp_tab_entry<WIDE>((uint32_t)j);
        ltab[j].rcp = rcp_f64(log_tab_centre((uint32_t)j));
        ltab[j].log = kLogTab[j];
    }
    const auto etab_at = [=](uint32_t j) { return etab[j]; };
    const auto ltab_at = [=](uint32_t j) { return ltab[j]; };

    if (init && WHAT == 0) {
        for (int q = tid; q < kSyncWords; q += kWG) a.sync[q] = 0u;
        for (int k = tid; k <= M; k += kWG) {
            const double tk = (double)k * a.T / (double)M;
            DateConst c;
            c.disc = exp(-a.r * tk);
            // Standardise x = S/K with the model's mean and sd of x given in
            // the money (ln x ~ N(m, s^2); E[x^q | x < 1] =
            // exp(q m + q^2 s^2/2) Phi(-m/s - q s)/Phi(-m/s), mirrored for
            // calls), so in-the-money abscissae are centred with unit spread
            // and the Hankel matrix stays well conditioned.  Falls back to
            // the unconditional moments when the region is negligible.
            const double m = log(a.S0 / a.K) + (a.r - 0.5 * a.sigma * a.sigma) * tk;
            const double sv = a.sigma * sqrt(tk);
            double mean = 0.0, sd = 0.0;
            if (k > 0) {
                const double z = a.is_call ? m / sv : -m / sv;     // ITM probability Phi(z)
                const double sg = a.is_call ? sv : -sv;
                const double p0 = 0.5 * erfc(-z * 0.70710678118654752);
                if (p0 > 1e-12) {
                    const double e1 = exp(m + 0.5 * sv * sv) * (0.5 * erfc(-(z + sg) * 0.70710678118654752)) / p0;
                    const double e2 = exp(2.0 * m + 2.0 * sv * sv) *
                                      (0.5 * erfc(-(z + 2.0 * sg) * 0.70710678118654752)) / p0;
                    const double var = e2 - e1 * e1;
                    if (var > 1e-12 * e1 * e1) { mean = e1; sd = sqrt(var); }
                }
                if (!(sd > 0.0)) {
                    mean = a.S0 / a.K * exp(a.r * tk);
                    sd = mean * sqrt(expm1(a.sigma * a.sigma * tk));
                }
            }
            c.xa = k > 0 ? 1.0 / (a.K * sd) : 0.0;
            c.xb = k > 0 ? -mean / sd : 0.0;
            c.pad = 0.0;
            a.datec[k] = c;
        }
    }

    for (int q = tid; q < len; q += kWG) dims[q] = sched[q].md >> 16;
    __syncthreads();
    for (int e = tid; e < len * 16; e += kWG) {
        const int h = (e >> 3) & 1, idx = e & 7;
        const uint32_t *v = V + (size_t)dims[e >> 4] * 32 + 3 * h;
        const uint32_t v0 = v[0], v1 = v[1], v2 = v[2];
        ttab[e] = (idx & 1 ? v0 : 0u) ^ (idx & 2 ? v1 : 0u) ^ (idx & 4 ? v2 : 0u);
    }

    if (w0 < w1) {
        const uint64_t n0 = (uint64_t)w0 << 6;
        const uint64_t g0 = n0 ^ (n0 >> 1);
        const int c = min(__builtin_ctzll((uint64_t)w0 + 1u) + 6, 31);
        for (int q = lane; q < len; q += 64) {
            const uint32_t j = dims[q];
            const uint32_t *v = V + (size_t)j * 32;
            // the block words carry the flipped sign bit (see Moro) and a
            // shifted point's shift
            uint32_t xa = (WHAT == 1 ? 0u : 0x80000000u) ^ (MID ? shift[j] : 0u);
            for (int b = 5; b < 32; ++b)
                if ((g0 >> b) & 1u) xa ^= v[b];
            xw[2 * q] = xa;
            xw[2 * q + 1] = xa ^ v[5] ^ v[c];
        }
    }
    __syncthreads();

    const int lo = lane < 63 ? lane + 1 : 0;
    const int gl = lo ^ (lo >> 1);
    const uint32_t *tL = ttab + (gl & 7), *tH = ttab + 8 + (gl >> 3);
    const uint32_t *tX = xw + (lane == 63 ? 1 : 0);

    // The inverse normal, the bridge and the exponent run in binary64 for
    // both storage types, so binary32 storage holds each path value rounded
    // once from its binary64 value (the correctly rounded value except where
    // that lies within a few binary64 ulps of a rounding boundary).  The
    // exercise decisions downstream react to path-value errors of one
    // binary32 ulp on some options (a binary32 inverse normal moved prices by
    // up to 7e-2).  The bridge runs
    // on the log-price X(t_m) = log S0 + mu m + vol W(m) (the schedule's
    // weights sum to 1, so interpolation carries the constant and the drift),
    // and S = exp(X): no per-date drift, volatility or S0 products.
    const double vol = a.vol;
    // Padding paths (past N) hold K rounded in the storage precision away
    // from the money, so h(S) <= 0 in binary64 and the sweep never counts
    // them in the money.
    T Kp = (T)a.K;
    if constexpr (sizeof(T) == 4) {
        if (!a.is_call && (double)Kp < a.K) Kp = nextafterf(Kp, INFINITY);
        if (a.is_call && (double)Kp > a.K) Kp = nextafterf(Kp, -INFINITY);
    }

    Window X = 0.0;
    X[0] = log(a.S0);                                   // X(t_0)
    X[kAnchorSlot] = X[0] + a.mu * (double)M;           // read by the root node only

    for (int64_t w = w0; w < w1; ++w) {
        const int64_t i = (w << 6) + lane;
        const bool valid = i < a.N;
        if (WHAT == 0 && (w << 6) >= a.N) {
            // padding block: out of the money on every date
            for (int s = 0; s < len; ++s) ((T *)a.S)[(size_t)((sched[s].md & 0xFFFFu) - 1u) * a.ld + i] = Kp;
            continue;
        }
        if constexpr (WHAT == 0) {
            // The inverse normal's two branches evaluated apart (the tail's
            // two logarithms dominate).  Every lane evaluates the (cheap)
            // central branch of a chunk's nodes up front (independent of one
            // another and of the bridge); the points in the tails are packed
            // into this wave's LDS staging (ballot and lane rank), their tail
            // values evaluated together, one point per lane, and read back by
            // their owners.  A whole chunk runs without branches or masked
            // regions (a point outside the tails writes to a spare word), so
            // the nodes' LDS reads are in flight together and their chains
            // interleave: with a branch per node every node waited for its
            // own node fields and table words in turn.
            char *const blk = (char *)a.S + (size_t)(w << 6) * sizeof(T);
            const uint64_t ldb = (uint64_t)a.ld * sizeof(T);
            const uint32_t lane_b = (uint32_t)lane * (uint32_t)sizeof(T);
            const auto chunk = [&](int s0, auto whole) {
                constexpr bool FULL = decltype(whole)::value;
                const auto has = [&](int q) { return FULL || s0 + q < len; };
                const uint32_t *pL = tL + s0 * 16, *pH = tH + s0 * 16, *pX = tX + s0 * 2;
                uint32_t x[kTailChunk];
                uint32_t slot[kTailChunk];   // LDS addresses
                double zc[kTailChunk];
                bool tl[kTailChunk];
                uint32_t ntail = 0;   // wave-uniform
#pragma unroll
                for (int q = 0; q < kTailChunk; ++q) x[q] = has(q) ? pX[2 * q] ^ pL[16 * q] ^ pH[16 * q] : 0u;
#pragma unroll
                for (int q = 0; q < kTailChunk; ++q) {
                    const double d = Moro<MID>::centered(x[q]);
                    zc[q] = Moro<MID>::central(d);
                    tl[q] = Moro<MID>::tail(d);
                    const uint64_t m = __builtin_amdgcn_ballot_w64(tl[q]);
                    // the lane's rank among the tails, as an address: the count
                    // starts at the staging's first slot
                    slot[q] = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, stage / 8u + ntail)) * 8u;
                    *(LdsU32)(tl[q] ? slot[q] : spare) = x[q];
                    ntail += (uint32_t)__builtin_popcountll(m);
                }
                wave_lds_fence();
                for (uint32_t t0 = 0; t0 < ntail; t0 += 64) {
                    // lanes past the last point evaluate what the staging
                    // holds (kept out of every result)
                    const uint32_t t = stage + (t0 + (uint32_t)lane) * 8u;
                    *(LdsF64)t = Moro<MID>::tail_value(*(LdsU32)t, ltab_at);
                }
                wave_lds_fence();
                // the nodes by scalar loads, all in flight together (loaded before
                // the first part, they take the scalar registers that its
                // constants need)
                uint32_t nmd[kTailChunk], nsl[kTailChunk];
                double nwl[kTailChunk], nwr[kTailChunk], nsd[kTailChunk];
#pragma unroll
                for (int q = 0; q < kTailChunk; ++q) {
                    GenNodeC *nd = (GenNodeC *)(sched + (has(q) ? s0 + q : s0));
                    nmd[q] = nd->md; nsl[q] = nd->slots; nwl[q] = nd->wl; nwr[q] = nd->wr; nsd[q] = nd->sd;
                }
                uint32_t off = lane_b;
                asm volatile("" : "+v"(off));   // (widened outside the loop it would be a 64-bit add per store)
                double zt[kTailChunk];
#pragma unroll
                for (int q = 0; q < kTailChunk; ++q) zt[q] = *(LdsF64)slot[q];
#pragma unroll
                for (int q = 0; q < kTailChunk; ++q) {
                    asm volatile("" : "+v"(zt[q]));   // (read by every lane: no masked regions)
                    zc[q] = vol * (tl[q] ? zt[q] : zc[q]);
                }
#pragma unroll
                for (int q = 0; q < kTailChunk; ++q) {
                    if (!has(q)) break;
                    const uint32_t mq = nmd[q] & 0xFFFFu;
                    const double xv = bridge_step(X, nsl[q], nwl[q], nwr[q], nsd[q], zc[q]);
                    const T Sv = (T)exp_tab<WIDE>(xv, etab_at);
                    using RowPtr = __attribute__((address_space(1))) char *;
                    RowPtr row = (RowPtr)blk + (uint64_t)(mq - 1u) * ldb;
                    asm volatile("" : "+s"(row));   // a scalar row base and the lane's 32-bit offset
                    *(__attribute__((address_space(1))) T *)(row + off) = Sv;
                }
                // the next chunk rewrites the staging only after every lane
                // has read its values back
                wave_lds_fence();
            };
            int s0 = 0;
            for (; s0 + kTailChunk <= len; s0 += kTailChunk) chunk(s0, std::true_type{});
            if (s0 < len) chunk(s0, std::false_type{});
            // the one block that straddles N: its padding paths over what the
            // chunks stored there (a wave's stores to one address stay in order)
            if (((w + 1) << 6) > a.N && !valid)
                for (int s = 0; s < len; ++s) ((T *)a.S)[(size_t)((sched[s].md & 0xFFFFu) - 1u) * a.ld + i] = Kp;
        } else
        for (int s = 0; s < len; ++s) {
            const int j = (int)dims[s];
            const uint32_t x = tX[2 * s] ^ tL[16 * s] ^ tH[16 * s];
            if (WHAT == 1) {
                if (valid) ((uint32_t *)a.S)[(size_t)j * a.ld + i] = x;
                continue;
            }
            const double d = Moro<MID>::centered(x);
            const double z = Moro<MID>::tail(d) ? Moro<MID>::tail_value(x, ltab_at) : Moro<MID>::central(d);
            if (valid) ((double *)a.S)[(size_t)j * a.ld + i] = z;
        }
        if (w + 1 < w1) {
            const int c = min(__builtin_ctzll((uint64_t)w + 2u) + 6, 31);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int q = lane; q < len; q += 64) {
                const uint32_t *v = V + (size_t)dims[q] * 32;
                const uint32_t xb = xw[2 * q + 1];
                xw[2 * q] = xb;
                xw[2 * q + 1] = xb ^ v[5] ^ v[c];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

// Bound by vector issue at the clock that binary64 power allows (2.07 GHz
// counted, a vector instruction every 4.1 cycles of each SIMD): 36 binary64
// and 24 other vector instructions per path-step, the LDS busy for 28 %.
// Four waves per SIMD (128 registers) hide the per-lane dependency chain of
// each path through the dates.  2^24 x 252, binary32: 10.1 ms with a branch
// per node, 9.2 with branch-free chunks of six, the {1/F, log F} table and
// tails in place, 8.7 with the indexed window and the exponent added (per call
// 15.76 -> 15.22 ms; both exponential forms in one kernel, 15.5, spill).  Few
// blocks run in segments: 30011 x 365 226 us of generation when one wave
// walked all the dates, about 45 now.  Shifted points took both branches of
// every point, with divisions: 8 x 2^17 x 100 513 -> 280 us.  blockIdx.y: the
// schedule segment.
template <typename T, int WHAT, bool MID, bool WIDE>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(4)))
gen_kernel(GenArgs a, const uint32_t *__restrict__ V, const GenNode *__restrict__ sched,
           const uint32_t *__restrict__ shift)
{
    const int64_t gw = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    const int64_t w0 = gw * a.R;
    const int64_t w1 = min(w0 + (int64_t)a.R, a.nblocks);
    // the sweep's partial-sum rows start each launch at tag 0
    if (WHAT == 0 && blockIdx.y == 0)
        for (int64_t q = (int64_t)blockIdx.x * kWG + threadIdx.x; q < a.rows_n; q += (int64_t)gridDim.x * kWG)
            a.rows[q] = 0ull;
    // (the last group of a segment holds the fewest paths: it writes the date
    // constants beside them)
    gen_body<T, WHAT, MID, WIDE>(a, V, sched + (size_t)blockIdx.y * a.seg_len, a.seg_len, shift,
                           blockIdx.x == gridDim.x - 1 && blockIdx.y == 0, w0, w1);
}

hipError_t launch_generate(const GenArgs &a, int fp64, hipStream_t s)
{
    const int64_t waves = (a.nblocks + a.R - 1) / a.R;
    const int64_t grid = (waves + kWaves - 1) / kWaves;
    const dim3 g((unsigned)grid, (unsigned)a.segs), b(kWG);
    const bool mid = a.shift != nullptr, wide = wide_exponent(a.S0, a.mu, a.vol, a.M);
    const size_t lds = gen_lds_bytes(a.seg_len);
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, lds, s, a, a.V, a.sched, a.shift); };
    if (a.what == 1) {
        go(gen_kernel<float, 1, false, false>);
    } else if (a.what == 2) {
        // the normals are binary64 for both storage types
        go(gen_kernel<double, 2, false, false>);
    } else if (fp64) {
        if (wide) mid ? go(gen_kernel<double, 0, true, true>) : go(gen_kernel<double, 0, false, true>);
        else      mid ? go(gen_kernel<double, 0, true, false>) : go(gen_kernel<double, 0, false, false>);
    } else {
        if (wide) mid ? go(gen_kernel<float, 0, true, true>) : go(gen_kernel<float, 0, false, true>);
        else      mid ? go(gen_kernel<float, 0, true, false>) : go(gen_kernel<float, 0, false, false>);
    }
    return hipGetLastError();
}

// Make the runtime load the generation kernels' code on the current device
// now rather than at their first launch (a first use allocates device memory
// for the code).
hipError_t preload_generate()
{
    hipFuncAttributes fa;
    hipError_t e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(&gen_kernel<float, 0, false, false>));
    if (e == hipSuccess) e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(&gen_kernel<double, 0, false, false>));
    return e;
}

// ---------------------------------------------------------------------------
// Dispatch over (precision, basis kind, paths per thread, degree).
// ---------------------------------------------------------------------------
static const void *sweep_lookup(int fp64, int laguerre, int ppt, int degree, int kind)
{
    if (fp64) return laguerre ? sweep_table_f64_lag(ppt, degree, kind) : sweep_table_f64_mono(ppt, degree, kind);
    return laguerre ? sweep_table_f32_lag(ppt, degree, kind) : sweep_table_f32_mono(ppt, degree, kind);
}

static const void *batch_lookup(int fp64, int laguerre, int ppt, int degree)
{
    if (fp64 == kMixed) return laguerre || ppt != 64 ? nullptr : sweep_table_mixed(degree);
    return sweep_lookup(fp64, laguerre, ppt, degree, 1);
}

static int blocks_per_cu(const void *f, int wg)
{
    if (!f) return 0;
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, wg, 0) != hipSuccess) return 0;
    return nb;
}

int sweep_blocks_per_cu(int fp64, int laguerre, int wg, int ppt, int degree)
{
    if (wg != kWG && wg != 512) return 0;
    return blocks_per_cu(sweep_lookup(fp64, laguerre, ppt, degree, wg == 512 ? 2 : 0), wg);
}

int sweep_batch_blocks_per_cu(int fp64, int laguerre, int ppt, int degree)
{
    const void *f = batch_lookup(fp64 & ~kAnyPlacement, laguerre, ppt, degree);
    const int n = blocks_per_cu(f, kWG);
    if (!(fp64 & kAnyPlacement) || n <= 1) return n;
    int dev = 0, lds_cu = 0;
    hipFuncAttributes fa;
    if (hipGetDevice(&dev) != hipSuccess || hipFuncGetAttributes(&fa, f) != hipSuccess || !fa.sharedSizeBytes ||
        hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess)
        return 1;
    const int sure = (int)(((size_t)lds_cu / fa.sharedSizeBytes + 1) / 2);
    return sure < 1 ? 1 : sure < n ? sure : n;
}

// Dynamic LDS that leaves room for one workgroup of `f` per CU (more than
// half of a CU's LDS in total), so a grid of at most one group per CU is
// spread over the CUs instead of doubling up on some; 0 if unavailable.
// Computed once per (device, kernel).
static size_t one_per_cu_lds(int dev, const void *f)
{
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, size_t> cache;
    std::lock_guard<std::mutex> lk(mu);
    const auto key = std::make_pair(dev, f);
    const auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int lds_cu = 0;
    hipFuncAttributes fa;
    size_t dyn = 0;
    if (hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) == hipSuccess &&
        hipFuncGetAttributes(&fa, f) == hipSuccess) {
        const size_t want = (size_t)lds_cu / 2 + 1024;
        if (fa.sharedSizeBytes < want) {
            dyn = want - fa.sharedSizeBytes;
            if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn) != hipSuccess) dyn = 0;
        }
    }
    cache[key] = dyn;
    return dyn;
}

hipError_t launch_sweep(const SweepArgs &a, int fp64, int wg, int ppt, hipStream_t s)
{
    if (wg != kWG && wg != 512) return hipErrorInvalidValue;
    const uint32_t G = (uint32_t)a.G;
    const bool spin = row_words(a.degree) == 16 ? spins_on_rows<16>(G) : spins_on_rows<32>(G);
    const bool keep = ppt * (fp64 ? 8 : 4) <= 64;
    // slab-resident tiles come in a call form (kind 3) and a put form (kind 2),
    // register-resident ones in a form for few groups (4) and one for more (2)
    const void *f = nullptr;
    if (wg == 512 && keep && spin) f = sweep_lookup(fp64, a.laguerre, ppt, a.degree, 4);
    else if (wg == 512 && a.is_call) f = sweep_lookup(fp64, a.laguerre, ppt, a.degree, 3);
    if (!f) f = sweep_lookup(fp64, a.laguerre, ppt, a.degree, wg == 512 ? 2 : 0);
    if (!f) return hipErrorInvalidValue;
    SweepArgs args = a;
    const void *Sp = a.S;
    void *params[] = {(void *)&args, (void *)&Sp};
    int dev = 0, cus = 0;
    size_t dyn = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && a.G <= cus)
        dyn = one_per_cu_lds(dev, f);
    // a plain launch: the grid is sized to what the device holds at once, and
    // the caller orders persistent sweeps on one device (a cooperative launch
    // measured 19 us slower per call, in the kernel's own event interval)
    // few groups of a register-resident tile: all on one XCD, where its compute
    // units hold one each; more of another tile are relayed, as dealt
    const uint32_t stride = a.xcd_stride > 1 ? (uint32_t)a.xcd_stride : kXcds;   // (else a test's)
    const bool strided = G > 1 && spin && keep && dyn > 0 && (uint64_t)G * stride <= (uint64_t)cus;
    args.xcd_stride = strided ? (int)stride : !spin && !keep && G <= kFlatMaxGroups ? 1 : 0;
    const uint32_t grid = strided ? G * stride : G;
    return hipLaunchKernel(f, dim3(grid), dim3((unsigned)wg), params, (unsigned)dyn, s);
}

// ---------------------------------------------------------------------------
// Batches: many options with uneven path and date counts in two launches.
//
// Generation: each workgroup owns a block range of one option (unit table
// built on the host).  Sweep: one persistent grid; workgroups
// claim (option, tile) slots from one or several queues in a fixed order (options
// by decreasing date count, each option's tiles contiguous; see claim_tile), run that tile through
// all of the option's dates with the option's own barrier words and partial
// slots, then claim again.  An option's result depends
// only on its own tiles and the fixed reduction order, not on which group ran
// which tile, so it is the same alone and in any mix.
// ---------------------------------------------------------------------------
__device__ __forceinline__ GenArgs gen_args_of(const BatchOpt &o, const uint32_t *V)
{
    GenArgs a;
    a.S = o.S;
    a.V = V;
    a.sched = o.sched;
    a.datec = o.datec;
    a.sync = o.sync;
    a.N = o.N;
    a.ld = o.ld;
    a.nblocks = o.ld / 64;
    a.M = o.M;
    a.segs = 1; a.seg_len = o.seg_len;
    a.R = 1;
    a.what = 0;
    a.pad = 0;
    a.S0 = o.S0; a.K = o.K; a.r = o.r; a.sigma = o.sigma; a.T = o.T;
    a.mu = o.mu; a.vol = o.vol;
    a.shift = nullptr;
    a.is_call = o.is_call;
    a.rows = o.rows;
    a.rows_n = 0;   // cleared by the option's first unit
    return a;
}

template <typename T, bool MID, bool WIDE>
__global__ void __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(4)))
gen_batch_kernel(const BatchOpt *__restrict__ opts, const GenUnit *__restrict__ units,
                 const uint32_t *__restrict__ V, uint32_t *gsync)
{
    const GenUnit u = units[blockIdx.x];
    const BatchOpt o = opts[u.opt];
    if (blockIdx.x == 0 && threadIdx.x < 16) gsync[threadIdx.x] = 0u;
    const GenArgs a = gen_args_of(o, V);
    if (u.b0 == 0 && u.seg == 0)   // the option's first unit clears its partial-sum rows
        for (int64_t q = threadIdx.x; q < o.rows_n; q += kWG) o.rows[q] = 0ull;
    const int64_t per = (u.b1 - u.b0 + kWaves - 1) / kWaves;
    const int64_t w0 = u.b0 + (int64_t)(threadIdx.x >> 6) * per;
    const int64_t w1 = min(w0 + per, u.b1);
    gen_body<T, 0, MID, WIDE>(a, V, o.sched + (size_t)u.seg * o.seg_len, o.seg_len, MID ? o.shift : nullptr,
                        u.b0 == 0 && u.seg == 0, w0, w1);
}

hipError_t launch_generate_batch(const BatchOpt *opts, const GenUnit *units, int n_units,
                                 const uint32_t *V, uint32_t *gsync, int max_seg_len, int fp64,
                                 bool shifted, hipStream_t s)
{
    const size_t lds = gen_lds_bytes(max_seg_len);
    const dim3 g(n_units), b(kWG);
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, lds, s, opts, units, V, gsync); };
    // shifted: randomised QMC, every option of the batch carries its digital shift
    const bool f64 = fp64 & 1, wide = fp64 & kGenWide;
    if (f64) {
        if (wide) shifted ? go(gen_batch_kernel<double, true, true>) : go(gen_batch_kernel<double, false, true>);
        else      shifted ? go(gen_batch_kernel<double, true, false>) : go(gen_batch_kernel<double, false, false>);
    } else {
        if (wide) shifted ? go(gen_batch_kernel<float, true, true>) : go(gen_batch_kernel<float, false, true>);
        else      shifted ? go(gen_batch_kernel<float, true, false>) : go(gen_batch_kernel<float, false, false>);
    }
    return hipGetLastError();
}

hipError_t launch_sweep_batch(const BatchOpt *opts, const int32_t *tile_opt, const BatchGlobal &g,
                              int grid, int fp64, int ppt, int degree, bool spread, hipStream_t s)
{
    const void *f = batch_lookup(fp64, g.laguerre, ppt, degree);
    if (!f) return hipErrorInvalidValue;
    const BatchOpt *o = opts;
    const int32_t *to = tile_opt;
    BatchGlobal gg = g;
    void *params[] = {(void *)&o, (void *)&to, (void *)&gg};
    int dev = 0;
    size_t dyn = 0;
    if (spread && hipGetDevice(&dev) == hipSuccess) dyn = one_per_cu_lds(dev, f);
    // grid sized by the caller so that every in-flight persistent grid is
    // resident together; the bounded waits end the kernel otherwise
    return hipLaunchKernel(f, dim3((unsigned)grid), dim3(kWG), params, (unsigned)dyn, s);
}

// ---------------------------------------------------------------------------
// The paper's own estimator (Section V, eqs. (10)-(11)): on the grid
// t_i = i dt, dt = T/(m+1), i = 1..m, the value at t_m is the larger of the
// exercise value and the Black–Scholes value over the last interval dt
// (eqs. (1)-(5)); going back, c_i = max(h(S_i), exp(-r dt) c_{i+1}); the price
// is exp(-r dt) times the path mean of c_1 (eq. (6)).  Every path is
// independent: no device-wide wait.  The paths come from
// the generation kernel run with m dates and horizon m dt.
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ T cnd(T x);
template <> __device__ __forceinline__ float cnd<float>(float x) { return 0.5f * erfcf(-x * 0.70710678118654752f); }
template <> __device__ __forceinline__ double cnd<double>(double x) { return 0.5 * erfc(-x * 0.70710678118654752); }

template <typename T>
__device__ __forceinline__ T bs_value(T S, T K, T r, T sig, T tau, bool call)
{
    const T sq = sig * sqrt(tau);
    const T d1 = (log(S / K) + (r + T(0.5) * sig * sig) * tau) / sq;
    const T d2 = d1 - sq;
    const T dk = K * exp(-r * tau);
    return call ? S * cnd<T>(d1) - dk * cnd<T>(d2) : dk * cnd<T>(-d2) - S * cnd<T>(-d1);
}

// A date of a thread's paths is one 16-byte load (4 binary32 or 2 binary64
// consecutive paths), kPaperAhead dates requested before the first is used:
// a path's steps depend only on its running maximum, so the kernel is bound
// by the loads in flight.  With one path a thread and a load a step, 2^20
// paths x 100 dates took 238 us (1.8 TB/s) in binary32.
constexpr int kPaperAhead = 8;

template <typename T>
__global__ void __launch_bounds__(kWG) paper_kernel(PaperArgs a, const T *__restrict__ S)
{
    constexpr int VW = 16 / sizeof(T);
    struct alignas(16) V { T v[VW]; };
    __shared__ double s_red[kWaves][32];
    __shared__ double s_red8[8][32];
    __shared__ double s_tot[32];
    __shared__ int s_flag[2];
    const T K = (T)a.K, r = (T)a.r, sig = (T)a.sigma, dt = (T)a.dt;
    const T disc = (T)exp(-a.r * a.dt);
    const bool call = a.is_call != 0;
    // sums about c = max(h(S0), 0): the variance below cancels only to the
    // order of (mean - c)^2 / variance
    const double h0 = call ? a.S0 - a.K : a.K - a.S0;
    const double csh = h0 > 0.0 ? h0 : 0.0;
    double acc[2] = {0.0, 0.0};
    // rows are padded to whole vectors (ld is a multiple of kLdAlign), so a
    // vector that straddles N reads padding, which is not counted
    for (int64_t i = ((int64_t)blockIdx.x * kWG + threadIdx.x) * VW; i < a.N; i += (int64_t)gridDim.x * kWG * VW) {
        T v[VW];
        const auto step = [&](const V &s, auto last) {
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                T h = call ? s.v[e] - K : K - s.v[e];
                h = h > T(0) ? h : T(0);
                T cont;
                if constexpr (decltype(last)::value) cont = bs_value<T>(s.v[e], K, r, sig, dt, call);
                else cont = disc * v[e];
                v[e] = h > cont ? h : cont;
            }
        };
        const T *col = S + i;
        const auto load = [&](int k) { return *reinterpret_cast<const V *>(col + (size_t)(k - 1) * a.ld); };
        V buf[kPaperAhead];
        int k = a.m - 1;   // dates m-1 .. 1 after the last point's
#pragma unroll
        for (int q = 0; q < kPaperAhead; ++q) buf[q] = load(k - q >= 1 ? k - q : 1);
        step(load(a.m), std::true_type{});
        for (; k >= kPaperAhead; k -= kPaperAhead) {
#pragma unroll
            for (int q = 0; q < kPaperAhead; ++q) {
                const V s = buf[q];
                const int kn = k - q - kPaperAhead;
                buf[q] = load(kn >= 1 ? kn : 1);
                step(s, std::false_type{});
            }
        }
#pragma unroll
        for (int q = 0; q < kPaperAhead - 1; ++q)
            if (k - q >= 1) step(buf[q], std::false_type{});
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            const double c = i + e < a.N ? (double)disc * (double)v[e] - csh : 0.0;
            acc[0] += c;
            acc[1] += c * c;
        }
    }
    const double at = group_sum<2>(acc, s_red, threadIdx.x);
    acc[0] = readlane_f64(at, 0);
    acc[1] = readlane_f64(at, 1);
    if (threadIdx.x == 0) {
        double *dst = a.part + (size_t)blockIdx.x * kPartStride;
        dst[0] = acc[0];
        dst[1] = acc[1];
        const uint32_t old = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        s_flag[0] = (old + 1u == gridDim.x) ? 1 : 0;
    }
    __syncthreads();
    if (!s_flag[0]) return;
    reduce_partials<2>(a.part, gridDim.x, s_tot, s_red8);
    if (threadIdx.x == 0) {
        const double n = (double)a.N;
        const double mean = csh + s_tot[0] / n;
        double var = a.N > 1 ? (s_tot[1] - s_tot[0] * (s_tot[0] / n)) / (n - 1.0) : 0.0;
        if (var < 0.0) var = 0.0;
        const double res[6] = {mean, sqrt(var / n), mean, 0.0, 0.0, 0.0};
        for (int q = 0; q < 6; ++q) a.result[q] = res[q];
        put_host_result(a.host_out, res);
    }
}

hipError_t launch_paper(const PaperArgs &a, int fp64, hipStream_t s)
{
    const int64_t per = (int64_t)kWG * (fp64 ? 2 : 4);   // paths a group takes per pass
    int64_t g = (a.N + per - 1) / per;
    if (g > kMaxGroups) g = kMaxGroups;
    if (fp64) hipLaunchKernelGGL((paper_kernel<double>), dim3((unsigned)g), dim3(kWG), 0, s, a, (const double *)a.S);
    else      hipLaunchKernelGGL((paper_kernel<float>), dim3((unsigned)g), dim3(kWG), 0, s, a, (const float *)a.S);
    return hipGetLastError();
}

}  // namespace amq
