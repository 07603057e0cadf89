// P2P: the near-field sum of Sec. 2.1, eq. (potentials-near) with the screened Stokeslet
// of eq. (g-near),
//   u^N_i = sum_{j,p : 0 < |r| < r_c} G^N(r) f_j,   r = x_i - x_j + p,
//   G^N(r) f = C(r) (f/|r| + r (r.f)/|r|^3) - (4 xi/sqrt(pi)) e^{-xi^2 |r|^2} f,
//   C(r) = erfc(xi |r|) + (2 xi |r|/sqrt(pi)) e^{-xi^2 |r|^2}.
// With x = xi |r| and E = e^{-x^2}, C = E (erfcx(x) + 2x/sqrt(pi)), so one exponential, one
// reciprocal square root and one short polynomial (screening.h) give both coefficients
//   a1 = C/|r| - (4 xi/sqrt(pi)) E   (of f)   and   a2 = C/|r|^3   (of r (r.f)).
//
// Work decomposition (MI355X).  Particles are sorted by tile (B^3 grid cells, edge about
// r_c/2.5).  One wavefront takes 64 consecutive targets of one tile, one target per lane,
// and walks the (2S+1)^3 neighbour tiles in unwrapped tile coordinates (each periodic image
// of a source is met at most once, also when a dimension has fewer than 2S+1 tiles),
// skipping tiles farther than r_c from the bounding box of its targets.  Lockstep over
// sources would run the expensive formula for every source that ANY lane accepts (about
// twice the useful pairs); instead:
//   1. the wave loads 64 candidate sources at a time (one per lane), keeps those within
//      r_c of the targets' bounding box and appends them, shifted into the targets'
//      periodic frame, to an LDS ring;
//   2. per 32 ring sources the accepted sources of each lane's target (r^2 < r_c^2, r^2 > 0) are
//      found as a mask;
//   3. the batch's pairs are evaluated one pair per lane, every lane busy (the balanced drain below).
#include "internal.h"
#include <algorithm>
#include <type_traits>
#include "screening.h"

namespace ewald {

namespace {

// Accuracy levels of the FP64 pair formula (template argument Lv), chosen from the plan's tol so
// that the formula's own error stays at least 30 times below it:
//   0 (tol < 1e-10): degree-16 screening polynomial (|dC| < 5e-15), library exponential, two
//     Newton steps on the hardware reciprocal, third-order rsqrt correction;
//   1 (1e-10 <= tol < 1e-8): erfcx(x) + 2x/sqrt(pi) as a polynomial in x fitted under the weight
//     e^{-x^2} (degree 19, |dC| < 7.2e-13), e^{-y} = 2^z (z = -y log2 e) as 2^n times a degree-8
//     Chebyshev polynomial of 2^s, z = n + s, n = rint(z) (relative error 1.1e-12; no range checks:
//     -61 < z <= 0 on the P2P range), one Newton step on rsqrt;
//   2 (tol >= 1e-8): degree 16 (|dC| < 4.0e-11) and a degree-7 polynomial of 2^s (5.6e-11), else as
//     level 1.
// The weighted polynomial needs no reciprocal: 16 instructions, as with the degree-10 polynomial in
// (x - 3)/(x + 3) (stresslet pairs take that form and its degree-12 sibling), of which one is
// quarter rate.  With the exponential, |dC| at levels 1 and 2: at most 1.6e-12 and 8.0e-11 (4.3e-12 and
// 2.9e-10 for those forms), for x > 1 9.5e-13 and 5.4e-11 (1.1e-12 and 7.4e-11), and
// (integral of dC^2 dx)^1/2, which enters a sum over uniform pairs, 1.2e-12 and 6.7e-11 (2.3e-12 and 1.3e-10).
// The minimax error is flat, so that beyond x = 2, where the others fall with C itself, it is the larger.
// All polynomials are stored divided by their leading coefficients (screening.h), so that Horner
// starts with an addition (an FMA cannot take two scalar-register coefficients).  The FP64 pair formula
// therefore returns its coefficients divided by post; the kernels multiply each target's and source's sum by post once, at the end.
// Levels 1 and 2 work (without stresslet sources) on positions scaled by a power of two p near
// kappa = xi sqrt(log2 e), which makes r the variable of polynomials whose coefficients the host multiplies by
// powers of kappa / p (a multiplication per pair less, whatever the box's size).  A power of two, so that the
// scaled positions and their differences are exact: scaling by kappa itself rounds every position once more,
// and the distance of two points 1e-8 apart was then off by 6.6e-10 at the median (7e-13 so, the formula's
// own error).  Against that form, one FMA a pair and the candidates' test for NaN: c2 P2P 17.47 -> 17.6 ms.
constexpr double kLog2e = 1.4426950408889634074;

struct PairArgs {
    double xi, xi2, rc2;
    double four_xi_over_sqrtpi;
    // FP64 formula of the launched level: z = zc r^2 (zc = -xi^2 log2 e); monic screening (ms,
    // x coefficient g = (2/sqrt(pi))/lead_s) and exponential (me) polynomials; a1 / post =
    // C'/r - h e' with h = (4 xi/sqrt(pi))/lead_s
    double zc, g, h, post, lead_s, lead_e;
    double lead_st;  // leading coefficient of ms (stresslet pairs)
    // scaled form (see above): p, the cutoff (p r_c)^2, h / p, zc / p^2; the sums' factor is post p
    double scale, rc2s, hs, zs;
    // polynomials passed by value, so that the coefficients sit in scalar registers (an FMA then
    // takes them as an operand, no per-pair register copies); mw: the weighted screening polynomial of
    // levels 1 and 2 in the scaled r, c32: the FP32 formula's
    double ms[kScreenDeg64];
    double mw[kScreenDegV1];
    double me[kExpDeg1];
    float c32[kScreenDeg32 + 1];
    float zc32;  // FP32 formula: -xi^2 log2 e
    double six_xi_over_sqrtpi, four_xi3_over_sqrtpi;  // stresslet screening
};

constexpr double kTwoOverSqrtPi = 1.1283791670955125739;

__device__ inline double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    return v;
}

__device__ inline double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}

// A value every lane of the wave already holds, made provably uniform for the compiler
// (so that addresses derived from it use scalar loads).
__device__ inline int uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline double uniform_d(double v)
{
    const unsigned long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(b & 0xffffffffull));
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// minimum over the wave of v in [0, 63], by six ballots (no cross-lane data movement: the
// shuffle form of this reduction put six dependent LDS round trips into every batch)
__device__ inline int wave_min_small(int v)
{
    int lo = 0;
#pragma unroll
    for (int b = 32; b >= 1; b >>= 1)
        if (__builtin_amdgcn_ballot_w64(v < lo + b) == 0ull) lo += b;
    return lo;
}

// sum of v over the wave, for every lane
__device__ inline int wave_sum_i(int v) { return __builtin_amdgcn_readlane(wave_scan(v), kWave - 1); }

// position of the k-th (from 0) set bit of m, for k < popcount(m): five halving steps
__device__ inline int select_bit(unsigned m, int k)
{
    int pos = 0;
#pragma unroll
    for (int s = 16; s >= 1; s >>= 1) {
        const int low = __popc(m & ((1u << s) - 1u));
        const bool up = low <= k;
        k = up ? k - low : k;
        m = up ? m >> s : m;
        pos = up ? pos + s : pos;
    }
    return pos;
}

// v | (v of lane l ^ 16) | (v of lane l ^ 32) | (v of lane l ^ 48), by the lane-swap instructions
// (VALU; a shuffle would take the LDS pipeline, which bounds the P2P kernels)
__device__ inline unsigned or_rows4(unsigned v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] | a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b[0] | b[1];
}

// number of set bits of m in the lanes below this one
__device__ inline int lanes_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// (erfcx(x) + 2x/sqrt(pi)) / lead_st for 0 <= x <= kScreenXmax: the monic polynomial of screening.h
// in t = (x - K)/(x + K) = 1 - 2K/(x + K), plus g x
template <int Lv>
__device__ inline double screen_q64(double x, const PairArgs& a)
{
    const double d = x + kScreenK;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    if (Lv == 0) r = fma(fma(-d, r, 1.0), r, r);
    const double t = fma(-2.0 * kScreenK, r, 1.0);
    constexpr int deg = Lv == 0 ? kScreenDeg64 : Lv == 1 ? kScreenDeg64s : kScreenDeg64f;
    const double* m = a.ms;
    double q = t + m[deg - 1];
#pragma unroll
    for (int k = deg - 2; k >= 0; --k) q = fma(q, t, m[k]);
    return fma(a.g, x, q);
}

// 2^z / lead_e for z = c r2, -61 < z <= 0: z = n + s, n = rint(z), |s| <= 1/2, 2^s from the monic
// polynomial of screening.h.  The factor c costs no multiplication: one FMA adds c r2 to 1.5 x 2^52, which rounds
// it to an integer in the sum's low bits (n, for ldexp), another subtracts it from c r2 unrounded.
template <int Lv>
__device__ inline double exp2_lead(double r2, double c, const PairArgs& a)
{
    constexpr double kRound = 6755399441055744.0;
    const double t = fma(c, r2, kRound);
    const double s = fma(c, r2, kRound - t);
    constexpr int deg = Lv == 1 ? kExpDeg1 : kExpDeg2;
    const double* m = a.me;
    double p = s + m[deg - 1];
#pragma unroll
    for (int k = deg - 2; k >= 0; --k) p = fma(p, s, m[k]);
    return ldexp(p, __double2loint(t));
}

// 1/sqrt(r2) for finite r2 > 0: hardware estimate y (error bound 2^29 ulp, ~2^-23
// relative), then with e = 1 - r2 y^2 one third-order correction y (1 + e/2 + 3e^2/8) (full
// FP64), or for levels 1 and 2 one Newton step y (1 + e/2) (relative error ~ 3e^2/8, below
// 1e-13).  No special values.
template <int Lv>
__device__ inline double rsqrt_pos(double r2)
{
    const double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-r2 * y, y, 1.0);
    if (Lv > 0) return fma(y * e, 0.5, y);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// (erfcx(x) + 2x/sqrt(pi)) / lead_s at the scaled r: the weighted polynomial of screening.h
template <int Lv>
__device__ inline double screen_w64(double r, const PairArgs& a)
{
    constexpr int deg = Lv == 1 ? kScreenDegV1 : kScreenDegV2;
    double q = r + a.mw[deg - 1];
#pragma unroll
    for (int k = deg - 2; k >= 0; --k) q = fma(q, r, a.mw[k]);
    return q;
}

// Coefficients of G^N(r) f = a1 f + b (r.f) r for 0 < r^2 < r_c^2 (FP64), divided by post:
// a1 = C/r - (4 xi/sqrt(pi)) e, b = C/r^3, with e = e^{-xi^2 r^2} = lead_e e' and C = e Q,
// Q = lead_s Q'.  Levels 1 and 2: r2 is (p r)^2, and a1, b are for the scaled r.
template <int Lv>
__device__ inline void coef64(double r2, const PairArgs& a, double& a1, double& b)
{
    const double rinv = rsqrt_pos<Lv>(r2);
    double e, q;
    if constexpr (Lv == 0) {
        e = exp(-a.xi2 * r2);
        q = screen_q64<Lv>(a.xi * r2 * rinv, a);
    } else {
        e = exp2_lead<Lv>(r2, a.zs, a);
        q = screen_w64<Lv>(r2 * rinv, a);
    }
    const double Cr = e * q * rinv;
    a1 = fma(Lv > 0 ? -a.hs : -a.h, e, Cr);
    b = Cr * (rinv * rinv);
}

// FP32 versions (FP32 bulk mode): hardware reciprocal, rsqrt and exp2 (1 ulp each, used
// as they come: a refinement step would only chase FP32's own rounding), degree-11
// polynomial.  e = 2^z with z = -xi^2 r^2 log2(e) formed in FP32: z reaches -61, where its
// rounding moves 2^z by up to 3e-6 relative, but the absolute error, 2^z |z| ln2 x 2^-24, stays
// below 8e-8 over the whole range (as for FP32 rounding of e itself); e multiplies the field
// terms, so this is the error that counts.
__device__ inline float screen_q32(float x, const PairArgs& a)
{
    const float d = x + (float)kScreenK;
    const float r = __builtin_amdgcn_rcpf(d);  // 1 ulp: no refinement needed in FP32
    const float u = fmaf((x - (float)kScreenK) * r, (float)kScreenA, (float)kScreenB);
    float q = a.c32[kScreenDeg32];
#pragma unroll
    for (int k = kScreenDeg32 - 1; k >= 0; --k) q = fmaf(q, u, a.c32[k]);
    return fmaf((float)kTwoOverSqrtPi, x, q);
}

__device__ inline void coef32(double r2d, const PairArgs& a, float& a1, float& b)
{
    const float r2 = (float)r2d;
    const float rinv = __builtin_amdgcn_rsqf(r2);  // 1 ulp: no refinement needed in FP32
    const float x = (float)a.xi * r2 * rinv;
    const float e = __builtin_amdgcn_exp2f(a.zc32 * r2);
    const float Cr = e * screen_q32(x, a) * rinv;
    a1 = fmaf(-(float)a.four_xi_over_sqrtpi, e, Cr);
    b = Cr * (rinv * rinv);
}

// Pair coefficients in the formula precision TF (double: FP64 path at accuracy level Lv; float: FP32
// bulk, Lv unused).
template <typename TF, int Lv>
struct Coef;
// post: the factor that the sums of eval's contributions take at the end
template <int Lv>
struct Coef<double, Lv> {
    __device__ static inline void eval(double r2, const PairArgs& a, double& a1, double& b)
    {
        coef64<Lv>(r2, a, a1, b);
    }
    __device__ static inline double post(const PairArgs& a) { return Lv > 0 ? a.post * a.scale : a.post; }
};
template <int Lv>
struct Coef<float, Lv> {
    __device__ static inline void eval(double r2, const PairArgs& a, float& a1, float& b) { coef32(r2, a, a1, b); }
    __device__ static inline double post(const PairArgs&) { return 1.0; }
};

// Stresslet pair (combined single and double layer sources, Sec. 2.3): with the screened
// remainder of T(r) = -6 r r r / |r|^5,
//   T^N_abc(r) S_bc = alpha r_a (r.S r) + beta (2 (S r)_a + tr(S) r_a)   (S symmetric),
//   alpha = -2 |r|^-3 (3 erfc(xi |r|) |r|^-2 + e^{-xi^2 r^2} (6 xi/(sqrt(pi) |r|) + 4 xi^3 |r|/sqrt(pi))),
//   beta = 4 xi^3 e^{-xi^2 r^2} / sqrt(pi).
// Both follow from the same exponential and screening polynomial as G^N:
// erfc(x) = C - (2x/sqrt(pi)) e^{-x^2}.
template <int Lv>
__device__ inline void coef64_st(double r2, const PairArgs& a, double& a1, double& b, double& al, double& be)
{
    const double rinv = rsqrt(r2);
    const double r = r2 * rinv;
    const double x = a.xi * r;
    const double e = Lv > 0 ? a.lead_e * exp2_lead<Lv>(r2, a.zc, a) : exp(-a.xi2 * r2);
    const double C = e * (a.lead_st * screen_q64<Lv>(x, a));
    const double rinv2 = rinv * rinv, rinv3 = rinv2 * rinv;
    a1 = fma(C, rinv, -a.four_xi_over_sqrtpi * e);
    b = C * rinv3;
    const double erfc_x = fma(-kTwoOverSqrtPi * x, e, C);
    al = -2.0 * rinv3 * fma(3.0 * erfc_x, rinv2, e * fma(a.six_xi_over_sqrtpi, rinv, a.four_xi3_over_sqrtpi * r));
    be = a.four_xi3_over_sqrtpi * e;
}

__device__ inline void coef32_st(double r2d, const PairArgs& a, float& a1, float& b, float& al, float& be)
{
    const float r2 = (float)r2d;
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float r = r2 * rinv;
    const float x = (float)a.xi * r;
    const float e = __builtin_amdgcn_exp2f(a.zc32 * r2);
    const float C = e * screen_q32(x, a);
    const float rinv2 = rinv * rinv, rinv3 = rinv2 * rinv;
    a1 = fmaf(C, rinv, -(float)a.four_xi_over_sqrtpi * e);
    b = C * rinv3;
    const float erfc_x = fmaf(-(float)kTwoOverSqrtPi * x, e, C);
    al = -2.0f * rinv3 *
         fmaf(3.0f * erfc_x, rinv2, e * fmaf((float)a.six_xi_over_sqrtpi, rinv, (float)a.four_xi3_over_sqrtpi * r));
    be = (float)a.four_xi3_over_sqrtpi * e;
}

template <typename TF, int Lv>
struct CoefSt;
template <int Lv>
struct CoefSt<double, Lv> {
    __device__ static inline void eval(double r2, const PairArgs& a, double& a1, double& b, double& al, double& be)
    {
        coef64_st<Lv>(r2, a, a1, b, al, be);
    }
};
template <int Lv>
struct CoefSt<float, Lv> {
    __device__ static inline void eval(double r2, const PairArgs& a, float& a1, float& b, float& al, float& be)
    {
        coef32_st(r2, a, a1, b, al, be);
    }
};

// c += alpha r (r.S r) + beta (2 S r + tr(S) r), S = (s0..s5) = (xx, yy, zz, xy, xz, yz)
template <typename TF>
__device__ inline void apply_st(TF al, TF be, TF rx, TF ry, TF rz, const TF* s, TF& c0, TF& c1, TF& c2)
{
    const TF t0 = s[0] * rx + s[3] * ry + s[4] * rz;
    const TF t1 = s[3] * rx + s[1] * ry + s[5] * rz;
    const TF t2 = s[4] * rx + s[5] * ry + s[2] * rz;
    const TF rsr = rx * t0 + ry * t1 + rz * t2;
    const TF g = al * rsr + be * (s[0] + s[1] + s[2]);
    const TF be2 = be + be;
    c0 += g * rx + be2 * t0;
    c1 += g * ry + be2 * t1;
    c2 += g * rz + be2 * t2;
}

// c = a1 f + b (r.f) r
template <typename TF>
__device__ inline void apply(TF a1, TF b, TF rx, TF ry, TF rz, TF f0, TF f1, TF f2, TF& c0, TF& c1, TF& c2)
{
    const TF rf = (rx * f0 + ry * f1 + rz * f2) * b;
    c0 = a1 * f0 + rf * rx;
    c1 = a1 * f1 + rf * ry;
    c2 = a1 * f2 + rf * rz;
}

constexpr int kRing = 128;   // LDS ring of filtered candidate sources
constexpr int kTest = 32;    // sources tested per round

// The number of ordered pairs within the cutoff that the near-field sum runs over, for measurement: every
// wave counts its targets' and adds the count to *pair_count (one integer atomic per wave).
__global__ __launch_bounds__(64) void k_count_pairs(const Rec64* __restrict__ rec, const int* __restrict__ start,
                                                    const int* __restrict__ chunk_off, Geometry g, PairArgs a,
                                                    unsigned long long* __restrict__ pair_count)
{
    __shared__ double ring[3][kRing];

    const int wave = uniform_i((int)blockIdx.x);
    const int lane = threadIdx.x;
    const int total = chunk_off[g.ntiles * g.nsys];  // chunks of all systems
    if (wave >= total) return;

    // tile of this wave: largest t with chunk_off[t] <= wave
    int lo = 0, hi = g.ntiles * g.nsys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (chunk_off[mid] <= wave) lo = mid; else hi = mid;
    }
    const int t = lo;
    const int per = 1 << (3 * g.log2B);
    const int t_end = start[(t + 1) * per];
    const int first = start[t * per] + (wave - chunk_off[t]) * kWave;
    const int i = first + lane;
    const bool active = i < t_end;
    const Rec64 me = rec[active ? i : first];

    // tile t of system sys (the systems of a batch have consecutive tile ranges)
    const int sys = t / g.ntiles, tl = t - sys * g.ntiles, tbase = sys * g.ntiles;
    const int tc[3] = {tl / (g.NT[1] * g.NT[2]), (tl / g.NT[2]) % g.NT[1], tl % g.NT[2]};
    double w[3], blo[3], bhi[3], tx[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        w[d] = g.B * g.h[d];
        blo[d] = uniform_d(wave_min(me.x[d]));
        bhi[d] = uniform_d(wave_max(me.x[d]));
        tx[d] = active ? me.x[d] : 1e30;  // an inactive lane accepts no pair
    }

    int rhead = 0, rcount = 0;
    unsigned long long counted = 0;

    // test the targets against ring sources [rhead, rhead + cnt)
    auto process = [&](int cnt) {
        int qn = 0;
        for (int j = 0; j < cnt; ++j) {
            const int slot = (rhead + j) & (kRing - 1);
            const double rx = tx[0] - ld1(ring[0][slot]), ry = tx[1] - ld1(ring[1][slot]), rz = tx[2] - ld1(ring[2][slot]);
            const double r2 = rx * rx + ry * ry + rz * rz;
            const bool pass = (r2 < a.rc2) & (r2 > 0.0);
            qn += __popcll(__ballot(pass));
        }
        counted += (unsigned long long)qn;
        wave_lds_sync();
    };

    for (int dx = -g.S[0]; dx <= g.S[0]; ++dx) {
        const int ux = tc[0] + dx;
        const int fx = floor_div(ux, g.NT[0]);
        const int wx = ux - fx * g.NT[0];
        const double shx = fx * g.L[0];
        const double gx = fmax(0.0, fmax(ux * w[0] - bhi[0], blo[0] - (ux + 1) * w[0]));
        for (int dy = -g.S[1]; dy <= g.S[1]; ++dy) {
            const int uy = tc[1] + dy;
            const int fy = floor_div(uy, g.NT[1]);
            const int wy = uy - fy * g.NT[1];
            const double shy = fy * g.L[1];
            const double gy = fmax(0.0, fmax(uy * w[1] - bhi[1], blo[1] - (uy + 1) * w[1]));
            if (gx * gx + gy * gy >= a.rc2) continue;
            for (int dz = -g.S[2]; dz <= g.S[2]; ++dz) {
                const int uz = tc[2] + dz;
                const int fz = floor_div(uz, g.NT[2]);
                const int wz = uz - fz * g.NT[2];
                const double shz = fz * g.L[2];
                const double gz = fmax(0.0, fmax(uz * w[2] - bhi[2], blo[2] - (uz + 1) * w[2]));
                if (gx * gx + gy * gy + gz * gz >= a.rc2) continue;
                const int nt = tbase + (wx * g.NT[1] + wy) * g.NT[2] + wz;
                const int sa = start[nt * per], sb = start[(nt + 1) * per];
                for (int base = sa; base < sb; base += kWave) {
                    const int s = base + lane;
                    bool keep = false;
                    double sx = 0, sy = 0, sz = 0;
                    if (s < sb) {
                        const Rec64& q = rec[s];
                        sx = q.x[0] + shx;
                        sy = q.x[1] + shy;
                        sz = q.x[2] + shz;
                        const double ex = fmax(0.0, fmax(blo[0] - sx, sx - bhi[0]));
                        const double ey = fmax(0.0, fmax(blo[1] - sy, sy - bhi[1]));
                        const double ez = fmax(0.0, fmax(blo[2] - sz, sz - bhi[2]));
                        keep = ex * ex + ey * ey + ez * ez < a.rc2;
                    }
                    const unsigned long long b = __ballot(keep);
                    if (keep) {
                        const int slot = (rhead + rcount + lanes_below(b)) & (kRing - 1);
                        ring[0][slot] = sx;
                        ring[1][slot] = sy;
                        ring[2][slot] = sz;
                    }
                    rcount += __popcll(b);
                    wave_lds_sync();
                    while (rcount >= kTest) {
                        process(kTest);
                        rhead = (rhead + kTest) & (kRing - 1);
                        rcount -= kTest;
                    }
                }
            }
        }
    }
    while (rcount > 0) {
        const int c = rcount < kTest ? rcount : kTest;
        process(c);
        rhead = (rhead + c) & (kRing - 1);
        rcount -= c;
    }
    if (lane == 0 && counted > 0) atomicAdd(pair_count, counted);
}

// ---------------------------------------------------------------- symmetric form
// G^N is even in r, so one evaluation of a pair (i, j) gives both G^N(r) f_j (to u_i) and
// G^N(r) f_i (to u_j).  Every unordered pair is visited once: a wave walks only the upper
// half of the neighbour-tile offsets D (lexicographically D > 0), plus its own tile (D = 0)
// restricted to sources with a larger sorted index than the target; the mirrored offset
// -D carries the same pairs.  The source side accumulates per ring entry in LDS and is
// added to u^N with one FP64 atomic per component and source when the entry retires.
// The sort zeroes u^N.  The order of those atomic additions varies between runs, so
// results agree to rounding, not bitwise (the one-sided kernel below is the reproducible
// variant).
//
// Balanced drain.  LDS traffic, not arithmetic, bounded an earlier form that put every
// accepted pair through an LDS queue (six LDS atomics and twelve operand loads per pair), so
// the target side is kept in registers where possible.  Per batch of 32 ring entries each
// lane tests its own target against all of them (a 32-bit mask; all lanes read the same
// entry, an LDS broadcast).  With Q accepted pairs the batch takes R = ceil(Q / 64) rounds
// of one pair per lane; a lane keeps up to R pairs of its own target (summed in registers)
// and puts the rest in a queue, from which lanes with fewer than R pairs take work in their
// spare rounds (target side by LDS atomics, about 15% of the pairs at uniform density).
// Each lane takes its own sources in cyclic order from its (lane mod c)-th accepted one (c its
// pair count), so that the lanes of a half-wave start on different sources also when their
// accepted sets are alike (fewer collisions on the batch's source accumulators).  The ring
// and target slots are read one value per LDS instruction (ld1).  With stresslet sources the
// same schedule carries the stresslet pair terms as well.
//
// Cutoff test on the matrix cores.  The targets' positions t' and the ring's sources s' are taken
// relative to the centre of the targets' bounding box, so that |s' - t'|^2 < r_c^2 can be tested
// in the expanded form |s'|^2 - 2 s'.t' < r_c^2 - |t'|^2 without cancellation beyond a few ulps of
// (box diagonal + r_c)^2.  A full batch past the own tile (32 sources x 64 targets) is eight
// v_mfma_f64_16x16x4f64 (sources as rows, targets as columns, the sums starting from |s'|^2) whose
// results' sign bits are the tests, instead of 32 broadcast LDS reads and six FP64 operations per
// source: c2 P2P 22.9 -> 21.3 ms, H 12.2 -> 11.3 ms.  The matrix instructions hold the SIMD for 64 cycles
// each (no vector instruction issues meanwhile), so the test costs 128 + 75 issue slots per batch (128 +
// 128 with comparisons and ballots); with the weighted polynomials on scaled positions c2 18.3 -> 17.85 ms,
// c3 165 -> 161 ms when it was made.  The own tile, whose
// pairs also need r > 0 and the index order, and the last, shorter batch keep the direct test;
// the direct difference of repeated positions is exactly 0 also in the centred frame (and scaled by
// a power of two, whether or not the compiler contracts the product into the difference).
constexpr int kSymRing = 64;
constexpr int kUnit = 8;  // consecutive sources dealt at a time to the waves of a chunk (a cache line of u^N)
constexpr int kFar = 1 << 30;  // ring key offset of sources outside the targets' own tile
// Balanced drain: batches of 32 ring entries.  Queue bound: with c_t <= 32 pairs per lane,
// Q = sum c_t and R = ceil(Q / 64) rounds, the excess sum over c_t >= R of (c_t - R) is at most
// Q (32 - R) / 32 <= 2 R (32 - R) <= 512.
constexpr int kBalBatch = 32;
constexpr int kBalExcess = 512;
static_assert(kBalBatch == 32 && kSymRing == 64, "the mask, ring and queue sizes assume 32-entry batches");

// wave ballot of a condition, without materialising it as an integer first
__device__ inline unsigned long long ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Cutoff test of a full batch past the own tile, |s' - t'|^2 < r_c^2  <=>  |s'|^2 - 2 s'.t' + |t'|^2 - r_c^2 < 0,
// for 32 sources x 64 targets by eight v_mfma_f64_16x16x4f64 (sources as rows): the accepted sources of
// each lane's target, as a mask.  On gfx950 lane l = 16 kq + i supplies A[i][kq] and B[kq][i] and
// receives D[4 r + kq][i], r = 0..3.  Batches start at ring slot 0 or 32 (32 entries at a time from a
// 64-slot ring), so the batch's slots need no wrap.  bt: the target operands.  off:
// coordinate mk (below 3) of the centre in the frame of ring[0..2], which s' and t' are relative to (0:
// the ring is centred itself).
__device__ inline unsigned accept_mask(double (&ring)[4][kSymRing], int rhead, const double (&bt)[4], int mi, int mk,
                                       double off)
{
    typedef double v4d __attribute__((ext_vector_type(4)));
    unsigned m = 0;
    // source operand A = (-2 x, -2 y, -2 z, 1): row rho of block mb is slot 8 (rho % 4) + 4 mb + rho / 4,
    // so that result item r of lane (kq, i) -- row 4 r + kq -- is slot 8 kq + 4 mb + r: a lane's eight
    // items are eight consecutive bits of the batch mask, and start from |s'|^2 of eight
    // consecutive slots
    double av[2];
    v4d cv[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const double xk = ld1(ring[mk < 3 ? mk : 0][rhead + 8 * (mi & 3) + 4 * mb + (mi >> 2)]);
        av[mb] = mk < 3 ? -2.0 * (xk - off) : 1.0;
        cv[mb] = *reinterpret_cast<const v4d*>(&ring[3][rhead + 8 * mk + 4 * mb]);
    }
    // the sign bit of an item is its test.  The bits of target 16 nb + i are spread over lanes
    // (kq, i), kq = 0..3: OR over the four rows, kept by the lanes of row nb (the target's own lane)
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        unsigned v = 0;
#pragma unroll
        for (int mb = 1; mb >= 0; --mb) {
            const v4d dd = __builtin_amdgcn_mfma_f64_16x16x4f64(av[mb], bt[nb], cv[mb], 0, 0, 0);
#pragma unroll
            for (int r = 3; r >= 0; --r)  // v = 2 v + sign
                v = __builtin_amdgcn_alignbit(v, (unsigned)__double2hiint(dd[r]), 31);
        }
        v = or_rows4(v << (8 * mk));
        m = mk == nb ? v : m;
        __builtin_amdgcn_sched_barrier(0);
    }
    return m;
}

// ST: stresslet sources too (srec: sorted symmetric tensors, 6 per particle); T^N is odd,
// so the source side of a pair takes -T^N(r) S_target.
template <typename TF, int Lv, bool ST>
__global__ __launch_bounds__(64) void k_p2p_sym(int n, const Rec64* __restrict__ rec,
                                                const double* __restrict__ srec,
                                                const int* __restrict__ start,
                                                const int* __restrict__ chunk_off, Geometry g,
                                                PairArgs a, double* __restrict__ u_near, int nsplit, bool by_unit)
{
    constexpr int NS = ST ? 6 : 1;
    constexpr bool kScaled = !ST && std::is_same<TF, double>::value && Lv > 0;
    using PairCoef = Coef<TF, Lv>;
    __shared__ double tgt[3][kWave];  // t' (x, y, z)
    __shared__ TF tgtf[3][kWave];
    __shared__ TF tgts[NS][kWave];
    __shared__ TF rings[NS][kSymRing];
    __shared__ double acc[3][kWave];
    __shared__ __align__(32) double ring[4][kSymRing];  // s' (x, y, z) and |s'|^2
    __shared__ TF ringf[3][kSymRing];
    __shared__ int ringk[kSymRing];
    constexpr int kB = kBalBatch;
    // FP32: a second copy of the batch's source accumulators, for the odd lanes, rotated by half (its
    // banks differ): the atomics' address and bank conflicts are most of the LDS pipeline's time (H P2P
    // 9.78 -> 9.47 ms, c4 49.8 -> 48.0).  In FP64 it costs a wave per SIMD (16 take 10240 bytes each) and
    // more than it saves: c2 17.6 -> 18.1 ms, and 17.8 with half the queue and two components copied.
    constexpr int kCopied = !ST && std::is_same<TF, float>::value ? 3 : 0;  // components with two copies
    __shared__ double racc[3 + kCopied][kB];
    __shared__ unsigned short queue[kBalExcess];
    static_assert(kSymRing == kWave, "one ring slot per lane");

    // plain block order: an XCD-aware order (each XCD sweeping a contiguous range) was
    // measured 12% slower here, unlike in G2P
    // nsplit waves share a chunk, each taking every nsplit-th of its neighbour tiles (shorter waves: a
    // smaller tail when the last waves of the launch run), or, by_unit, every nsplit-th unit of kUnit
    // consecutive sources, counted through the tiles: small inputs, whose sources may all lie in a tile or
    // two, and whose longest wave is the launch.  Batches of 64 left uneven shares (1e3: 0.037 -> 0.027 ms, 3e4 0.222 ->
    // 0.159, 2e4 in two clusters 0.300 -> 0.264, 1.5e5 0.436 -> 0.426, 24 systems 0.182 -> 0.161); single sources spread the
    // waves' atomics on u^N over eight times the cache lines (the clusters 0.345).
    const int wave = uniform_i((int)blockIdx.x) / nsplit;
    const int part = uniform_i((int)blockIdx.x) % nsplit;
    const int lane = threadIdx.x;
    const int total = chunk_off[g.ntiles * g.nsys];  // chunks of all systems
    if (wave >= total) return;

    int lo = 0, hi = g.ntiles * g.nsys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (chunk_off[mid] <= wave) lo = mid; else hi = mid;
    }
    const int t = lo;
    const int per = 1 << (3 * g.log2B);
    const int t_end = start[(t + 1) * per];
    const int first = start[t * per] + (wave - chunk_off[t]) * kWave;
    const int i = first + lane;
    const bool active = i < t_end;
    const Rec64 me = rec[active ? i : first];
    const double pos = me.x[0] + me.x[1] + me.x[2];
    const bool live = active && pos == pos;  // else the lane accepts no pair (see p2p_candidate)

    // tile t of system sys (the systems of a batch have consecutive tile ranges)
    const int sys = t / g.ntiles, tl = t - sys * g.ntiles, tbase = sys * g.ntiles;
    const int tc[3] = {tl / (g.NT[1] * g.NT[2]), (tl / g.NT[2]) % g.NT[1], tl % g.NT[2]};
    // positions relative to the centre of the targets' bounding box (see the cutoff test above)
    double w[3], blo[3], bhi[3], cen[3], tx[3], oacc[3];
    const double rc2 = kScaled ? a.rc2s : a.rc2;  // of the (scaled) positions relative to the centre
    double tlim = -rc2;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        w[d] = g.B * g.h[d];
        blo[d] = uniform_d(wave_min(me.x[d]));
        bhi[d] = uniform_d(wave_max(me.x[d]));
        cen[d] = uniform_d(0.5 * (blo[d] + bhi[d]));
        tx[d] = live ? me.x[d] - cen[d] : 1e30;
        if (kScaled) tx[d] *= a.scale;
        tlim += tx[d] * tx[d];
        tgt[d][lane] = tx[d];
        tgtf[d][lane] = (TF)me.f[d];
        acc[d][lane] = 0.0;
        if (lane < kB) racc[d][lane] = 0.0;
        if (d < kCopied && lane < kB) racc[3 + d][lane] = 0.0;
        oacc[d] = 0.0;
    }
    if (ST) {
        const int ii = active ? i : first;
#pragma unroll
        for (int c = 0; c < NS; ++c) tgts[c][lane] = (TF)srec[6 * (int64_t)ii + c];
    }
    __syncthreads();
    const int mi = lane & 15, mk = lane >> 4;  // lane = 16 mk + mi
    // target operands of the cutoff test's matrix instructions (see process): B = (x, y, z,
    // |t'|^2 - r_c^2) of targets 16 nb + mi
    double bt[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        const double l = __shfl(tlim, 16 * nb + mi, kWave);
        bt[nb] = mk < 3 ? tgt[mk < 3 ? mk : 0][16 * nb + mi] : l;
    }
    // the stresslet formula (CoefSt) returns its coefficients unscaled
    const double post = ST ? 1.0 : PairCoef::post(a);

    int rhead = 0, rcount = 0;
    const int lane_at = by_unit ? (lane / kUnit) * kUnit * nsplit + lane % kUnit : lane;
    int turn = part;  // tiles or units to pass over before the next of this wave's
    auto skip = [&]() {
        const bool other = turn > 0;  // another wave of this chunk takes it
        turn = other ? turn - 1 : nsplit - 1;
        return other;
    };

    auto process = [&](int cnt) {
        // 1. test: bit j of m is set when this lane's target pairs with batch entry j (all
        //    lanes read the same entry: LDS broadcast)
        //    Sources of other tiles are never at r = 0 and always follow the wave's own
        //    tile in the ring, so a batch whose first entry is not of the own tile needs
        //    only the cutoff test.
        unsigned m = 0;
        const bool own_tile = uniform_i(ringk[rhead]) < kFar;
        if (own_tile) {
            for (int j = 0; j < cnt; ++j) {
                const int slot = (rhead + j) & (kSymRing - 1);
                const double rx = tx[0] - ld1(ring[0][slot]), ry = tx[1] - ld1(ring[1][slot]), rz = tx[2] - ld1(ring[2][slot]);
                const double r2 = rx * rx + ry * ry + rz * rz;
                const bool pass = (r2 < rc2) & (r2 > 0.0) & (ringk[slot] > i);
                m = pass ? (m | (1u << j)) : m;
            }
        } else if (cnt == kB) {
            m = accept_mask(ring, rhead, bt, mi, mk, 0.0);
        } else {
            for (int j = 0; j < cnt; ++j) {
                const int slot = (rhead + j) & (kSymRing - 1);
                const double rx = tx[0] - ld1(ring[0][slot]), ry = tx[1] - ld1(ring[1][slot]), rz = tx[2] - ld1(ring[2][slot]);
                const bool pass = rx * rx + ry * ry + rz * rz < rc2;
                m = pass ? (m | (1u << j)) : m;
            }
        }
        const int c = __popc(m);
        const int qn = wave_sum_i(c);
        const int rounds = (qn + kWave - 1) / kWave;
        // 2. a lane keeps up to `rounds` of its target's pairs, taken in cyclic order from its
        //    (lane mod c)-th accepted source (c: its number of pairs), so that the lanes of a half-wave
        //    start on different sources even when their accepted sets are alike (a
        //    rotation by the lane number alone sent the lanes whose start lies outside a common
        //    band of accepted sources to the band's first source together: same-address LDS
        //    atomics); the excess goes to the queue, for lanes that run out of pairs of their own
        const int rot = c ? select_bit(m, lane % c) : 0;
        const unsigned rm0 = rot ? ((m >> rot) | (m << (kB - rot))) : m;
        unsigned rm = rm0;
        const int own_n = c < rounds ? c : rounds;
        int ex = c - own_n;
        int qx = 0;
        for (;;) {
            const bool wr = ex > 0;
            const unsigned long long bw = ballot(wr);
            if (bw == 0) break;
            if (wr) {
                const int p = 31 - __clz(rm);
                rm ^= 1u << p;
                queue[qx + lanes_below(bw)] = (unsigned short)(lane | (((p + rot) & (kB - 1)) << 6));
                --ex;
            }
            qx += __popcll(bw);
        }
        __syncthreads();
        // 3. `rounds` rounds of one pair per lane; a lane's own target's side is summed in
        //    registers, the source side goes to the batch's source accumulators.
        // The pair (target tt at position p with force tf, ring slot): c = G^N(r) f_source for
        // the target, d = G^N(-r) f_target for the source (r = p - x_source)
        auto pair = [&](double p0, double p1, double p2, TF tf0, TF tf1, TF tf2, int tt, int slot, TF& c0,
                        TF& c1, TF& c2, TF& d0, TF& d1, TF& d2) {
            const double rx = p0 - ld1(ring[0][slot]);
            const double ry = p1 - ld1(ring[1][slot]);
            const double rz = p2 - ld1(ring[2][slot]);
            const double r2 = rx * rx + ry * ry + rz * rz;
            TF a1, b;
            if constexpr (ST) {
                TF al, be;
                CoefSt<TF, Lv>::eval(r2, a, a1, b, al, be);
                apply<TF>(a1, b, (TF)rx, (TF)ry, (TF)rz, ld1(ringf[0][slot]), ld1(ringf[1][slot]), ld1(ringf[2][slot]), c0,
                          c1, c2);
                apply<TF>(a1, b, (TF)rx, (TF)ry, (TF)rz, tf0, tf1, tf2, d0, d1, d2);
                TF ss[6], st[6];
#pragma unroll
                for (int c = 0; c < 6; ++c) {
                    ss[c] = ld1(rings[c][slot]);
                    st[c] = -ld1(tgts[c][tt]);  // T^N(-r) = -T^N(r)
                }
                apply_st<TF>(al, be, (TF)rx, (TF)ry, (TF)rz, ss, c0, c1, c2);
                apply_st<TF>(al, be, (TF)rx, (TF)ry, (TF)rz, st, d0, d1, d2);
            } else {
                PairCoef::eval(r2, a, a1, b);
                apply<TF>(a1, b, (TF)rx, (TF)ry, (TF)rz, ld1(ringf[0][slot]), ld1(ringf[1][slot]), ld1(ringf[2][slot]), c0,
                          c1, c2);
                apply<TF>(a1, b, (TF)rx, (TF)ry, (TF)rz, tf0, tf1, tf2, d0, d1, d2);
            }
        };
        // the source accumulator of component d and batch entry sl that this lane adds to
        const int odd = lane & 1, turned = odd * (kB / 2);
        auto source_sum = [&](int d, int sl) -> double& {
            return d < kCopied ? racc[d + (odd ? 3 : 0)][(sl + turned) & (kB - 1)] : racc[d][sl];
        };
        // 3a. rounds in which every lane still takes a pair of its own target (about a third
        //     at uniform density): no queue, no ballot, and the target's position and force
        //     come from registers
        const int own_all = wave_min_small(own_n);
        // the lane's target (position, force).  At the reduced-cost FP64 levels the all-own rounds
        // sum the target side straight into the FMAs, and a lane that runs out of pairs of its
        // own overwrites these registers with a donated pair's target in the queue rounds (c2
        // P2P -1.4%); at level 0 and in FP32 both cost more registers or time than they save
        constexpr bool kRegTarget = std::is_same<TF, double>::value && Lv > 0;
        double px = tx[0], py = tx[1], pz = tx[2];
        TF mf0 = (TF)me.f[0], mf1 = (TF)me.f[1], mf2 = (TF)me.f[2];
        for (int r = 0; r < own_all; ++r) {
            const int sl = (__builtin_ctz(rm) + rot) & (kB - 1);
            rm &= rm - 1;
            const int slot = rhead + sl;
            if constexpr (!ST && kRegTarget) {
                // the target side summed straight into the FMAs: oacc += a1 f_s + b (r.f_s) r
                const double rx = px - ld1(ring[0][slot]), ry = py - ld1(ring[1][slot]), rz = pz - ld1(ring[2][slot]);
                double a1, b;
                PairCoef::eval(rx * rx + ry * ry + rz * rz, a, a1, b);
                const double s0 = ld1(ringf[0][slot]), s1 = ld1(ringf[1][slot]), s2 = ld1(ringf[2][slot]);
                const double rs = (rx * s0 + ry * s1 + rz * s2) * b;
                oacc[0] = fma(rs, rx, fma(a1, s0, oacc[0]));
                oacc[1] = fma(rs, ry, fma(a1, s1, oacc[1]));
                oacc[2] = fma(rs, rz, fma(a1, s2, oacc[2]));
                const double rt = (rx * mf0 + ry * mf1 + rz * mf2) * b;
                atomicAdd(&source_sum(0, sl), fma(a1, mf0, rt * rx));
                atomicAdd(&source_sum(1, sl), fma(a1, mf1, rt * ry));
                atomicAdd(&source_sum(2, sl), fma(a1, mf2, rt * rz));
                continue;
            }
            TF c0, c1, c2, d0, d1, d2;
            pair(px, py, pz, mf0, mf1, mf2, lane, slot, c0, c1, c2, d0, d1, d2);
            oacc[0] += (double)c0;
            oacc[1] += (double)c1;
            oacc[2] += (double)c2;
            atomicAdd(&source_sum(0, sl), (double)d0);
            atomicAdd(&source_sum(1, sl), (double)d1);
            atomicAdd(&source_sum(2, sl), (double)d2);
        }
        // 3b. the remaining rounds, one pair per lane: the lane's own target while it has
        //     pairs, then queue entries in order (target side by LDS atomics)
        int qb = 0;
        for (int r = own_all; r < rounds; ++r) {
            // every lane reads a queue entry (in range, used only by donated lanes)
            const bool own = r < own_n;
            const unsigned long long bi = ballot(!own);
            const int q = qb + lanes_below(bi);
            qb += __popcll(bi);
            const bool don = !own && q < qx;
            const int e = queue[q < qx ? q : 0];
            const int pb = __builtin_ctz(rm);  // used by own lanes only (rm != 0)
            if constexpr (!kRegTarget) rm = own ? (rm & (rm - 1)) : rm;
            const int tt = own ? lane : (e & (kWave - 1));
            const int sl = own ? ((pb + rot) & (kB - 1)) : ((e >> 6) & (kB - 1));
            const int slot = rhead + sl;
            // own lanes take their target from registers, donated lanes from LDS (the volatile
            // loads stay under the branch, so own lanes add no LDS traffic)
            TF c0, c1, c2, d0, d1, d2;
            if constexpr (kRegTarget) {
                // a lane that is not own in this round is not own in any later one: it
                // overwrites its target registers
                if (!own) {
                    px = ld1(tgt[0][tt]);
                    py = ld1(tgt[1][tt]);
                    pz = ld1(tgt[2][tt]);
                    mf0 = ld1(tgtf[0][tt]);
                    mf1 = ld1(tgtf[1][tt]);
                    mf2 = ld1(tgtf[2][tt]);
                }
                pair(px, py, pz, mf0, mf1, mf2, tt, slot, c0, c1, c2, d0, d1, d2);
                if (own) {
                    // an empty volatile asm keeps this a branch (the if-converted form takes
                    // two selects per component)
                    asm volatile("");
                    oacc[0] += (double)c0;
                    oacc[1] += (double)c1;
                    oacc[2] += (double)c2;
                    rm &= rm - 1;
                }
            } else {
                double q0 = px, q1 = py, q2 = pz;
                TF g0 = mf0, g1 = mf1, g2 = mf2;
                if (!own) {
                    q0 = ld1(tgt[0][tt]);
                    q1 = ld1(tgt[1][tt]);
                    q2 = ld1(tgt[2][tt]);
                    g0 = ld1(tgtf[0][tt]);
                    g1 = ld1(tgtf[1][tt]);
                    g2 = ld1(tgtf[2][tt]);
                }
                pair(q0, q1, q2, g0, g1, g2, tt, slot, c0, c1, c2, d0, d1, d2);
                if (own) {
                    oacc[0] += (double)c0;
                    oacc[1] += (double)c1;
                    oacc[2] += (double)c2;
                }
            }
            if (don) {
                atomicAdd(&acc[0][tt], (double)c0);
                atomicAdd(&acc[1][tt], (double)c1);
                atomicAdd(&acc[2][tt], (double)c2);
            }
            if (own || don) {
                atomicAdd(&source_sum(0, sl), (double)d0);
                atomicAdd(&source_sum(1, sl), (double)d1);
                atomicAdd(&source_sum(2, sl), (double)d2);
            }
        }
        __syncthreads();
        // retire the cnt ring sources: their source-side sums go to u^N
        if (lane < cnt) {
            const int slot = (rhead + lane) & (kSymRing - 1);
            double v[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                v[d] = racc[d][lane];
                racc[d][lane] = 0.0;
                if (d < kCopied) {
                    const int e = (lane + kB / 2) & (kB - 1);
                    v[d] += racc[3 + d][e];
                    racc[3 + d][e] = 0.0;
                }
            }
            if (v[0] != 0.0 || v[1] != 0.0 || v[2] != 0.0) {
                const int64_t jj = ringk[slot] & (kFar - 1);
                unsafeAtomicAdd(&u_near[jj], post * v[0]);
                unsafeAtomicAdd(&u_near[(int64_t)n + jj], post * v[1]);
                unsafeAtomicAdd(&u_near[2 * (int64_t)n + jj], post * v[2]);
            }
        }
        __syncthreads();
    };

    for (int dx = 0; dx <= g.S[0]; ++dx) {
        const int ux = tc[0] + dx;
        const int fx = floor_div(ux, g.NT[0]);
        const int wx = ux - fx * g.NT[0];
        const double shx = fx * g.L[0];
        const double gx = fmax(0.0, fmax(ux * w[0] - bhi[0], blo[0] - (ux + 1) * w[0]));
        for (int dy = (dx == 0 ? 0 : -g.S[1]); dy <= g.S[1]; ++dy) {
            const int uy = tc[1] + dy;
            const int fy = floor_div(uy, g.NT[1]);
            const int wy = uy - fy * g.NT[1];
            const double shy = fy * g.L[1];
            const double gy = fmax(0.0, fmax(uy * w[1] - bhi[1], blo[1] - (uy + 1) * w[1]));
            if (gx * gx + gy * gy >= a.rc2) continue;
            for (int dz = (dx == 0 && dy == 0 ? 0 : -g.S[2]); dz <= g.S[2]; ++dz) {
                const int uz = tc[2] + dz;
                const int fz = floor_div(uz, g.NT[2]);
                const int wz = uz - fz * g.NT[2];
                const double shz = fz * g.L[2];
                const double gz = fmax(0.0, fmax(uz * w[2] - bhi[2], blo[2] - (uz + 1) * w[2]));
                if (gx * gx + gy * gy + gz * gz >= a.rc2) continue;
                if (!by_unit && skip()) continue;
                const bool own = (dx == 0 && dy == 0 && dz == 0);
                const int nt = tbase + (wx * g.NT[1] + wy) * g.NT[2] + wz;
                // own tile: sources below the first target can pair with none of them
                const int sa = own ? first : start[nt * per], sb = start[(nt + 1) * per];
                const int koff = own ? 0 : kFar;
                const int step = by_unit ? kWave * nsplit : kWave;
                int base = by_unit ? sa + turn * kUnit : sa;
                for (; base < sb; base += step) {
                    const int s = base + lane_at;
                    bool keep = false;
                    double sx = 0, sy = 0, sz = 0, n2 = 0, f0 = 0, f1 = 0, f2 = 0;
                    if (s < sb) {
                        const Rec64& q = rec[s];
                        sx = q.x[0] + shx;
                        sy = q.x[1] + shy;
                        sz = q.x[2] + shz;
                        f0 = q.f[0];
                        f1 = q.f[1];
                        f2 = q.f[2];
                        const double ex = fmax(0.0, fmax(blo[0] - sx, sx - bhi[0]));
                        const double ey = fmax(0.0, fmax(blo[1] - sy, sy - bhi[1]));
                        const double ez = fmax(0.0, fmax(blo[2] - sz, sz - bhi[2]));
                        sx -= cen[0];
                        sy -= cen[1];
                        sz -= cen[2];
                        if (kScaled) {
                            sx *= a.scale;
                            sy *= a.scale;
                            sz *= a.scale;
                        }
                        n2 = sx * sx + sy * sy + sz * sz;
                        keep = p2p_candidate(ex * ex + ey * ey + ez * ez, n2, a.rc2);
                    }
                    // append in two halves so the 64-slot ring never holds more than 63
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const bool mine = keep && ((lane >> 5) == half);
                        const unsigned long long bm = __ballot(mine);
                        if (mine) {
                            const int slot = (rhead + rcount + lanes_below(bm)) & (kSymRing - 1);
                            ring[0][slot] = sx;
                            ring[1][slot] = sy;
                            ring[2][slot] = sz;
                            ring[3][slot] = n2;
                            ringf[0][slot] = (TF)f0;
                            ringf[1][slot] = (TF)f1;
                            ringf[2][slot] = (TF)f2;
                            ringk[slot] = koff + s;
                            if (ST) {
#pragma unroll
                                for (int c = 0; c < NS; ++c) rings[c][slot] = (TF)srec[6 * (int64_t)s + c];
                            }
                        }
                        rcount += __popcll(bm);
                        __syncthreads();
                        while (rcount >= kB) {
                            process(kB);
                            rhead = (rhead + kB) & (kSymRing - 1);
                            rcount -= kB;
                        }
                    }
                }
                if (by_unit) {
                    turn = (base - sa) / kUnit - (sb - sa + kUnit - 1) / kUnit;
                    while (turn >= nsplit) turn -= nsplit;
                }
            }
        }
    }
    while (rcount > 0) {
        const int c = rcount < kB ? rcount : kB;
        process(c);
        rhead = (rhead + c) & (kSymRing - 1);
        rcount -= c;
    }
    if (active) {
        unsafeAtomicAdd(&u_near[i], post * (acc[0][lane] + oacc[0]));
        unsafeAtomicAdd(&u_near[(int64_t)n + i], post * (acc[1][lane] + oacc[1]));
        unsafeAtomicAdd(&u_near[2 * (int64_t)n + i], post * (acc[2][lane] + oacc[2]));
    }
}

// ---------------------------------------------------------------- one-sided form
// The deterministic mode's kernel: a wave's targets meet every source around them (each pair is evaluated
// from both of its sides), so that a sum is made by one block, in a fixed order: registers and the
// wave's own LDS, no global atomics.  The balanced drain above without its source side: a lane keeps
// up to R of its target's pairs, in the order of the ring (lanes that accept the same source read it
// together), and the excess goes through the queue to lanes without pairs of their own.
// The own tile comes first, so that only a wave's first batches need r > 0.  NW waves share a chunk, wave
// w takes the sources w, w + NW, ... of a row, and their sums are added in wave order.
// Sources are dealt one by one along a row of tiles, so that the waves of a chunk get alike shares of
// every region around it (by batches of 64 in the order of the sort, the largest share of eight waves was
// 1.39 times the mean at 3e4, and the block waits for it: 0.36 -> 0.31 ms at 3e4, 31.5 -> 29.2 at 1e6).
// Bound by FP64 issue, and at small sizes by the waves in flight: 1e6 uniform at 1e-8, 128^3, 25.8 ms (33.9
// with every pair through an LDS queue and its three LDS atomics); 3e4, KB, 0.31 (0.48).
template <typename TF, int Lv, int NW>
__global__ __launch_bounds__(64 * NW, sizeof(TF) == 8 && Lv == 0 ? 4 : 5) void k_p2p_one(int n, const Rec64* __restrict__ rec,
                                                     const int* __restrict__ start,
                                                     const int* __restrict__ chunk_off, Geometry g, PairArgs a,
                                                     double* __restrict__ u_near)
{
    constexpr bool kScaled = std::is_same<TF, double>::value && Lv > 0;
    using PairCoef = Coef<TF, Lv>;
    constexpr int kB = kBalBatch;
    __shared__ double tgt_[NW][3][kWave];  // (x, y, z)
    __shared__ double acc_[NW][3][kWave];
    __shared__ __align__(32) double ring_[NW][4][kSymRing];  // (x, y, z) and |s'|^2
    __shared__ TF ringf_[NW][3][kSymRing];
    __shared__ unsigned short queue_[NW][kBalExcess];

    const int wave = uniform_i((int)blockIdx.x);
    const int wid = uniform_i((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    double(&tgt)[3][kWave] = tgt_[wid];
    double(&acc)[3][kWave] = acc_[wid];
    double(&ring)[4][kSymRing] = ring_[wid];
    TF(&ringf)[3][kSymRing] = ringf_[wid];
    unsigned short(&queue)[kBalExcess] = queue_[wid];
    const int total = chunk_off[g.ntiles * g.nsys];  // chunks of all systems
    if (wave >= total) return;

    // tile of this wave: largest t with chunk_off[t] <= wave
    int lo = 0, hi = g.ntiles * g.nsys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (chunk_off[mid] <= wave) lo = mid; else hi = mid;
    }
    const int t = lo;
    const int per = 1 << (3 * g.log2B);
    const int t_end = start[(t + 1) * per];
    const int first = start[t * per] + (wave - chunk_off[t]) * kWave;
    const int i = first + lane;
    const bool active = i < t_end;
    const Rec64 me = rec[active ? i : first];
    const double pos = me.x[0] + me.x[1] + me.x[2];
    const bool live = active && pos == pos;  // else the lane accepts no pair (see p2p_candidate)

    // tile t of system sys (the systems of a batch have consecutive tile ranges)
    const int sys = t / g.ntiles, tl = t - sys * g.ntiles, tbase = sys * g.ntiles;
    const int tc[3] = {tl / (g.NT[1] * g.NT[2]), (tl / g.NT[2]) % g.NT[1], tl % g.NT[2]};
    double w[3], blo[3], bhi[3], cen[3], tx[3], oacc[3];
    // Positions are the particles' own (times the power of two of the reduced-cost levels), so that the
    // differences of the pairs are the direct ones, exact for close pairs and 0 for a target and its own
    // record; the matrix test alone takes them relative to the centre of the targets' bounding box (t', s').
    const double rc2 = kScaled ? a.rc2s : a.rc2, scale = kScaled ? a.scale : 1.0;
    double tlim = -rc2;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        w[d] = g.B * g.h[d];
        blo[d] = uniform_d(wave_min(me.x[d]));
        bhi[d] = uniform_d(wave_max(me.x[d]));
        cen[d] = uniform_d(0.5 * (blo[d] + bhi[d]) * scale);
        tx[d] = live ? me.x[d] * scale : 1e30;
        const double tc = live ? tx[d] - cen[d] : 1e30;
        tlim += tc * tc;
        tgt[d][lane] = tx[d];
        acc[d][lane] = 0.0;
        oacc[d] = 0.0;
    }
    wave_lds_sync();
    const int mi = lane & 15, mk = lane >> 4;  // lane = 16 mk + mi
    const double cen_k = mk == 0 ? cen[0] : mk == 1 ? cen[1] : cen[2];
    double bt[4];  // target operands of accept_mask
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        const double l = __shfl(tlim, 16 * nb + mi, kWave);
        bt[nb] = mk < 3 ? tgt[mk < 3 ? mk : 0][16 * nb + mi] - cen_k : l;
    }

    int rhead = 0, rcount = 0;
    int own_left = 0;  // ring entries of the own tile

    auto process = [&](int cnt) {
        unsigned m = 0;
        if (own_left == 0 && cnt == kB) {
            m = accept_mask(ring, rhead, bt, mi, mk, cen_k);
        } else {
            for (int j = 0; j < cnt; ++j) {
                const int slot = (rhead + j) & (kSymRing - 1);
                const double rx = tx[0] - ld1(ring[0][slot]), ry = tx[1] - ld1(ring[1][slot]), rz = tx[2] - ld1(ring[2][slot]);
                const double r2 = rx * rx + ry * ry + rz * rz;
                const bool pass = (r2 < rc2) & (r2 > 0.0);
                m = pass ? (m | (1u << j)) : m;
            }
        }
        own_left = own_left > cnt ? own_left - cnt : 0;
        const int c = __popc(m);
        const int qn = wave_sum_i(c);
        const int rounds = (qn + kWave - 1) / kWave;
        const int own_n = c < rounds ? c : rounds;
        // the excess, from the mask's upper end, to the queue
        unsigned rm = m;
        int ex = c - own_n;
        int qx = 0;
        for (;;) {
            const bool wr = ex > 0;
            const unsigned long long bw = ballot(wr);
            if (bw == 0) break;
            if (wr) {
                const int p = 31 - __clz(rm);
                rm ^= 1u << p;
                queue[qx + lanes_below(bw)] = (unsigned short)(lane | (p << 6));
                --ex;
            }
            qx += __popcll(bw);
        }
        wave_lds_sync();
        // c = G^N(r) f_source of the pair (target at p, ring slot)
        auto pair = [&](double p0, double p1, double p2, int slot, double& c0, double& c1, double& c2) {
            const double rx = p0 - ld1(ring[0][slot]), ry = p1 - ld1(ring[1][slot]), rz = p2 - ld1(ring[2][slot]);
            TF a1, b, e0, e1, e2;
            PairCoef::eval(rx * rx + ry * ry + rz * rz, a, a1, b);
            apply<TF>(a1, b, (TF)rx, (TF)ry, (TF)rz, ld1(ringf[0][slot]), ld1(ringf[1][slot]), ld1(ringf[2][slot]),
                      e0, e1, e2);
            c0 = (double)e0;
            c1 = (double)e1;
            c2 = (double)e2;
        };
        // rounds in which every lane takes a pair of its own target: summed in registers
        const int own_all = wave_min_small(own_n);
        double px = tx[0], py = tx[1], pz = tx[2];
        for (int r = 0; r < own_all; ++r) {
            const int slot = rhead + __builtin_ctz(rm);
            rm &= rm - 1;
            double c0, c1, c2;
            pair(px, py, pz, slot, c0, c1, c2);
            oacc[0] += c0;
            oacc[1] += c1;
            oacc[2] += c2;
        }
        // the rest: a lane without a pair of its own takes a queued one (its target by LDS atomics; a
        // lane that is not own in a round is not own in any later one)
        int qb = 0;
        for (int r = own_all; r < rounds; ++r) {
            const bool own = r < own_n;
            const unsigned long long bi = ballot(!own);
            const int q = qb + lanes_below(bi);
            qb += __popcll(bi);
            const bool don = !own && q < qx;
            const int e = queue[q < qx ? q : 0];
            const int tt = e & (kWave - 1);
            const int slot = rhead + (own ? __builtin_ctz(rm) : (e >> 6) & (kB - 1));
            if (!own) {
                px = ld1(tgt[0][tt]);
                py = ld1(tgt[1][tt]);
                pz = ld1(tgt[2][tt]);
            }
            double c0, c1, c2;
            pair(px, py, pz, slot, c0, c1, c2);
            if (own) {
                asm volatile("");  // keeps this a branch
                oacc[0] += c0;
                oacc[1] += c1;
                oacc[2] += c2;
                rm &= rm - 1;
            }
            if (don) {
                atomicAdd(&acc[0][tt], c0);
                atomicAdd(&acc[1][tt], c1);
                atomicAdd(&acc[2][tt], c2);
            }
        }
        wave_lds_sync();
    };

    // sources [sa, sb) of the tiles with the shift (shx, shy, shz)
    auto sources = [&](int sa, int sb, double shx, double shy, double shz, bool own) {
        for (int base = sa; base < sb; base += kWave * NW) {
            const int s = base + lane * NW + wid;
            bool keep = false;
            double sx = 0, sy = 0, sz = 0, n2 = 0, f0 = 0, f1 = 0, f2 = 0;
            if (s < sb) {
                const Rec64& q = rec[s];
                sx = q.x[0] + shx;
                sy = q.x[1] + shy;
                sz = q.x[2] + shz;
                f0 = q.f[0];
                f1 = q.f[1];
                f2 = q.f[2];
                const double ex = fmax(0.0, fmax(blo[0] - sx, sx - bhi[0]));
                const double ey = fmax(0.0, fmax(blo[1] - sy, sy - bhi[1]));
                const double ez = fmax(0.0, fmax(blo[2] - sz, sz - bhi[2]));
                sx *= scale;
                sy *= scale;
                sz *= scale;
                const double cx = sx - cen[0], cy = sy - cen[1], cz = sz - cen[2];
                n2 = cx * cx + cy * cy + cz * cz;
                keep = p2p_candidate(ex * ex + ey * ey + ez * ez, n2, a.rc2);
            }
            // append in two halves so the 64-slot ring never holds more than 63
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const bool mine = keep && ((lane >> 5) == half);
                const unsigned long long bm = ballot(mine);
                if (mine) {
                    const int slot = (rhead + rcount + lanes_below(bm)) & (kSymRing - 1);
                    ring[0][slot] = sx;
                    ring[1][slot] = sy;
                    ring[2][slot] = sz;
                    ring[3][slot] = n2;
                    ringf[0][slot] = (TF)f0;
                    ringf[1][slot] = (TF)f1;
                    ringf[2][slot] = (TF)f2;
                }
                rcount += __popcll(bm);
                if (own) own_left += __popcll(bm);
                wave_lds_sync();
                if (rcount >= kB) {
                    process(kB);
                    rhead = (rhead + kB) & (kSymRing - 1);
                    rcount -= kB;
                }
            }
        }
    };
    // the own tile (row -1), then the rows of tiles along z, whose consecutive tiles in reach (of one
    // periodic image) are consecutive sources
    const int ny = 2 * g.S[1] + 1, nrow = (2 * g.S[0] + 1) * ny;
    for (int row = -1; row < nrow; ++row) {
        const int dx = row < 0 ? 0 : row / ny - g.S[0], dy = row < 0 ? 0 : row % ny - g.S[1];
        const int ux = tc[0] + dx, uy = tc[1] + dy;
        const int fx = floor_div(ux, g.NT[0]), fy = floor_div(uy, g.NT[1]);
        const double shx = fx * g.L[0], shy = fy * g.L[1];
        const double gx = fmax(0.0, fmax(ux * w[0] - bhi[0], blo[0] - (ux + 1) * w[0]));
        const double gy = fmax(0.0, fmax(uy * w[1] - bhi[1], blo[1] - (uy + 1) * w[1]));
        if (gx * gx + gy * gy >= a.rc2) continue;
        const int line = tbase + ((ux - fx * g.NT[0]) * g.NT[1] + uy - fy * g.NT[1]) * g.NT[2];
        const int z0 = row < 0 ? 0 : -g.S[2], z1 = row < 0 ? 0 : g.S[2];
        int sa = 0, sb = 0, image = 0;  // the run of tiles so far
        for (int dz = z0; dz <= z1 + 1; ++dz) {
            const int uz = tc[2] + dz, fz = floor_div(uz, g.NT[2]);
            const double gz = fmax(0.0, fmax(uz * w[2] - bhi[2], blo[2] - (uz + 1) * w[2]));
            const bool own = dx == 0 && dy == 0 && dz == 0;
            const bool take = dz <= z1 && gx * gx + gy * gy + gz * gz < a.rc2 && own == (row < 0);
            const int nt = line + uz - fz * g.NT[2];
            if (take && sb > sa && fz == image) {
                sb = start[(nt + 1) * per];
                continue;
            }
            sources(sa, sb, shx, shy, image * g.L[2], row < 0);
            sa = sb = 0;
            if (take) {
                sa = start[nt * per];
                sb = start[(nt + 1) * per];
                image = fz;
            }
        }
    }
    if (rcount > 0) process(rcount);
#pragma unroll
    for (int d = 0; d < 3; ++d) acc[d][lane] += oacc[d];
    if (NW > 1) __syncthreads();
    if (active && wid == 0) {
        const double post = PairCoef::post(a);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double v = acc_[0][d][lane];
#pragma unroll
            for (int k = 1; k < NW; ++k) v += acc_[k][d][lane];
            u_near[d * (int64_t)n + i] = post * v;
        }
    }
}

}  // namespace

namespace {

PairArgs pair_args(const Plan& pl, int lv)
{
    PairArgs a;
    a.xi = pl.xi;
    a.xi2 = pl.xi * pl.xi;
    a.rc2 = pl.rc * pl.rc;
    a.four_xi_over_sqrtpi = 4.0 * pl.xi / sqrt(M_PI);
    a.six_xi_over_sqrtpi = 6.0 * pl.xi / sqrt(M_PI);
    a.four_xi3_over_sqrtpi = 4.0 * pl.xi * pl.xi * pl.xi / sqrt(M_PI);
    const double* ms = lv == 2 ? kScreenM64f : lv == 1 ? kScreenM64s : kScreenM64;
    const int ds = lv == 2 ? kScreenDeg64f : lv == 1 ? kScreenDeg64s : kScreenDeg64;
    for (int k = 0; k < kScreenDeg64; ++k) a.ms[k] = k < ds ? ms[k] : 0.0;
    a.lead_st = lv == 2 ? kScreenLead64f : lv == 1 ? kScreenLead64s : kScreenLead64;
    const double* mw = lv == 2 ? kScreenV2 : kScreenV1;
    const int dw = lv == 2 ? kScreenDegV2 : kScreenDegV1;
    // X = kappa r = ratio (scale r): the monic polynomial in X is ratio^dw times the one of these coefficients
    const double kappa = pl.xi * sqrt(kLog2e);
    a.scale = exp2(rint(log2(kappa)));
    const double ratio = kappa / a.scale;
    for (int k = 0; k < kScreenDegV1; ++k) a.mw[k] = k < dw ? mw[k] * pow(ratio, k - dw) : 0.0;
    a.lead_s = lv == 0 ? kScreenLead64 : (lv == 2 ? kScreenLeadV2 : kScreenLeadV1) * pow(ratio, dw);
    const double* me = lv == 2 ? kExpM2 : kExpM1;
    const int de = lv == 2 ? kExpDeg2 : kExpDeg1;
    for (int k = 0; k < kExpDeg1; ++k) a.me[k] = k < de ? me[k] : 0.0;
    a.lead_e = lv == 0 ? 1.0 : lv == 2 ? kExpLead2 : kExpLead1;
    a.zc = -a.xi2 * kLog2e;
    a.zc32 = (float)a.zc;
    a.rc2s = a.rc2 * (a.scale * a.scale);
    a.zs = a.zc / (a.scale * a.scale);
    a.g = kTwoOverSqrtPi / a.lead_st;
    a.h = a.four_xi_over_sqrtpi / a.lead_s;
    a.hs = a.h / a.scale;
    a.post = a.lead_s * a.lead_e;
    for (int k = 0; k <= kScreenDeg32; ++k) a.c32[k] = (float)kScreenC32[k];
    return a;
}

__global__ void k_zero_u64(unsigned long long* p) { *p = 0ull; }

}  // namespace

hipError_t launch_count_pairs(const Plan& pl, const Work& w, int n, unsigned long long* count, hipStream_t s,
                              int nsys)
{
    hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(1), 0, s, count);
    if (n > 0) {
        const PairArgs a = pair_args(pl, 0);
        Geometry g = pl.g;
        g.nsys = nsys;
        const int64_t waves = (int64_t)g.ntiles * nsys + (n + kWave - 1) / kWave;
        hipLaunchKernelGGL(k_count_pairs, dim3((unsigned)waves), dim3(kWave), 0, s, (const Rec64*)w.rec, w.start,
                           w.chunk_off, g, a, count);
    }
    return hipGetLastError();
}

// the FP64 pair formula's accuracy level for a plan's tolerance (see PairArgs)
static int pair_level(double tol) { return tol >= 1e-8 ? 2 : tol >= 1e-10 ? 1 : 0; }

// Waves per chunk of the deterministic kernel, by the plan alone (a system's sums must not depend on
// what else is evaluated with it): more where even the plan's largest input has few chunks.  P2P ms at
// 1 / 2 / 4 / 8 / 16 waves: 24 chunks (1e3 uniform, FP64) 0.214 / 0.123 / 0.078 / 0.064 / 0.074; 533 (3e4, KB)
// 1.16 / 0.73 / 0.39 / 0.31 / 0.35; 1536 (6.6e4) 0.48 / 0.33 / 0.28 / 0.34 / 0.55; 3637 (2e5) 2.00 / 1.67 / 1.48 /
// 1.67 / 2.34; 19721 (1e6, 256^3) 4.83 / 4.87 / 4.98 / 6.47 / 10.3, (1e6, 128^3) 26.4 / 26.0 / 25.3 / 29.2 / 39.6.
// Blocks of four waves leave a CU room for five of them, of eight (61 KB of LDS) for two.
template <typename TF, int Lv>
void launch_p2p_det(const Plan& pl, const Work& w, int n, hipStream_t s, const Geometry& g, const PairArgs& a,
                    dim3 grid)
{
    const int64_t chunks = (int64_t)pl.g.ntiles + (pl.p.n_max + kWave - 1) / kWave;
    auto launch = [&](auto kernel, int nw) {
        hipLaunchKernelGGL(kernel, grid, dim3(nw * kWave), 0, s, n, (const Rec64*)w.rec, w.start, w.chunk_off, g, a,
                           w.u_near);
    };
    if (chunks < 1024) launch(k_p2p_one<TF, Lv, 8>, 8);
    else launch(k_p2p_one<TF, Lv, 4>, 4);
}

template <typename TF, int Lv, bool ST>
void launch_p2p_sym(const Work& w, int n, hipStream_t s, const Geometry& g, const PairArgs& a, dim3 grid, int split,
                    bool by_unit)
{
    hipLaunchKernelGGL((k_p2p_sym<TF, Lv, ST>), grid, dim3(kWave), 0, s, n, (const Rec64*)w.rec, w.srec, w.start,
                       w.chunk_off, g, a, w.u_near, split, by_unit);
}

hipError_t launch_p2p(const Plan& pl, const Work& w, int n, hipStream_t s, bool st, int nsys)
{
    if (n <= 0) return hipSuccess;
    const bool f64 = pl.mode == EWALD_FP64;
    const int lv = f64 ? pair_level(pl.p.tol) : -1;  // -1: the FP32 formula
    const PairArgs a = pair_args(pl, lv < 0 ? 0 : lv);
    Geometry g = pl.g;
    g.nsys = nsys;
    const int64_t waves = (int64_t)g.ntiles * nsys + (n + kWave - 1) / kWave;
    const dim3 grid((unsigned)waves);
    if (pl.deterministic && !st) {
        // FP32 bulk accumulates in FP64 as well: LDS atomic adds of FP64 are fast on
        // gfx950, those of FP32 are not (measured: 3x slower kernel)
        switch (lv) {
        case 0: launch_p2p_det<double, 0>(pl, w, n, s, g, a, grid); break;
        case 1: launch_p2p_det<double, 1>(pl, w, n, s, g, a, grid); break;
        case 2: launch_p2p_det<double, 2>(pl, w, n, s, g, a, grid); break;
        default: launch_p2p_det<float, 0>(pl, w, n, s, g, a, grid); break;
        }
        return hipGetLastError();
    }
    // Symmetric kernel: waves per chunk.  Three shorten the launch's tail; more fill the chip where the chunks
    // are few, and even out the chunks of clustered inputs, until a wave's own start and end outweigh its
    // share.  P2P ms by waves per chunk:
    //                                          3      5      7      13     21     33     49     65
    //     24 chunks (1e3, FP64)              0.061  0.046  0.041  0.034  0.029  0.027   -    0.024
    //     40 chunks (2e3)                      -      -      -      -      -    0.039  0.032  0.033
    //     62 chunks (3.4e3)                    -      -      -      -      -    0.042  0.051  0.047
    //    441 chunks (2e4 in 2 clusters, FP32) 1.01  0.61   0.55   0.36   0.26   0.27    -    0.26
    //    533 chunks (3e4, FP64)              0.23   0.19   0.16   0.16   0.16   0.19    -    0.26
    //   1544 chunks (6.6e4, FP32)            0.56   0.54   0.54   0.59   0.67   0.76    -    1.08
    //   3368 chunks (1.5e5, FP64)            0.426  0.418  0.449  0.54   0.69   0.83    -    1.26
    //   3412 chunks (24 systems of 5e3, FP32) 0.16  0.17   0.19   0.25   0.31   0.40    -    0.66
    // (49 up to 48 chunks: between the two sizes measured on its sides.)  Odd, so that the waves of a chunk,
    // consecutive blocks, spread over the XCDs (with 8 or 16, all the chunks' first waves, the heaviest,
    // meet on one).  With stresslet sources fewer waves fit a CU (16 KB of LDS each) and the pairs cost more:
    //                                          3      5      7      13     21     33
    //   1294 chunks (5e4 at 1e-8)            0.218  0.216  0.239  0.30   0.35   0.44
    //   5200 chunks (3e5, FP32)              1.70   1.64   1.67   1.70   1.88   2.22
    // What is dealt: units of kUnit sources below 8192 chunks (see the kernel), neighbour tiles above, where on
    // uniform inputs a wave's compact batches are worth more than even shares; three waves, ms by tiles / units:
    //   uniform    5200 chunks 1.36 / 1.24; 8784 (3e5, FP64) 0.58 / 0.63; 11909 (5e5) 1.12 / 1.16; 19721 (1e6 on 256^3)
    //              3.50 / 3.61, (c2) 17.6 / 18.4, (H) 9.47 / 9.93; 78884 (c4) 48.0 / 50.3
    //   clustered  5200 (3e5 in 30, FP64) 11.4 / 7.9; 8784 (3e5 in 30) 7.5-8.5 / 5.6; 11909 (5e5 in 50) 11.0 / 9.4;
    //              19721 (1e6 in 100) 21.1 / 19.3, FP32 16.0 / 13.5; 189018 (c3) 164.7 / 167.4
    // Chunks are counted as the launch's bound, tiles and n / 64, before the particles are known, so that
    // clustered inputs of 3e5 to 1e6 go by tiles, which is the slower side for them.
    const int64_t fill = ((st ? 4608 : 9216) / waves) | 1;
    const int64_t least = st && waves < 8192 ? 5 : 3, most = waves <= 48 ? 49 : 33;
    const int kSplit = (int)std::min<int64_t>(most, std::max(least, fill));
    const bool by_unit = waves < 8192;
    const dim3 sgrid((unsigned)(waves * kSplit));
    if (st) {
        switch (lv) {
        case 0: launch_p2p_sym<double, 0, true>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
        case 1: launch_p2p_sym<double, 1, true>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
        case 2: launch_p2p_sym<double, 2, true>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
        default: launch_p2p_sym<float, 0, true>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
        }
        return hipGetLastError();
    }
    switch (lv) {
    case 0: launch_p2p_sym<double, 0, false>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
    case 1: launch_p2p_sym<double, 1, false>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
    case 2: launch_p2p_sym<double, 2, false>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
    default: launch_p2p_sym<float, 0, false>(w, n, s, g, a, sgrid, kSplit, by_unit); break;
    }
    return hipGetLastError();
}

}  // namespace ewald
