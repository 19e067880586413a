// Device building blocks: Philox4x32-10, per-period weather terms, the FBP
// rate evaluation of one cell, and the directional rates of eq. (1).
// Everything is templated on the arithmetic type R (double or float).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "fuel_table.h"
#include "ln64.h"
#include "types.h"

namespace c2f {

// ------------------------------------------------------------------ math
// Explicit precision dispatch so float code never widens to double.
__device__ __forceinline__ double m_exp(double x) { return exp(x); }
__device__ __forceinline__ float m_exp(float x) { return expf(x); }
__device__ __forceinline__ double m_expm1(double x) { return expm1(x); }
__device__ __forceinline__ float m_expm1(float x) { return expm1f(x); }
__device__ __forceinline__ double m_log(double x) { return ln_f64(x); }
__device__ __forceinline__ float m_log(float x) { return logf(x); }
__device__ __forceinline__ double m_pow(double x, double y) { return pow(x, y); }
__device__ __forceinline__ float m_pow(float x, float y) { return powf(x, y); }
__device__ __forceinline__ double m_sqrt(double x) { return sqrt(x); }
__device__ __forceinline__ float m_sqrt(float x) { return sqrtf(x); }
__device__ __forceinline__ double m_sin(double x) { return sin(x); }
__device__ __forceinline__ float m_sin(float x) { return sinf(x); }
__device__ __forceinline__ double m_cos(double x) { return cos(x); }
__device__ __forceinline__ float m_cos(float x) { return cosf(x); }
__device__ __forceinline__ double m_floor(double x) { return floor(x); }
__device__ __forceinline__ float m_floor(float x) { return floorf(x); }
__device__ __forceinline__ double m_atan2(double y, double x) { return atan2(y, x); }
__device__ __forceinline__ float m_atan2(float y, float x) { return atan2f(y, x); }
__device__ __forceinline__ double m_fmod(double x, double y) { return fmod(x, y); }
__device__ __forceinline__ float m_fmod(float x, float y) { return fmodf(x, y); }

// Reciprocals: v_rcp_f32 (1 ulp) for FP32; v_rcp_f64 refined by two Newton
// steps for FP64 (about 1 ulp).  a * recip(b) replaces the long
// correctly-rounded division sequences on the rate path.
__device__ __forceinline__ float recip(float b) { return __builtin_amdgcn_rcpf(b); }
__device__ __forceinline__ double recip(double b) {
    double r = __builtin_amdgcn_rcp(b);
    r = fma(fma(-b, r, 1.0), r, r);
    r = fma(fma(-b, r, 1.0), r, r);
    return r;
}

// Powers on the rate path: x >= 0 (a rate-curve base, 1 - exp(-0.03 WSV),
// or a wind speed) and y a positive fuel constant below 5, as exp(y ln x).
// A relative error of about one ulp in ln x becomes an absolute error of
// |y ln x| ulp in the exponent, so the result keeps a relative error of a
// few ulp for these bases, at a third of the instructions of the general
// pow() (which rounds exactly and handles every special case).  FP32 uses
// the hardware base-2 logarithm and exponential.  x = 0 gives 0.
__device__ __forceinline__ double rate_pow(double x, double y) { return exp(y * ln_f64(x)); }
__device__ __forceinline__ float rate_pow(float x, float y) { return exp2f(y * log2f(x)); }

// cos(2 pi u) for the Box-Muller draw, without a general argument reduction.
__device__ __forceinline__ double cos_2pi(double u) { return cospi(2.0 * u); }
__device__ __forceinline__ float cos_2pi(float u) { return cospif(2.0f * u); }

// ln(1 - x) for 0 <= x <= 0.99 in FP32 from one logarithm: with u = 1 - x
// rounded, ln(u) x / (1 - u) corrects the rounding of u (the log1p form of
// Goldberg, 1991; 1 - u is exact here), so a small x keeps its full
// relative precision.
__device__ __forceinline__ float log_1m(float x) {
    const float u = 1.0f - x;
    if (u == 1.0f) return -x;
    return logf(u) * (x * __builtin_amdgcn_rcpf(1.0f - u));
}

template <typename R> struct Const;
template <> struct Const<double> { static constexpr double pi = 3.14159265358979323846; };
template <> struct Const<float> { static constexpr float pi = 3.14159265358979323846f; };

// --------------------------------------------------------------- Philox
// Philox4x32-10 block function (Salmon et al., SC'11): ten rounds of two
// 32x32->64 multiplies, key bumped by the Weyl constants between rounds.
// Each product is formed once in 64 bits (one v_mad_u64_u32 instead of a
// low and a high multiply).
__device__ __forceinline__ uint4 philox4x32_10(uint4 x, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * x.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * x.z;
        x = make_uint4((uint32_t)(p1 >> 32) ^ x.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ x.w ^ k1,
                       (uint32_t)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return x;
}

// Counter layout shared by every random draw: (cell, period, rep, tag).
// Tags: 0 ROS noise, 1-2 rounding uniforms for axes 0-3 / 4-7,
// 3 ignition cell, 4 weather scenario (per-rep draws use cell = period = ~0).
__device__ __forceinline__ uint4 draw(uint64_t seed, uint32_t cell, uint32_t period, uint32_t rep,
                                      uint32_t tag) {
    return philox4x32_10(make_uint4(cell, period, rep, tag), (uint32_t)seed, (uint32_t)(seed >> 32));
}

// 24-bit uniform in [0, 1) from the high bits of a 32-bit word (exact in float).
template <typename R>
__device__ __forceinline__ R unit24(uint32_t x) {
    return (R)(x >> 8) * (R)(1.0 / 16777216.0);
}

// ------------------------------------------------------- weather terms
// Per (scenario, period) quantities that do not depend on the cell; kept in
// a table computed once per weather upload.  Layout of one row:
//   [0] f(F)   [1] ISZ = 0.208 f(F)   [2] WS sin(WAZ)   [3] WS cos(WAZ)
//   [4 + f] BUI effect of fuel f      [23 + f] 1 - exp(-b_f ISZ) of pure fuel f
//   [42 + f] surface fuel consumption of fuel f

template <typename R>
struct CoefR {
    R a, b, c, q, bui0;
};

// Rate of spread of one unmixed fuel: a (1 - exp(-b ISI))^c.
template <typename R>
__device__ __forceinline__ R rsi_pure(const CoefR<R>& k, R isi) {
    return k.a * rate_pow(-m_expm1(-k.b * isi), k.c);
}

// ----------------------------------------------------------- cell rates
__device__ __forceinline__ int rec_fuel(uint32_t info) { return (int)(info & 0xFFu); }
__device__ __forceinline__ uint32_t rec_nbmask(uint32_t info) { return (info >> 8) & 0xFFu; }
__device__ __forceinline__ int rec_gx(uint32_t g) { return (int)(int16_t)(g & 0xFFFFu); }
__device__ __forceinline__ int rec_gn(uint32_t g) { return (int)(int16_t)(g >> 16); }

// Landscape-wide constants of the mixed, grass and crowning fuels.
template <typename R>
struct LandR {
    R pc_w;    // percent conifer / 100 (M-1, M-2)
    R cf;      // grass curing factor (O-1a, O-1b)
    R cell_m;  // cell width, metres
    R pdf_w;   // percent dead fir / 100 (M-3, M-4)
    R fme_r;   // C-6 foliar moisture effect / its average 0.778
    const R* csi;   // critical surface intensity for crowning per fuel, kW/m
};

__device__ __forceinline__ bool is_grass(int f) { return f == kO1a || f == kO1b; }
__device__ __forceinline__ bool is_mix_pc(int f) { return f == kM1 || f == kM2; }
__device__ __forceinline__ bool is_mix_pdf(int f) { return f == kM3 || f == kM4; }

template <typename R>
__device__ __forceinline__ R rsi_fuel(const CoefR<R>* coef, int f, R isi, const LandR<R>& L) {
    // Mixedwoods blend a conifer curve with D-1: M-1/M-2 the C-2 curve by
    // percent conifer, M-3/M-4 their dead-fir curve by percent dead fir
    // (M-2 and M-4 take 0.2 of D-1).  Every lane evaluates its own (or the
    // C-2) curve, and the D-1 curve only runs when some lane of the wave is
    // a mixedwood.
    const bool mix_pc = is_mix_pc(f), mixed = mix_pc || is_mix_pdf(f);
    R r = rsi_pure(coef[mix_pc ? (int)kC2 : f], isi);
    if (__any(mixed)) {
        const R d1 = rsi_pure(coef[kD1], isi);
        if (mixed) {
            const R w = mix_pc ? L.pc_w : L.pdf_w;
            const R wd1 = (f == kM2 || f == kM4) ? (R)0.2 * ((R)1 - w) : ((R)1 - w);
            r = w * r + wd1 * d1;
        }
    }
    return is_grass(f) ? r * L.cf : r;
}

// Slope-equivalent wind speed (km/h).  The slope-adjusted zero-wind rate
// RSF = SF x RSZ inverted on the fuel's rate curve gives ISF = ln(1 - (RSF /
// (CF a))^(1/c)) / -b with the curve's 0.01 floor inside the logarithm.
// Because RSZ = CF a (1 - exp(-b ISZ))^c, (RSF / (CF a))^(1/c) is exactly
// SF^(1/c) (1 - exp(-b ISZ)): sfc/sfd carry SF^(1/c) per cell and the row
// carries 1 - exp(-b ISZ) per fuel.  Mixedwood takes the percent-conifer
// weighted ISF of the C-2 and D-1 curves.
__device__ __forceinline__ double isf_curve(const CoefR<double>& k, double sfc, double g) {
    double t = 1.0 - sfc * g;
    if (t < 0.01) t = 0.01;
    return -ln_f64(t) * recip(k.b);
}

// WSE of a slope-adjusted spread index.
__device__ __forceinline__ double wse_of_isf(double isf, const double* row) {
    const double ff = row[0], isz = row[1];
    double wse = ln_f64(isf * recip(isz)) * (1.0 / 0.05039);
    if (wse > 40.0) {
        wse = (isf < 0.999 * 2.496 * ff) ? 28.0 - ln_f64(1.0 - isf * recip(2.496 * ff)) * (1.0 / 0.0818) : 112.45;
    }
    return wse;
}

template <typename LAND>
__device__ __forceinline__ double slope_wind(const CoefR<double>* coef, int f, double sfc, double sfd,
                                          const double* row, const LAND& L) {
    // every lane inverts its own (or the C-2) curve; the D-1 curve only runs
    // when some lane of the wave is mixedwood
    const bool mix_pc = is_mix_pc(f), mixed = mix_pc || is_mix_pdf(f);
    const int fa = mix_pc ? (int)kC2 : f;
    double isf = isf_curve(coef[fa], sfc, row[kRowG + fa]);
    if (__any(mixed)) {
        const double d1 = isf_curve(coef[kD1], sfd, row[kRowG + kD1]);
        if (mixed) {
            const double w = mix_pc ? L.pc_w : L.pdf_w;
            isf = w * isf + (1.0 - w) * d1;
        }
    }
    return wse_of_isf(isf, row);
}

// The same in FP32 for the ordinary branch (WSE <= 40 km/h).  ln(1 - x) is
// taken with log1p accuracy (log_1m), so a gentle slope (x close to the zero-slope value)
// keeps full relative precision in ISF, and WSE = ln(ISF / ISZ) / 0.05039
// then carries an absolute error of a few 1e-6 km/h.  Near and above the
// 40 km/h branch point the caller switches to slope_wind in FP64, and so it
// does where ill is set: x = SF^(1/c) (1 - exp(-b ISZ)) above 0.8, where
// ln(1 - x) multiplies the relative error of x by x / (1 - x) and the 0.01
// floor of the curve is near (steep slopes in fast fuels).
constexpr float kIllX = 0.8f;

__device__ __forceinline__ float isf_curve32(const CoefR<float>& k, float x) {
    return -log_1m(x > 0.99f ? 0.99f : x) * recip(k.b);
}

__device__ __forceinline__ float slope_wind32(const CoefR<float>* coef, int f, float sfc, float sfd,
                                              const float* row, const LandR<float>& L, bool& ill) {
    const bool mix_pc = is_mix_pc(f), mixed = mix_pc || is_mix_pdf(f);
    const int fa = mix_pc ? (int)kC2 : f;
    const float xo = sfc * row[kRowG + fa];
    float isf = isf_curve32(coef[fa], xo);
    ill = xo > kIllX;
    if (__any(mixed)) {
        const float xd = sfd * row[kRowG + kD1];
        const float d1 = isf_curve32(coef[kD1], xd);
        if (mixed) {
            const float w = mix_pc ? L.pc_w : L.pdf_w;
            isf = w * isf + (1.0f - w) * d1;
            ill = ill || xd > kIllX;
        }
    }
    return m_log(isf * recip(row[1])) * (1.0f / 0.05039f);
}

// Head and back rates, length-to-breadth ratio and the effective wind
// vector (east, north components; its direction is the head direction).
template <typename R>
struct CellRates {
    R h, b, lb, lbm1, wx, wy, wsv;   // lbm1 = LB - 1, kept separately for accuracy
    R rss;                           // C-6: its surface head rate; other fuels: h
    // WSV lies within kEdgeWsv km/h of a speed where the model switches
    // form and its value jumps: f(W) at 40 km/h, grass LB at 1 km/h.  An
    // FP32 evaluation there may take the other branch than FP64.
    bool edge;
    // (rates of a quad or a lane) how much further than usual an FP32
    // evaluation may lie from FP64 here, 1 or more: grass whose wind and slope
    // nearly cancel, since the direction of what is left, and a rate in front
    // with it, carries their rounding, from WSV below 1 / kCancel of the wind;
    // C-6 that starts to crown (c6_rate's gain), from kC6Gain
    R widen;
};

constexpr float kEdgeWsv = 1e-3f;
constexpr float kCancel = 16.0f;
constexpr float kC6Gain = 6.0f;

// CellRates::widen of a cell's wind; (wx, wy): the weather's part of it.
template <typename R>
__device__ __forceinline__ R widen_wind(R wsv, bool grass, R wx, R wy) {
    const R w = (R)fabs(wx) + (R)fabs(wy), c = (R)kCancel * wsv;
    return grass && c < w ? w * recip(c) : (R)1;
}

// C-6 crown fire: the surface rate rss at spread index isi becomes rss +
// CFB (RSC - rss), RSC = 60 (1 - exp(-0.0497 ISI)) FME / 0.778 and CFB =
// 1 - exp(-0.23 (rss - RSO)) above the critical surface rate RSO = CSI /
// (300 SFC), 0 below it.
// gain: how many times over the rate follows a relative change of rss and RSO,
// where it crowns.
template <typename R>
__device__ __forceinline__ R c6_rate(R rss, R isi, R rso, R fme_r, R& gain) {
    const R cfb = rss > rso ? -m_expm1((R)-0.23 * (rss - rso)) : (R)0;
    const R lift = (R)60 * -m_expm1((R)-0.0497 * isi) * fme_r - rss;
    const R r = rss + cfb * lift;
    gain = rss > (R)0.9999 * rso ? (R)0.23 * ((R)1 - cfb) * (R)fabs(lift) * (rss + rso) * recip(r) : (R)0;
    return r;
}

// Unit vector pointing upslope (east, north) from the Horn numerators.
template <typename R>
__device__ __forceinline__ void upslope_unit(int gx, int gn, R& ux, R& uy) {
    const R ig = recip(m_sqrt((R)gx * (R)gx + (R)gn * (R)gn));
    ux = (R)gx * ig;
    uy = (R)gn * ig;
}
// The same of a cell's record, which holds the FP32 one.
__device__ __forceinline__ void upslope(const CellRec& rec, float& ux, float& uy) {
    ux = rec.ux;
    uy = rec.uy;
}
__device__ __forceinline__ void upslope(const CellRec& rec, double& ux, double& uy) {
    upslope_unit<double>(rec_gx(rec.grad), rec_gn(rec.grad), ux, uy);
}

// Everything is evaluated in R.  In FP32 the slope-equivalent wind switches
// to FP64 from 39 km/h up: inverting the rate curve near its asymptote (the
// WSE > 40 branch) turns a relative error of 1e-7 in ISF into ~1e-4 in WSE.
// It does so too where the inversion's argument is ill-conditioned
// (slope_wind32's ill).
// row64 is the FP64 weather row of the same (scenario, period).
template <typename R>
__device__ __forceinline__ CellRates<R> cell_rates(const CoefR<R>* coef, const CoefR<double>* coef64,
                                                const CellRec& rec, const R* row, const double* row64,
                                                const LandR<R>& L, const LandR<double>& L64) {
    const int f = rec_fuel(rec.info), gx = rec_gx(rec.grad), gn = rec_gn(rec.grad);
    R wx = row[2], wy = row[3];
    if ((gx | gn) != 0) {
        R wse = (R)0;
        bool need64 = true;
        if constexpr (sizeof(R) == 4) {
            bool ill;
            wse = slope_wind32(coef, f, (float)rec.sfc, (float)rec.sfd, row, L, ill);
            need64 = ill || !(wse < 39.0f);
        }
        if (need64) wse = (R)slope_wind(coef64, f, rec.sfc, rec.sfd, row64, L64);
        R ux, uy;
        upslope(rec, ux, uy);
        wx += wse * ux;
        wy += wse * uy;
    }
    const R wsv = m_sqrt(wx * wx + wy * wy);
    // exp(0.05039 WSV) is f(W) up to 40 km/h, and its reciprocal is the back
    // fire's wind function at every speed
    const R ew = m_exp((R)0.05039 * wsv);
    const R fw = (wsv <= (R)40) ? ew : (R)12 * -m_expm1((R)-0.0818 * (wsv - (R)28));
    const R be = row[kRowBE + f];
    const R isz = row[1];
    CellRates<R> out;
    const R isi_h = isz * fw, isi_b = isz * recip(ew);
    out.h = rsi_fuel(coef, f, isi_h, L) * be;
    out.b = rsi_fuel(coef, f, isi_b, L) * be;
    out.rss = out.h;
    if (__any(f == kC6)) {
        if (f == kC6) {
            const R sfc = row[kRowSFC + kC6];
            const R rso = sfc > (R)0 ? L.csi[kC6] * recip((R)300 * sfc) : (R)3.0e38;
            R gain;
            out.h = c6_rate<R>(out.rss, isi_h, rso, L.fme_r, gain);
            out.b = c6_rate<R>(out.b, isi_b, rso, L.fme_r, gain);
        }
    }
    // LB - 1: grass 1.1 WSV^0.464 - 1 (0 below 1 km/h), other fuels
    // 8.729 (1 - exp(-0.030 WSV))^2.155, as one power per lane
    const bool grass = is_grass(f);
    const R lbase = grass ? wsv : -m_expm1((R)-0.030 * wsv);
    const R lpow = rate_pow(lbase, grass ? (R)0.464 : (R)2.155);
    out.lbm1 = grass ? ((wsv >= (R)1) ? (R)1.1 * lpow - (R)1 : (R)0) : (R)8.729 * lpow;
    out.lb = (R)1 + out.lbm1;
    out.wx = wx;
    out.wy = wy;
    out.wsv = wsv;
    out.edge = fabs((double)wsv - 40.0) < (double)kEdgeWsv || (grass && fabs((double)wsv - 1.0) < (double)kEdgeWsv);
    out.widen = (R)1;
    return out;
}

// FBP slope factor of a cell from its Horn numerators: SF = exp(3.533
// (GS/100)^1.2) with GS = 100 |g| / (8 cs) percent, capped at 10 from 70 %.
__device__ __forceinline__ double slope_factor(int gx, int gn, double cell_m) {
    if ((gx | gn) == 0) return 1.0;
    const double gs = 100.0 * sqrt((double)gx * (double)gx + (double)gn * (double)gn) / (8.0 * cell_m);
    return (gs >= 70.0) ? 10.0 : exp(3.533 * pow(gs / 100.0, 1.2));
}


// Lognormal rate multiplier with mean 1 for (cell, period, rep).
template <typename R>
__device__ __forceinline__ R noise_mult(uint64_t seed, uint32_t cell, uint32_t period, uint32_t rep,
                                        R sigma) {
    if (sigma == (R)0) return (R)1;
    const uint4 x = draw(seed, cell, period, rep, 0u);
    const R u1 = ((R)(x.x >> 8) + (R)1) * (R)(1.0 / 16777216.0);
    const R u2 = unit24<R>(x.y);
    const R z = m_sqrt((R)-2 * m_log(u1)) * cos_2pi(u2);
    return m_exp(sigma * z - (R)0.5 * sigma * sigma);
}

// Directional rates along the 8 axes (eq. (1)): with a = (H+B)/2 (eq. (2)),
// e^2 = 1 - 1/LB^2 (eq. (4) with FROS = a/LB), cos(phi) the cosine between
// the axis and the head direction, the front half (cos phi > 0) spreads at
// a(1-e^2)/(1 - e cos phi) and the back half at a(1-e^2).  Each rate is then
// scaled by the noise multiplier mu.  e is formed from LB - 1 directly and
// the denominator is evaluated as (1 - e) + e (1 - cos phi) with
// 1 - e = LB^-2 / (1 + e) and
// 1 - cos phi = |w/|w| - u|^2 / 2, which avoids the cancellation of
// 1 - e cos phi near the head direction when LB is large.
template <typename R>
__device__ __forceinline__ void axis_rates(const CellRates<R>& cr, R mu, R* x8) {
    const R a = (R)0.5 * (cr.h + cr.b);
    const R il = recip(cr.lb);
    const R il2 = il * il;
    const R base = a * il2;                           // a (1 - e^2)
    const R e = m_sqrt(cr.lbm1 * (cr.lbm1 + (R)2)) * il;   // sqrt(1 - 1/LB^2)
    const R one_m_e = il2 * recip((R)1 + e);
    const R inv_wsv = (cr.wsv > (R)0) ? recip(cr.wsv) : (R)0;
    const R cx = cr.wx * inv_wsv, cy = cr.wy * inv_wsv;   // unit head direction
    const R s = (R)0.70710678118654752440;
    const R ux[8] = {(R)1, s, (R)0, -s, (R)-1, -s, (R)0, s};
    const R uy[8] = {(R)0, s, (R)1, s, (R)0, -s, (R)-1, -s};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const R c = ux[k] * cx + uy[k] * cy;
        R r = base;
        if (c > (R)0) {
            const R dx = cx - ux[k], dy = cy - uy[k];
            r = base * recip(one_m_e + e * ((R)0.5 * (dx * dx + dy * dy)));
        }
        x8[k] = mu * r;
    }
}

// The same rates floored to integer m/min after adding u_k: 1/2, or the
// 24-bit uniforms of the words ua (axes 0-3) and ub (axes 4-7).
template <typename R>
__device__ __forceinline__ void axis_rates_q(const CellRates<R>& cr, R mu, bool stochastic, uint4 ua, uint4 ub,
                                             int32_t* q) {
    const R a = (R)0.5 * (cr.h + cr.b);
    const R il = recip(cr.lb);
    const R il2 = il * il;
    const R base = a * il2;
    const R e = m_sqrt(cr.lbm1 * (cr.lbm1 + (R)2)) * il;
    const R one_m_e = il2 * recip((R)1 + e);
    const R inv_wsv = (cr.wsv > (R)0) ? recip(cr.wsv) : (R)0;
    const R cx = cr.wx * inv_wsv, cy = cr.wy * inv_wsv;
    const R s = (R)0.70710678118654752440;
    const R ux[8] = {(R)1, s, (R)0, -s, (R)-1, -s, (R)0, s};
    const R uy[8] = {(R)0, s, (R)1, s, (R)0, -s, (R)-1, -s};
    const uint32_t w[8] = {ua.x, ua.y, ua.z, ua.w, ub.x, ub.y, ub.z, ub.w};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const R c = ux[k] * cx + uy[k] * cy;
        R r = base;
        if (c > (R)0) {
            const R dx = cx - ux[k], dy = cy - uy[k];
            r = base * recip(one_m_e + e * ((R)0.5 * (dx * dx + dy * dy)));
        }
        const R u = stochastic ? unit24<R>(w[k]) : (R)0.5;
        const R v = m_floor(mu * r + u);
        q[k] = (v < (R)1073741824) ? (int32_t)v : 1073741824;
    }
}

}  // namespace c2f

namespace c2f {

// FBP coefficient tables in each translation unit's constant memory.
static __constant__ CoefR<double> kCoef64[kNumFuels] = {C2F_FUEL_ROWS};
static __constant__ CoefR<float> kCoef32[kNumFuels] = {C2F_FUEL_ROWS};

template <typename R> __device__ __forceinline__ const CoefR<R>* coef_table();
template <> __device__ __forceinline__ const CoefR<double>* coef_table<double>() { return kCoef64; }
template <> __device__ __forceinline__ const CoefR<float>* coef_table<float>() { return kCoef32; }

template <typename R> __device__ __forceinline__ LandR<R> land_consts(const LandDev* L);
template <> __device__ __forceinline__ LandR<double> land_consts<double>(const LandDev* L) {
    return LandR<double>{L->pc_w64, L->cf64, L->cell_m64, L->pdf_w64, L->fme_r64, L->csi64};
}
template <> __device__ __forceinline__ LandR<float> land_consts<float>(const LandDev* L) {
    return LandR<float>{L->pc_w32, L->cf32, L->cell_m32, L->pdf_w32, L->fme_r32, L->csi32};
}

// Crown base height and crown fuel load per fuel.
static __constant__ CrownCoef kCrown[kNumFuels] = {C2F_CROWN_ROWS};

// Head fire intensity (kW/m) of a cell from its rates, before the noise
// multiplier: 300 TFC ROS with TFC = SFC + CFL CFB, the crown fraction
// burned CFB = 1 - exp(-0.23 (S - RSO)) above the critical surface rate RSO
// = CSI / (300 SFC) (S the head rate, the surface rate for C-6; 0 for fuels
// that do not crown).  *cfb (may be NULL) receives CFB.
// *steep (may be NULL): the fuel starts to crown and TFC follows a relative
// change of S or RSO more than kHfiGain times over.
constexpr float kHfiGain = 64.0f;
template <typename R, typename LAND>
__device__ __forceinline__ R head_intensity(const CellRates<R>& cr, int f, const R* row, const LAND& L,
                                            R* cfb_out, bool* steep = nullptr) {
    R sfc = row[kRowSFC + f];
    if (is_mix_pc(f)) sfc = L.pc_w * row[kRowSFC + kC2] + ((R)1 - L.pc_w) * row[kRowSFC + kD1];
    const R cfl = (R)kCrown[f].cfl;
    R cfb = (R)0;
    if (steep) *steep = false;
    if (cfl > (R)0 && sfc > (R)0) {
        const R rso = L.csi[f] * recip((R)300 * sfc);
        if (cr.rss > rso) cfb = -m_expm1((R)-0.23 * (cr.rss - rso));
        if (steep)
            *steep = cr.rss > (R)0.9999 * rso &&
                     (R)0.23 * ((R)1 - cfb) * cfl * (cr.rss + rso) > (R)kHfiGain * (sfc + cfb * cfl);
    }
    if (cfb_out) *cfb_out = cfb;
    return (R)300 * (sfc + cfb * cfl) * cr.h;
}

// What the evaluation of one cell by one thread needs besides the cell:
// coefficient tables, landscape constants, the scenario's weather rows and the
// random stream.
template <typename R>
struct RateCtx {
    const CoefR<R>* coef;
    const CoefR<double>* coef64;
    LandR<R> L;
    LandR<double> L64;
    const R* rows;          // first row of the replication's scenario
    const double* rows64;
    uint64_t seed;
    R sigma;
    int rounding;
    uint32_t rep;
    float hfi_min;   // burn-out threshold on the head fire intensity, kW/m (0 = off)
};

// Weather scenario and ignition cell of replication `rep` of a job
// (Section 3.1, uncertainty sources (1) and (3)): a fixed scenario or
// (x S) >> 32 from Philox tag 4; a fixed cell, the burnable cell (x |B|) >> 32
// of the row-major burnable list from tag 3, the burnable cell nearest the
// centre, or a draw from the ignition map: with running weight sums C and
// total W, the first cell whose C exceeds floor(x W / 2^32).  ign = -1 when
// there is nothing to ignite.
__device__ __forceinline__ void rep_draws(const Job& job, uint32_t rep, int& scen, int& ign) {
    scen = job.scen_fixed;
    if (job.scen_mode == 1) {
        const uint4 x = draw(job.seed, 0xFFFFFFFFu, 0xFFFFFFFFu, rep, 4u);
        scen = (int)(((uint64_t)x.x * (uint64_t)job.n_scen) >> 32);
    }
    ign = -1;
    if (job.ign_mode == 0) {
        ign = job.ign_cell;
    } else if (job.ign_mode == 1) {
        const int nbn = job.land->n_burnable;
        if (nbn > 0) {
            const uint4 x = draw(job.seed, 0xFFFFFFFFu, 0xFFFFFFFFu, rep, 3u);
            ign = job.burnable[((uint64_t)x.x * (uint64_t)nbn) >> 32];
        }
    } else if (job.ign_mode == 2) {
        ign = job.land->centre_cell;
    } else if (job.ign_mode == 4) {
        ign = job.n_seeds > 0 ? job.seeds[0].x : -1;   // the earliest entry of the list
    } else if (job.ign_total > 0) {
        const uint4 x = draw(job.seed, 0xFFFFFFFFu, 0xFFFFFFFFu, rep, 3u);
        const uint64_t W = job.ign_total;
        // floor(x W / 2^32) without overflow: W < 2^63
        const uint64_t t = (uint64_t)x.x * (W >> 32) + (((uint64_t)x.x * (W & 0xFFFFFFFFull)) >> 32);
        // first index with C[i] > t (C is non-decreasing, C[n-1] = W > t)
        int64_t lo = 0, hi = (int64_t)job.rows * job.cols - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (job.ign_cdf[mid] > t) hi = mid;
            else lo = mid + 1;
        }
        ign = (int)lo;
    }
}

// Does period p lie inside the daily burning window (the first burn_hours
// hours of every day from the start of the run; assumption A5)?  The
// period length divides 60 minutes whenever a window is set, so a period
// lies wholly inside or outside it.
__device__ __forceinline__ bool burning_period(const Job& job, int p) {
    if (job.burn_hours <= 0) return true;
    return (int)(((int64_t)p * job.period_min) % 1440) < job.burn_hours * 60;
}

// Does the ignition-point list hold an entry of period p?
__device__ __forceinline__ bool seeds_at(const Job& job, int p) {
    for (int k = 0; k < job.n_seeds; ++k)
        if (job.seeds[k].y == p) return true;
    return false;
}

// Integer axis rates (m/min) of a cell in a period: eq. (1) rates scaled by
// the noise multiplier, then floor(x + u) with u = 1/2 or a Philox uniform.
// Returns true when the cell burns out on its head fire intensity (A5 (iv)):
// an intensity threshold is set and the intensity, with the noise
// multiplier on the rate, is below it.
template <typename R>
__device__ __forceinline__ bool axis_q(const RateCtx<R>& X, const CellRec& rec, uint32_t cell, uint32_t period,
                                       int32_t* q) {
    const size_t ro = (size_t)period * kRowLen;
    const CellRates<R> cr = cell_rates<R>(X.coef, X.coef64, rec, X.rows + ro, X.rows64 + ro, X.L, X.L64);
    const R mu = noise_mult<R>(X.seed, cell, period, X.rep, X.sigma);
    uint4 ua = make_uint4(0u, 0u, 0u, 0u), ub = ua;
    if (X.rounding != 0) {
        ua = draw(X.seed, cell, period, X.rep, 1u);
        ub = draw(X.seed, cell, period, X.rep, 2u);
    }
    axis_rates_q<R>(cr, mu, X.rounding != 0, ua, ub, q);
    if (X.hfi_min > 0.f) {
        const R hfi = head_intensity(cr, rec_fuel(rec.info), X.rows + ro, X.L, (R*)nullptr) * mu;
        return !((double)hfi >= (double)X.hfi_min);
    }
    return false;
}

// Integer rates of an FP64 result from an FP32 evaluation where that is
// exact: where x32 + u lies more than kMixMargin max(1, x32), times
// CellRates::widen, from an integer, floor(x64 + u) is the same integer; and
// where the FP32 intensity lies more than kMixMarginH of the threshold, widened
// likewise, from it, the burn-out test agrees.  Every other cell, and one whose
// CellRates::edge or head_intensity's steep is set, takes the FP64 evaluation.
//
// The FP32 evaluation reads the FP64 weather row rounded once.  (A row formed in
// FP32 turned the wind by up to 3e-5 degrees, which a wind against a steep slope
// magnifies, and lost the digits of C-1's consumption at low FFMC.)  Largest
// differences from FP64, over widen, that a search found which climbs towards
// them (6e10 cells: 18 fuels, slopes of up to 75 %, FFMC 40-101, BUI up to 300,
// wind up to 400 km/h, seven sets of curing, foliar moisture from 1 to 300 %,
// percent conifer and dead fir): 1.06e-5 of max(1, x) in grass, 9.6e-6 in C-6,
// 3.9e-6 in the others; intensities 4.4e-5 relative.  With the library's functions
// in place of MathFast's 9.5e-6, 9.1e-6, 3.8e-6 and 5.1e-5; with FP32 rows and
// without widen and steep 1.0e-4, 1.7e-4, 1.9e-5 and 2.9e-2.  The margins are
// 2.8 and 4.5 times the first figures.
//
// The noise multiplier exp(sigma z - sigma^2 / 2) adds to that: z may be off by
// 4.9e-7 of its radius and 5.77 times 1.3e-7 of its cosine, and the exponent is
// rounded three times at up to 5.77 sigma where the multiplier is not tiny (and
// where it is, so is the rate).  That is below 2.3e-6 sigma; 1.4e-6 sigma was the
// most over 3.4e8 draws at each of six sigma from 0.15 to 8 (1.3e-6 with the
// library's functions).  Both margins grow by kMixSigma sigma.
constexpr double kMixMargin = 3e-5;
constexpr double kMixMarginH = 2e-4;
constexpr double kMixSigma = 3e-6;

// Head rate times the noise multiplier: the receiving cell's ignition test.
template <typename R>
__device__ __forceinline__ R head_rate(const RateCtx<R>& X, const CellRec& rec, uint32_t cell, uint32_t period) {
    const size_t ro = (size_t)period * kRowLen;
    const CellRates<R> cr = cell_rates<R>(X.coef, X.coef64, rec, X.rows + ro, X.rows64 + ro, X.L, X.L64);
    return cr.h * noise_mult<R>(X.seed, cell, period, X.rep, X.sigma);
}

// ---------------------------------------------------------- four lanes a cell
// The propagation kernel gives a cell to a quad: four neighbouring lanes,
// lane k of which takes the opposite axes k and k + 4.  What the axes share
// is split by role instead of being repeated: the rate curves a (1 -
// exp(-b x))^c of the head and the back fire and the length-to-breadth curve
// of the same form run side by side in lanes 0, 1 and 2, the two slope
// inversions of a mixedwood in lanes 0 and 1, and the random blocks of tags
// 0, 1 and 2 in lanes 0, 1 and 2.  Every value is formed by the operations of
// cell_rates, noise_mult and axis_rates, in their order, so the results are
// the same bits.  All four lanes of a quad are active together and agree on
// every branch.

template <int CTRL>
__device__ __forceinline__ uint32_t quad_perm(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// x of lane K of the quad.
template <int K>
__device__ __forceinline__ uint32_t quad_lane(uint32_t x) { return quad_perm<K * 0x55>(x); }
template <int K>
__device__ __forceinline__ float quad_lane(float x) { return __uint_as_float(quad_lane<K>(__float_as_uint(x))); }
template <int K>
__device__ __forceinline__ double quad_lane(double x) {
    return __hiloint2double((int)quad_lane<K>((uint32_t)__double2hiint(x)),
                            (int)quad_lane<K>((uint32_t)__double2loint(x)));
}
// Bitwise or over the quad, in every lane.
__device__ __forceinline__ uint32_t quad_or(uint32_t x) {
    x |= quad_perm<0xB1>(x);          // lane ^ 1
    return x | quad_perm<0x4E>(x);    // lane ^ 2
}

// Entries of a quad's coefficient tables: the fuels, then the length-to-
// breadth curves 8.729 (1 - exp(-0.030 WSV))^2.155 and (grass, on the wind
// speed itself) 1.1 WSV^0.464.
constexpr int kCurveLB = kNumFuels;
constexpr int kNumCurves = kNumFuels + 2;

template <typename R>
__device__ __forceinline__ CoefR<R> curve_entry(int i) {
    if (i < kNumFuels) return coef_table<R>()[i];
    return i == kCurveLB ? CoefR<R>{(R)8.729, (R)0.030, (R)2.155, (R)0, (R)0}
                         : CoefR<R>{(R)1.1, (R)0, (R)0.464, (R)0, (R)0};
}

// Landscape constants in LDS (LandR's fields, with the intensities beside them).
template <typename R>
struct LandLds {
    R pc_w, cf, pdf_w, fme_r;
    R csi[kNumFuels];
};
template <typename R> __device__ __forceinline__ void load_land(const LandDev* D, LandLds<R>& L, int f);
template <> __device__ __forceinline__ void load_land<double>(const LandDev* D, LandLds<double>& L, int f) {
    L.csi[f] = D->csi64[f];
    if (f == 0) {
        L.pc_w = D->pc_w64;
        L.cf = D->cf64;
        L.pdf_w = D->pdf_w64;
        L.fme_r = D->fme_r64;
    }
}
template <> __device__ __forceinline__ void load_land<float>(const LandDev* D, LandLds<float>& L, int f) {
    L.csi[f] = D->csi32[f];
    if (f == 0) {
        L.pc_w = D->pc_w32;
        L.cf = D->cf32;
        L.pdf_w = D->pdf_w32;
        L.fme_r = D->fme_r32;
    }
}

// What the evaluations of one replication and period read from LDS: the
// curves, the period's weather rows and the landscape's constants in one
// precision.
template <typename R>
struct EvalLds {
    CoefR<R> coef[kNumCurves];
    R row[kRowLen];
    LandLds<R> L;
};
// The rest, uniform over the work group.
struct EvalRep {
    uint64_t seed;
    uint32_t rep;
    int32_t rounding;
    float sigma, hfi_min;
    float margin;   // mix_margin(sigma)
};
// The rounding margin of a replication, the same in every lane: in a scalar
// register (formed in every pass it made groups of 256 threads spill).
__device__ __forceinline__ float mix_margin(float sigma) {
    const float m = fmaf((float)kMixSigma, sigma, (float)kMixMargin + 2e-7f);
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(m)));
}
// That of the head fire intensity.
__device__ __forceinline__ double intensity_margin(const EvalRep& e) {
    return (double)e.margin + (kMixMarginH - kMixMargin);
}

// The functions an evaluation uses: those of cell_rates and noise_mult, or
// (FP32 only) the hardware's base-2 logarithm and exponential, square root and
// cosine of a fraction of a turn.
template <typename R>
struct MathOf {
    static __device__ __forceinline__ R exp_wind(R x) { return m_exp(x); }
    static __device__ __forceinline__ R exp_noise(R x) { return m_exp(x); }
    static __device__ __forceinline__ R one_minus_exp(R y) { return -m_expm1(-y); }   // 1 - exp(-y)
    static __device__ __forceinline__ R log(R x) { return m_log(x); }
    static __device__ __forceinline__ R sqrt(R x) { return m_sqrt(x); }
    static __device__ __forceinline__ R cos_turn(R u) { return cos_2pi(u); }
    static __device__ __forceinline__ R pow(R x, R y) { return rate_pow(x, y); }
    static __device__ __forceinline__ R log1m(R x) { return log_1m(x); }
};
// Largest errors over grids of 2^24 arguments, and those of the library's
// FP32 functions: ln of the noise draw's u1, as the radius sqrt(-2 ln u1),
// 4.9e-7 absolute (5.3e-7); the cosine 1.3e-7 absolute (0.5e-7); ln over
// [1, 11] 1.6e-7 relative (1.6e-7); ln(1 - x) over (0, 0.99] 2.6e-7 relative
// (2.6e-7); the square root 0.9e-7 relative; exp_wind over winds of 0 to 150
// km/h 1.4e-7 relative (0.8e-7; 5.0e-7 without the correction of the
// product's rounding); exp_noise over [-10, 20] 1.3e-7 relative for each unit of
// max(1, |x|) (0.8e-7); one_minus_exp over [1e-6, 40] 2.8e-7 relative (0.9e-7);
// pow over bases of 1e-5 to 1 and the rate curves' exponents 2.3e-6 relative
// (2.3e-6), 3.0e-7 (3.0e-7) over grass' winds.
struct MathFast {
    static constexpr float kLog2e = 1.44269504088896340736f, kLog2eLow = 1.925963033e-8f;
    static constexpr float kLn2 = 0.69314718055994530942f;
    static __device__ __forceinline__ float exp_wind(float x) {
        const float p = x * kLog2e;
        const float d = fmaf(x, kLog2eLow, fmaf(x, kLog2e, -p));   // what p lost
        const float y = __builtin_amdgcn_exp2f(p);
        return fmaf(y * d, kLn2, y);
    }
    static __device__ __forceinline__ float exp_noise(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }
    // 1 - exp(-y), y >= 0: with u = exp(-y) rounded, 1 - u where u < 1/2, and
    // above it (1 - u) y / -ln(u), which corrects the rounding of u (Kahan's
    // form; Higham, Accuracy and Stability of Numerical Algorithms, 1.14.1)
    static __device__ __forceinline__ float one_minus_exp(float y) {
        const float p = y * -kLog2e;
        const float u = __builtin_amdgcn_exp2f(p);
        const float d = 1.0f - u;
        const float r = d * (p * __builtin_amdgcn_rcpf(__builtin_amdgcn_logf(u)));
        return u < 0.5f ? d : (u == 1.0f ? y : r);
    }
    static __device__ __forceinline__ float log(float x) { return __builtin_amdgcn_logf(x) * kLn2; }
    static __device__ __forceinline__ float sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
    static __device__ __forceinline__ float cos_turn(float u) { return __builtin_amdgcn_cosf(u); }
    static __device__ __forceinline__ float pow(float x, float y) {
        return __builtin_amdgcn_exp2f(y * __builtin_amdgcn_logf(x));
    }
    static __device__ __forceinline__ float log1m(float x) {
        const float u = 1.0f - x;
        const float r = log(u) * (x * __builtin_amdgcn_rcpf(1.0f - u));
        return u == 1.0f ? -x : r;
    }
};

// FP64 slope wind of an FP32 evaluation near the inversion's asymptote.
// Rare, and kept out of line: inlined, its constants and temporaries take
// registers from the FP32 evaluation around it.
static inline __device__ __attribute__((noinline)) float slope_wind_rare(const EvalLds<double>* x, int f, double sfc,
                                                                  double sfd) {
    return (float)slope_wind(x->coef, f, sfc, sfd, x->row, x->L);
}

template <typename R, typename M>
__device__ __forceinline__ R quad_slope_wind(const EvalLds<R>& x, const EvalLds<double>& x64, const CellRec& rec,
                                             int f, int role) {
    const bool mix_pc = is_mix_pc(f), mixed = mix_pc || is_mix_pdf(f);
    const int fs = role == 1 ? (int)kD1 : mix_pc ? (int)kC2 : f;
    const R g = x.row[kRowG + fs], b = x.coef[fs].b;
    if constexpr (sizeof(R) == 4) {
        const float t = (role == 1 ? (float)rec.sfd : (float)rec.sfc) * g;
        const float l = -M::log1m(t > 0.99f ? 0.99f : t) * recip(b);
        const uint32_t over = t > kIllX ? 1u : 0u;
        const float own = quad_lane<0>(l), d1 = quad_lane<1>(l);
        const uint32_t o0 = quad_lane<0>(over), o1 = quad_lane<1>(over);
        float isf = own;
        if (mixed) {
            const float w = mix_pc ? x.L.pc_w : x.L.pdf_w;
            isf = w * own + (1.0f - w) * d1;
        }
        const float wse = M::log(isf * recip(x.row[1])) * (1.0f / 0.05039f);
        if (o0 != 0u || (mixed && o1 != 0u) || !(wse < 39.0f)) return slope_wind_rare(&x64, f, rec.sfc, rec.sfd);
        return wse;
    } else {
        double t = 1.0 - (role == 1 ? rec.sfd : rec.sfc) * g;
        if (t < 0.01) t = 0.01;
        const double l = -ln_f64(t) * recip(b);
        const double own = quad_lane<0>(l), d1 = quad_lane<1>(l);
        double isf = own;
        if (mixed) {
            const double w = mix_pc ? x.L.pc_w : x.L.pdf_w;
            isf = w * own + (1.0 - w) * d1;
        }
        return wse_of_isf(isf, x.row);
    }
}

// cell_rates of a quad's cell; `role` is the lane's number in the quad.
template <typename R, typename M>
__device__ __forceinline__ CellRates<R> quad_cell_rates(const EvalLds<R>& x, const EvalLds<double>& x64,
                                                        const CellRec& rec, int role) {
    const int f = rec_fuel(rec.info);
    R wx = x.row[2], wy = x.row[3];
    if (rec.grad != 0u) {
        const R wse = quad_slope_wind<R, M>(x, x64, rec, f, role);
        R ux, uy;
        upslope(rec, ux, uy);
        wx += wse * ux;
        wy += wse * uy;
    }
    const R wsv = M::sqrt(wx * wx + wy * wy);
    const R ew = M::exp_wind((R)0.05039 * wsv);
    R fw = ew;
    if (!(wsv <= (R)40)) fw = (R)12 * M::one_minus_exp((R)0.0818 * (wsv - (R)28));
    const R isz = x.row[1];
    // lane 0: the head curve, lane 1: the back curve, lane 2: LB (lane 3
    // repeats the head curve)
    const bool grass = is_grass(f), mix_pc = is_mix_pc(f), mixed = mix_pc || is_mix_pdf(f);
    const R rew = recip(ew);
    const R isi = isz * (role == 1 ? rew : fw);
    const CoefR<R>& k = x.coef[role == 2 ? kCurveLB + (int)grass : mix_pc ? (int)kC2 : f];
    R base = M::one_minus_exp(k.b * (role == 2 ? wsv : isi));
    base = (role == 2 && grass) ? wsv : base;
    const R curve = k.a * M::pow(base, k.c);
    R r = curve;
    if (__any(mixed)) {
        const R d1 = x.coef[kD1].a * M::pow(M::one_minus_exp(x.coef[kD1].b * isi), x.coef[kD1].c);
        if (mixed) {
            const R w = mix_pc ? x.L.pc_w : x.L.pdf_w;
            const R wd1 = (f == kM2 || f == kM4) ? (R)0.2 * ((R)1 - w) : ((R)1 - w);
            r = w * r + wd1 * d1;
        }
    }
    if (grass) r = r * x.L.cf;
    r = r * x.row[kRowBE + f];
    CellRates<R> out;
    out.rss = quad_lane<0>(r);
    out.widen = widen_wind<R>(wsv, grass, x.row[2], x.row[3]);
    if (__any(f == kC6)) {
        if (f == kC6) {
            const R sfc = x.row[kRowSFC + kC6];
            const R rso = sfc > (R)0 ? x.L.csi[kC6] * recip((R)300 * sfc) : (R)3.0e38;
            R gain;
            r = c6_rate<R>(r, isi, rso, x.L.fme_r, gain);
            out.widen = (R)fmax((R)1, (R)fmax(quad_lane<0>(gain), quad_lane<1>(gain)) * (R)(1.0f / kC6Gain));
        }
    }
    out.h = quad_lane<0>(r);
    out.b = quad_lane<1>(r);
    const R lb = quad_lane<2>(curve);
    out.lbm1 = grass ? ((wsv >= (R)1) ? lb - (R)1 : (R)0) : lb;
    out.lb = (R)1 + out.lbm1;
    out.wx = wx;
    out.wy = wy;
    out.wsv = wsv;
    // wsv - 40 and wsv - 1 are exact wherever they are small
    out.edge = (R)fabs(wsv - (R)40) < (R)kEdgeWsv || (grass && (R)fabs(wsv - (R)1) < (R)kEdgeWsv);
    return out;
}

// The random words of a quad's cell: u1, u2 of the noise draw (tag 0) and,
// with stochastic rounding, the words of the lane's two axes (tags 1, 2).
struct QuadWords {
    uint32_t n1, n2, wa, wb;
};
__device__ __forceinline__ QuadWords quad_words(uint64_t seed, uint32_t cell, uint32_t period, uint32_t rep,
                                                int role) {
    // the key schedule is kept inside the pass: hoisted out of the loops its
    // twenty words take scalar registers from everything else
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    asm volatile("" : "+s"(k0), "+s"(k1));
    const uint4 x = philox4x32_10(make_uint4(cell, period, rep, (uint32_t)role), k0, k1);
    QuadWords o;
    o.n1 = quad_lane<0>(x.x);
    o.n2 = quad_lane<0>(x.y);
    // the exchanges come before the selection: a lane reads its neighbours
    // while all four are active
    const uint32_t a0 = quad_lane<1>(x.x), a1 = quad_lane<1>(x.y), a2 = quad_lane<1>(x.z), a3 = quad_lane<1>(x.w);
    const uint32_t b0 = quad_lane<2>(x.x), b1 = quad_lane<2>(x.y), b2 = quad_lane<2>(x.z), b3 = quad_lane<2>(x.w);
    const uint32_t a01 = (role & 1) ? a1 : a0, a23 = (role & 1) ? a3 : a2;
    const uint32_t b01 = (role & 1) ? b1 : b0, b23 = (role & 1) ? b3 : b2;
    o.wa = (role & 2) ? a23 : a01;
    o.wb = (role & 2) ? b23 : b01;
    return o;
}

// noise_mult from the draw's words.
template <typename R, typename M>
__device__ __forceinline__ R noise_of(uint32_t n1, uint32_t n2, R sigma) {
    const R u1 = ((R)(n1 >> 8) + (R)1) * (R)(1.0 / 16777216.0);
    const R u2 = unit24<R>(n2);
    const R z = M::sqrt((R)-2 * M::log(u1)) * M::cos_turn(u2);
    return M::exp_noise(sigma * z - (R)0.5 * sigma * sigma);
}

// The rates of axes `role` (xa) and `role` + 4 (xb).  The axes point opposite
// ways, so at most one of them lies in the front half.
template <typename R, typename M>
__device__ __forceinline__ void quad_axis_rates(const CellRates<R>& cr, R mu, int role, R& xa, R& xb) {
    const R a = (R)0.5 * (cr.h + cr.b);
    const R il = recip(cr.lb);
    const R il2 = il * il;
    const R base = a * il2;
    const R e = M::sqrt(cr.lbm1 * (cr.lbm1 + (R)2)) * il;
    const R one_m_e = il2 * recip((R)1 + e);
    const R inv_wsv = (cr.wsv > (R)0) ? recip(cr.wsv) : (R)0;
    const R cx = cr.wx * inv_wsv, cy = cr.wy * inv_wsv;
    const R s = (R)0.70710678118654752440;
    const R ux = role == 0 ? (R)1 : role == 1 ? s : role == 2 ? (R)0 : -s;
    const R uy = role == 0 ? (R)0 : role == 2 ? (R)1 : s;
    const R c = ux * cx + uy * cy;
    const bool fa = c > (R)0, fb = c < (R)0;
    const R dx = cx - (fb ? -ux : ux), dy = cy - (fb ? -uy : uy);
    const R front = base * recip(one_m_e + e * ((R)0.5 * (dx * dx + dy * dy)));
    xa = mu * (fa ? front : base);
    xb = mu * (fb ? front : base);
}

template <typename R>
__device__ __forceinline__ int32_t quantise(R x, R u) {
    const R v = m_floor(x + u);
    return (v < (R)1073741824) ? (int32_t)v : 1073741824;
}

// The FP64 evaluation of a quad whose FP32 one lies near a rounding boundary:
// about 0.1 % of evaluations, kept out of line as slope_wind_rare is.
struct QuadRates {
    int32_t qa, qb;
    uint32_t faint;
};
static inline __device__ __attribute__((noinline)) QuadRates quad_axis_q_rare(const EvalLds<double>* x, const EvalRep* e,
                                                                       uint32_t info, uint32_t grad, double sfc,
                                                                       double sfd, QuadWords w, int role) {
    CellRec rec;
    rec.info = info;
    rec.grad = grad;
    rec.ux = rec.uy = 0.f;   // the FP64 evaluation forms its own
    rec.sfc = sfc;
    rec.sfd = sfd;
    const CellRates<double> cr = quad_cell_rates<double, MathOf<double>>(*x, *x, rec, role);
    const double mu = e->sigma == 0.f ? 1.0 : noise_of<double, MathOf<double>>(w.n1, w.n2, (double)e->sigma);
    double xa, xb;
    quad_axis_rates<double, MathOf<double>>(cr, mu, role, xa, xb);
    QuadRates o;
    o.qa = quantise<double>(xa, e->rounding != 0 ? unit24<double>(w.wa) : 0.5);
    o.qb = quantise<double>(xb, e->rounding != 0 ? unit24<double>(w.wb) : 0.5);
    o.faint = 0u;
    if (e->hfi_min > 0.f) {
        const double hfi = head_intensity(cr, rec_fuel(rec.info), x->row, x->L, (double*)nullptr) * mu;
        o.faint = hfi >= (double)e->hfi_min ? 0u : 1u;
    }
    return o;
}

// floor(x + u) of an FP64 rate known in FP32, if x32 + u lies clear of an
// integer by the margin (sets exact = false if not).  The sum is formed in
// FP32: its rounding, below 6.0e-8 (x + 1), and that of the distance from the
// integer's middle widen kMixMargin by less than 2e-7 max(1, x).  Rates from
// 16500 m/min up never pass.
__device__ __forceinline__ int32_t quantise_mixed(float x, float u, float margin, bool& exact) {
    const float v = x + u;
    const float k = floorf(v);
    const float clear = fmaf(-margin, fmaxf(1.0f, x), 0.5f);
    exact = exact && fabsf((v - k) - 0.5f) < clear;
    return (int32_t)k;
}

// The random part of a quad's evaluation: its words, and in FP32 the noise
// multiplier.  It needs nothing of the cell's record, so the caller forms it
// while the record is on its way.
struct QuadDraws {
    QuadWords w;
    float mu;
};
template <bool MIXED>
__device__ __forceinline__ QuadDraws quad_draws(const EvalRep& e, uint32_t cell, uint32_t period, int role) {
    using M = typename std::conditional<MIXED, MathFast, MathOf<float>>::type;
    QuadDraws d{{0u, 0u, 0u, 0u}, 1.f};
    if (e.sigma != 0.f || e.rounding != 0) d.w = quad_words(e.seed, cell, period, e.rep, role);
    if (e.sigma != 0.f) d.mu = noise_of<float, M>(d.w.n1, d.w.n2, e.sigma);
    return d;
}

// axis_q of a quad's cell: FP32 rates (MIXED false), or the integer rates of
// an FP64 evaluation.
template <bool MIXED>
__device__ __forceinline__ bool quad_axis_q(const EvalLds<float>& x, const EvalLds<double>& x64, const EvalRep& e,
                                            const EvalRep* e_lds, const CellRec& rec, const QuadDraws& d, int role,
                                            int32_t& qa, int32_t& qb) {
    const QuadWords w = d.w;
    const float mu = d.mu;
    if constexpr (!MIXED) {
        const CellRates<float> cr = quad_cell_rates<float, MathOf<float>>(x, x64, rec, role);
        float xa, xb;
        quad_axis_rates<float, MathOf<float>>(cr, mu, role, xa, xb);
        qa = quantise<float>(xa, e.rounding != 0 ? unit24<float>(w.wa) : 0.5f);
        qb = quantise<float>(xb, e.rounding != 0 ? unit24<float>(w.wb) : 0.5f);
        if (e.hfi_min > 0.f) {
            const float hfi = head_intensity(cr, rec_fuel(rec.info), x.row, x.L, (float*)nullptr) * mu;
            return !((double)hfi >= (double)e.hfi_min);
        }
        return false;
    } else {
        const CellRates<float> cr = quad_cell_rates<float, MathFast>(x, x64, rec, role);
        float xa, xb;
        quad_axis_rates<float, MathFast>(cr, mu, role, xa, xb);
        bool exact = !cr.edge;
        const float margin = e.margin * cr.widen;
        qa = quantise_mixed(xa, e.rounding != 0 ? unit24<float>(w.wa) : 0.5f, margin, exact);
        qb = quantise_mixed(xb, e.rounding != 0 ? unit24<float>(w.wb) : 0.5f, margin, exact);
        bool faint = false;
        if (e.hfi_min > 0.f) {
            bool steep;
            const double hfi =
                (double)(head_intensity(cr, rec_fuel(rec.info), x.row, x.L, (float*)nullptr, &steep) * mu);
            const double hm = (double)e.hfi_min;
            exact = exact && !steep && fabs(hfi - hm) > intensity_margin(e) * (double)cr.widen * hm;
            faint = !(hfi >= hm);
        }
        // a NaN rate fails the comparison above and goes the FP64 way
        if (quad_or(exact ? 0u : 1u) == 0u) return faint;
        const QuadRates o = quad_axis_q_rare(&x64, e_lds, rec.info, rec.grad, rec.sfc, rec.sfd, w, role);
        qa = o.qa;
        qb = o.qb;
        return o.faint != 0u;
    }
}

// ------------------------------------------------------------ one lane a cell
// The same evaluation with a lane to each cell, for passes wide enough to
// fill 64 of them: the axes' shared part is then formed once a cell instead
// of four times.  The operations and their order are those of the quad, so
// the rates are the same bits.  A cell that needs FP64 anywhere (its slope
// wind, or its integer rates near a boundary) is only reported: a quad takes
// it instead, so that no call and none of the FP64 constants are here.
template <typename M>
__device__ __forceinline__ float curve32(const CoefR<float>& k, float y) {
    return k.a * M::pow(M::one_minus_exp(k.b * y), k.c);
}

template <typename M>
__device__ __forceinline__ CellRates<float> lane_cell_rates(const EvalLds<float>& x, const CellRec& rec, bool& plain) {
    const int f = rec_fuel(rec.info);
    const bool grass = is_grass(f), mix_pc = is_mix_pc(f), mixed = mix_pc || is_mix_pdf(f);
    const int fa = mix_pc ? (int)kC2 : f;
    const bool any_mixed = __any(mixed);
    plain = true;
    float wx = x.row[2], wy = x.row[3];
    if (rec.grad != 0u) {
        const float t = (float)rec.sfc * x.row[kRowG + fa];
        float isf = -M::log1m(t > 0.99f ? 0.99f : t) * recip(x.coef[fa].b);
        bool ill = t > kIllX;
        if (any_mixed) {
            if (mixed) {
                const float td = (float)rec.sfd * x.row[kRowG + kD1];
                const float d1 = -M::log1m(td > 0.99f ? 0.99f : td) * recip(x.coef[kD1].b);
                const float w = mix_pc ? x.L.pc_w : x.L.pdf_w;
                isf = w * isf + (1.0f - w) * d1;
                ill = ill || td > kIllX;
            }
        }
        const float wse = M::log(isf * recip(x.row[1])) * (1.0f / 0.05039f);
        plain = !ill && wse < 39.0f;
        wx += wse * rec.ux;
        wy += wse * rec.uy;
    }
    const float wsv = M::sqrt(wx * wx + wy * wy);
    const float ew = M::exp_wind(0.05039f * wsv);
    float fw = ew;
    if (!(wsv <= 40.0f)) fw = 12.0f * M::one_minus_exp(0.0818f * (wsv - 28.0f));
    const float isz = x.row[1], be = x.row[kRowBE + f];
    const float isi_h = isz * fw, isi_b = isz * recip(ew);
    float h = curve32<M>(x.coef[fa], isi_h), b = curve32<M>(x.coef[fa], isi_b);
    if (any_mixed) {
        if (mixed) {
            const float w = mix_pc ? x.L.pc_w : x.L.pdf_w;
            const float wd1 = (f == kM2 || f == kM4) ? 0.2f * (1.0f - w) : (1.0f - w);
            h = w * h + wd1 * curve32<M>(x.coef[kD1], isi_h);
            b = w * b + wd1 * curve32<M>(x.coef[kD1], isi_b);
        }
    }
    if (grass) {
        h = h * x.L.cf;
        b = b * x.L.cf;
    }
    h = h * be;
    b = b * be;
    CellRates<float> out;
    out.rss = h;
    out.widen = widen_wind<float>(wsv, grass, x.row[2], x.row[3]);
    if (f == kC6) {
        const float sfc = x.row[kRowSFC + kC6];
        const float rso = sfc > 0.f ? x.L.csi[kC6] * recip(300.0f * sfc) : 3.0e38f;
        float gain_h, gain_b;
        h = c6_rate<float>(h, isi_h, rso, x.L.fme_r, gain_h);
        b = c6_rate<float>(b, isi_b, rso, x.L.fme_r, gain_b);
        out.widen = fmaxf(1.0f, fmaxf(gain_h, gain_b) * (1.0f / kC6Gain));
    }
    out.h = h;
    out.b = b;
    const CoefR<float>& k = x.coef[kCurveLB + (int)grass];
    float base = M::one_minus_exp(k.b * wsv);
    base = grass ? wsv : base;
    const float lb = k.a * M::pow(base, k.c);
    out.lbm1 = grass ? (wsv >= 1.0f ? lb - 1.0f : 0.0f) : lb;
    out.lb = 1.0f + out.lbm1;
    out.wx = wx;
    out.wy = wy;
    out.wsv = wsv;
    out.edge = fabsf(wsv - 40.0f) < kEdgeWsv || (grass && fabsf(wsv - 1.0f) < kEdgeWsv);
    return out;
}

// The rates of all eight axes, pair by pair (axes k and k + 4 point opposite
// ways, so at most one of them lies in the front half).
template <typename M>
__device__ __forceinline__ void lane_axis_rates(const CellRates<float>& cr, float mu, float* x8) {
    const float a = 0.5f * (cr.h + cr.b);
    const float il = recip(cr.lb);
    const float il2 = il * il;
    const float base = a * il2;
    const float e = M::sqrt(cr.lbm1 * (cr.lbm1 + 2.0f)) * il;
    const float one_m_e = il2 * recip(1.0f + e);
    const float inv_wsv = (cr.wsv > 0.0f) ? recip(cr.wsv) : 0.0f;
    const float cx = cr.wx * inv_wsv, cy = cr.wy * inv_wsv;
    const float s = 0.70710678118654752440f;
    const float ux[4] = {1.0f, s, 0.0f, -s}, uy[4] = {0.0f, s, 1.0f, s};
    const float back = mu * base;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float c = ux[k] * cx + uy[k] * cy;
        const bool fb = c < 0.0f;
        const float dx = cx - (fb ? -ux[k] : ux[k]), dy = cy - (fb ? -uy[k] : uy[k]);
        const float front = mu * (base * recip(one_m_e + e * (0.5f * (dx * dx + dy * dy))));
        x8[k] = c > 0.0f ? front : back;
        x8[k + 4] = fb ? front : back;
    }
}

// The random part of one cell a lane: the noise multiplier and the eight
// rounding words (1/2 as a 24-bit fraction without stochastic rounding).
template <bool MIXED>
__device__ __forceinline__ float lane_draws(const EvalRep& e, uint32_t cell, uint32_t period, uint32_t* w) {
    using M = typename std::conditional<MIXED, MathFast, MathOf<float>>::type;
    uint32_t k0 = (uint32_t)e.seed, k1 = (uint32_t)(e.seed >> 32);
    asm volatile("" : "+s"(k0), "+s"(k1));   // as in quad_words
    float mu = 1.f;
    if (e.sigma != 0.f) {
        const uint4 n = philox4x32_10(make_uint4(cell, period, e.rep, 0u), k0, k1);
        mu = noise_of<float, M>(n.x, n.y, e.sigma);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = 0x80000000u;
    if (e.rounding != 0) {
        const uint4 ua = philox4x32_10(make_uint4(cell, period, e.rep, 1u), k0, k1);
        const uint4 ub = philox4x32_10(make_uint4(cell, period, e.rep, 2u), k0, k1);
        w[0] = ua.x, w[1] = ua.y, w[2] = ua.z, w[3] = ua.w;
        w[4] = ub.x, w[5] = ub.y, w[6] = ub.z, w[7] = ub.w;
    }
    return mu;
}

// axis_q of one cell a lane, called by the whole wave together.  done = false:
// the cell needs a quad and the rates have no meaning.
template <bool MIXED>
__device__ __forceinline__ bool lane_axis_q(const EvalLds<float>& x, const EvalRep& e, const CellRec& rec, float mu,
                                            const uint32_t* w, int32_t* q, bool& done) {
    using M = typename std::conditional<MIXED, MathFast, MathOf<float>>::type;
    const CellRates<float> cr = lane_cell_rates<M>(x, rec, done);
    if constexpr (MIXED) done = done && !cr.edge;
    bool faint = false;
    if (e.hfi_min > 0.f) {
        bool steep;
        const double hfi = (double)(head_intensity(cr, rec_fuel(rec.info), x.row, x.L, (float*)nullptr, &steep) * mu);
        const double hm = (double)e.hfi_min;
        if constexpr (MIXED) done = done && !steep && fabs(hfi - hm) > intensity_margin(e) * (double)cr.widen * hm;
        faint = !(hfi >= hm);
    }
    float x8[8];
    lane_axis_rates<M>(cr, mu, x8);
    const float margin = MIXED ? e.margin * cr.widen : 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float u = unit24<float>(w[k]);
        if constexpr (MIXED) q[k] = quantise_mixed(x8[k], u, margin, done);
        else q[k] = quantise<float>(x8[k], u);
    }
    return faint;
}

// head_rate with the context in LDS, out of line: used only where an
// ignition threshold is set.
template <typename R>
static inline __device__ __attribute__((noinline)) R head_rate_lds(const EvalLds<R>* x, const EvalLds<double>* x64,
                                                            const EvalRep* e, const CellRec* cells, uint32_t cell,
                                                            uint32_t period) {
    const CellRec rec = cells[cell];
    const LandR<R> L{x->L.pc_w, x->L.cf, (R)0, x->L.pdf_w, x->L.fme_r, x->L.csi};
    const LandR<double> L64{x64->L.pc_w, x64->L.cf, 0.0, x64->L.pdf_w, x64->L.fme_r, x64->L.csi};
    const CellRates<R> cr = cell_rates<R>(x->coef, x64->coef, rec, x->row, x64->row, L, L64);
    return cr.h * noise_mult<R>(e->seed, cell, period, e->rep, (R)e->sigma);
}

}  // namespace c2f
