// Stage kernels of the eta-based, well-balanced central-upwind scheme
// (Brodtkorb & Holm, arXiv 1912.02457) for gfx950.
//
// Work decomposition: one wavefront owns a strip of 64 consecutive columns
// (60 output columns plus a 2-column halo on each side) and marches down a
// block of rows with a sliding register window.  Neighbours along x come from
// the adjacent lanes (cross-lane shuffles), neighbours along y from the rows
// kept in registers, so every face flux is evaluated once and reused by the
// two cells that share the face.  LDS holds only the boundary state of a
// tile's relaxation zones (FrsTable, 3.2 KB a wave).  Global loads are
// 64-float (256 B) row segments.  Ghost cells sit in a 2-cell frame around
// every plane, written by the stage that produces the state (swe_device.h).
//
// Arithmetic follows the paper in float32 with two exact rewritings:
//   * the rest-state pressure g R_f^2/2 with R_f = max(H_f, 0) is taken out
//     of the pressure flux g h_f^2/2 and out of the bathymetry source
//     (g/2dx)(h^E + h^W)(H_E - H_W); the two parts cancel exactly, so M is
//     unchanged, but the float32 flux difference no longer carries the
//     cancellation of g H^2/2 ~ 4e7 at 3000 m (section "Accuracy, precision
//     and GPUs" motivates eta for the same reason).  The source then reads
//     (g/2dx)[(eta^E + eta^W)(H_E - H_W) + min(H_E,0)^2 - min(H_W,0)^2]:
//     below the datum only the eta part remains, above it (dry land, H < 0)
//     nothing is subtracted and a dry cell stays exactly at rest;
//   * the north-vector projection of the Coriolis term (section "Coriolis
//     force") returns f (hv, -hu) for every angle; the default variant uses
//     that identity, PROJ = true evaluates the projection literally.
#include <hip/hip_ext.h>

#include "swe_device.h"
#include "swe_maps.h"

namespace swe {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Plane accesses by 32-bit element offset.  The byte offset is formed in 32
// bits (every plane is below 4 GiB, checked at init), so the access uses the
// scalar-base + 32-bit vector-offset addressing form and needs no 64-bit
// address arithmetic per lane.
__device__ __forceinline__ float ld(const float *__restrict__ base, uint32_t off)
{
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + (off << 2));
}
__device__ __forceinline__ void st(float *__restrict__ base, uint32_t off, float v)
{
    *reinterpret_cast<float *>(reinterpret_cast<char *>(base) + (off << 2)) = v;
}
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// The same value, opaque to the compiler (an empty asm on a VGPR, no
// instruction).  A store whose offset comes from another basic block gets
// that offset as a 64-bit value and a 64-bit address add per plane; an
// offset made opaque in the store's own block is widened there, so the
// stores take the scalar-base form like the loads.
__device__ __forceinline__ uint32_t local_off(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Rounding errors of the compensated state are stored in 16 bits: the upper
// half of the float32 error, rounded to nearest (ties away from zero), i.e. a
// bfloat16.  An error is at most half an ulp of its value, so the pair keeps
// the value to about 2^-10 of a float32 ulp.  A load takes two more bits of
// address arithmetic and one shift; a store one add.
__device__ __forceinline__ uint32_t ld_lo(const uint16_t *__restrict__ base, uint32_t off)
{
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(base) + (off << 1));
}
__device__ __forceinline__ float lo_value(uint32_t bits) { return __uint_as_float(bits << 16); }
__device__ __forceinline__ void st_lo(uint16_t *__restrict__ base, uint32_t off, float v)
{
    *reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(base) + (off << 1)) =
        (uint16_t)((__float_as_uint(v) + 0x8000u) >> 16);
}

// a + b = s + err exactly (Knuth's TwoSum, no assumption on the magnitudes)
__device__ __forceinline__ float two_sum(float a, float b, float &err)
{
    const float s = a + b, bp = s - a, ap = s - bp;
    err = (a - ap) + (b - bp);
    return s;
}

constexpr uint32_t kSign = 0x80000000u;
__device__ __forceinline__ float flip_sign(float x, uint32_t s) { return __uint_as_float(__float_as_uint(x) ^ s); }

// rounding errors of the own cell's stored Q^n (0) and Q* (1) values, as
// stored: the shift to a float comes where they are used (next to the load it
// would wait for it)
struct Lo {
    uint32_t e0, u0, v0, e1, u1, v1;
};

// Value held by lane-1 / lane+1 through a whole-wave DPP shift (wave_shr:1
// and wave_shl:1 of the GFX9 DPP controls; a VALU operand modifier, no LDS
// round trip).  Lane 0 / lane 63 receive 0 (bound_ctrl: the lane without a
// source reads zero, so no old value has to be set up first); they are halo
// lanes whose results are never stored.
constexpr int kDppWaveShl1 = 0x130;
constexpr int kDppWaveShr1 = 0x138;
__device__ __forceinline__ int from_left(int v) { return __builtin_amdgcn_update_dpp(0, v, kDppWaveShr1, 0xF, 0xF, true); }
__device__ __forceinline__ int from_right(int v) { return __builtin_amdgcn_update_dpp(0, v, kDppWaveShl1, 0xF, 0xF, true); }
__device__ __forceinline__ float from_left(float v) { return __int_as_float(from_left(__float_as_int(v))); }
__device__ __forceinline__ float from_right(float v) { return __int_as_float(from_right(__float_as_int(v))); }

// A wave-uniform lane mask as a per-lane condition (no vector instruction),
// and the mask of the lanes whose left / right neighbour is in a mask.
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// Uniform conditions of the row loop, the usual case in line: the other one's
// code moves out of the loop's way (and out of its instruction cache lines).
__device__ __forceinline__ bool likely(bool c) { return __builtin_expect(c, 1); }
__device__ __forceinline__ bool unlikely(bool c) { return __builtin_expect(c, 0); }
__device__ __forceinline__ uint64_t left_in(uint64_t m) { return m << 1; }
__device__ __forceinline__ uint64_t right_in(uint64_t m) { return m >> 1; }

// eq. desing_ours; h^2/(2 kappa) + kappa/2 is formed as (h h + kappa^2) /
// (2 kappa), one uniform operand per instruction.  That value q is never
// below |h| (equal only at |h| = kappa) and is below kappa exactly when |h|
// is, so max(|h|, min(q, kappa)) is the median of |h|, q and kappa.
template <class D>
__device__ __forceinline__ float desing(float h, const D &d)
{
    const float q = fmaf(h, h, d.kappa_sq) * d.inv2kappa;
    const float m = __builtin_amdgcn_fmed3f(fabsf(h), q, d.kappa);
    // sign(h) with sign(0) = +1: adding +0 turns a -0 into +0
    return copysignf(m, h + 0.f);
}

// TWICE the generalized minmod of theta*backward, central, theta*forward
// differences dm, dp: minmod(2 theta dm, dm + dp, 2 theta dp), given as its
// three candidates a = 2 theta dm, b = dm + dp, c = 2 theta dp (scaling by
// two is exact, so callers take a quarter of it where the slope's half is
// used, bitwise the same as halving the minmod).  The median of two numbers
// and 0 is the smaller one in magnitude if they agree in sign, else 0; b has
// the common sign of a and c, so two medians give the minmod of all three.
// Along y each row's 2 theta multiple serves the faces below and above it.
__device__ __forceinline__ float limited2(float a, float b, float c)
{
    return __builtin_amdgcn_fmed3f(__builtin_amdgcn_fmed3f(a, c, 0.f), b, 0.f);
}

// limited2 along x, the forward difference being the right neighbour's
// backward one: its 2 theta multiple is the neighbour's product, moved by
// one lane (the same bits as multiplying the moved difference)
__device__ __forceinline__ float limited2_x(float dm, float th2)
{
    const float a = th2 * dm;
    return limited2(a, dm + from_right(dm), from_right(a));
}

// value of lane `k` (the same k in every lane) of a double
__device__ __forceinline__ double lane_value(double v, int k)
{
    const uint64_t b = __double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, k), hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Interval k and weight s of time tau in a table of n increasing snapshot
// times, clamped at its ends.  Called with all lanes of the wave active: the
// lanes compare 64 entries at once, so a table of up to 63 times takes one
// load and one of up to 63 * 63 two.  (A scalar scan from the front is one
// dependent load per snapshot passed: 80 to 240 snapshots into a boundary
// record, a step of the 1024 x 1024 beach took 112 us with it and takes 47
// with this search, and a 331 x 217 channel under 25 snapshots of gridded
// wind 19.6 and 16.6 us.)
// `early`: the lane's entry of a table of up to 63 times, loaded beforehand
// (first_times), or null.
__device__ __forceinline__ double first_times(int n, const double *ts)
{
    const int lane = threadIdx.x & (kWave - 1);
    return ts[min(lane, n - 1)];
}
__device__ __forceinline__ void time_weights(int n, const double *ts, double tau, int &k, double &s,
                                             const double *early = nullptr)
{
    k = 0;
    s = 0.0;
    if (n <= 1) return;
    const int lane = threadIdx.x & (kWave - 1);
    int base = 0, len = n;  // the last time <= tau is entry base .. base + len - 1
    while (len > kWave - 1) {
        const int stride = (len + kWave - 2) / (kWave - 1), at = base + lane * stride;
        const bool le = lane * stride < len && ts[at < n ? at : n - 1] <= tau;
        const int cnt = __popcll(__builtin_amdgcn_ballot_w64(le));
        base += (cnt > 0 ? cnt - 1 : 0) * stride;
        len = min(stride, n - base);
    }
    const double t = early && n < kWave ? *early : ts[min(base + lane, n - 1)];
    const int cnt = __popcll(__builtin_amdgcn_ballot_w64(lane < len && t <= tau));
    const int a = cnt > 0 ? cnt - 1 : 0;  // lane of that entry
    if (base + a >= n - 1) { k = n - 2; s = 1.0; return; }
    const double ta = lane_value(t, a), tb = lane_value(t, a + 1);
    if (base + a == 0 && tau <= ta) return;
    k = base + a;
    s = (tau - ta) / (tb - ta);
}

// Wave-wide maximum of unsigned numbers, the same scalar in every lane.  Steps
// within rows of 16 lanes, then the last lane of a row (and of the lower half)
// to those above; a lane without a source takes 0.  Cross-lane moves of the
// vector unit: six dependent trips through LDS (__shfl_xor) took 0.2 us, at
// the start of every stage 1 and the end of every stage 2 (us a step with them
// and without: 128 x 128 bump 9.62 and 9.26, 331 x 217 channel 12.2 and 12.0,
// 777 x 333 bay 14.5 and 14.2).
template <int CTRL>
__device__ __forceinline__ uint32_t max_step(uint32_t v)
{
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max_step<0x111>(v);  // row_shr:1, 2, 4, 8
    v = max_step<0x112>(v);
    v = max_step<0x114>(v);
    v = max_step<0x118>(v);
    v = max_step<0x142>(v);  // row_bcast:15, 31
    v = max_step<0x143>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// wave-wide maximum of a float that may be anything (NaN is passed over)
__device__ __forceinline__ float wave_max_any(float v)
{
    for (int off = kWave / 2; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
    return v;
}

// CFL accumulator of one parity: maximum over the slots (all lanes get it)
__device__ __forceinline__ uint32_t read_wmax(const Ctrl *c, int parity, int lane)
{
    return wave_max(c->wslot[parity][lane & (kCflSlots - 1)][0]);
}


// What the forcing of a tile needs whatever its time, issued with its first
// rows instead of after the time step is known, one more wait for memory at the
// head of every wave: the first snapshot of the uniform wind and the times of
// the tables (us a step before and now: 128 x 128 bump 9.3 and 9.1, 512 x 512
// 14.6 and 14.0, 331 x 217 channel 12.0 and 11.7, 777 x 333 bay 14.2 and 13.8,
// beach 38.5 and 38.1).
struct WindStart {
    float x, y;
    double t, t10;
};
template <class D>
__device__ __forceinline__ WindStart load_wind(const D &d)
{
    WindStart w{0.f, 0.f, 0.0, 0.0};
    if (d.nw > 0) {
        w.x = d.wind[0];
        w.y = d.wind[1];
        if (d.nw > 1) w.t = first_times(d.nw, d.wind_t);
    }
    if (d.w10n > 1) w.t10 = first_times(d.w10n, d.w10_t);
    return w;
}

template <class D>
__device__ __forceinline__ void wind_at(const D &d, double tau, const WindStart &w, float &wx, float &wy)
{
    if (d.nw <= 0) { wx = wy = 0.f; return; }
    double ax = w.x, ay = w.y;
    if (d.nw > 1) {
        int k; double s;
        time_weights(d.nw, d.wind_t, tau, k, s, &w.t);
        ax = d.wind[2 * k];
        ay = d.wind[2 * k + 1];
        ax = (1.0 - s) * ax + s * (double)d.wind[2 * k + 2];
        ay = (1.0 - s) * ay + s * (double)d.wind[2 * k + 3];
    }
    wx = (float)(ax * d.inv_rho_w);
    wy = (float)(ay * d.inv_rho_w);
}



// A domain block read through the scalar cache where it is used: in the rare
// parts of a tile (frame copies, relaxation zone, boundary tables) the fields
// come from here, so that they hold no scalar registers over the row loop
// (beyond the 102 there are, every use of a spilled one costs a vector
// instruction).  The empty asm keeps the loads from moving out of the loop.
using DomK = const __attribute__((address_space(4))) Dom;
__device__ __forceinline__ DomK &cold(DomK *p)
{
    asm volatile("" : "+s"(p));
    return *p;
}
// A uniform value whose tests stay where they are written: a test moved out
// of the row loop becomes a 64-bit lane mask, two more scalar registers.
__device__ __forceinline__ int here(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}

struct F3 { float e, p, q; };

// eq. numerical_flux for a face with depth Hf between a left state (eL,pL,qL)
// and a right state; p is the momentum normal to the face, q the transverse
// one.  Desingularised velocities, face momenta recomputed as h u, wave
// speeds a+ >= 0 >= a-, transverse momentum upwinded on the mass flux.
// Written with the weights alpha = a+/(a+ - a-), 1 - alpha and
// gamma = a+ a-/(a+ - a-); when a+ = a- = 0 (both sides dry and at rest)
// alpha = 1/2, gamma = 0 give the average of the two physical fluxes.  No
// branches, so the flux of a face can be interleaved with other work.
// The pressure uses the perturbation form (see the file header).
template <class D>
__device__ __forceinline__ F3 cu_flux(float eL, float pL0, float qL0, float eR, float pR0, float qR0,
                                      float Hf, const D &d)
{
    float hL = eL + Hf, hR = eR + Hf;
    float rL = rcp(desing(hL, d)), rR = rcp(desing(hR, d));
    float uL = pL0 * rL, vL = qL0 * rL, uR = pR0 * rR, vR = qR0 * rR;
    // h* = h where the water is deep: the face momentum is h u = p itself
    float pL = hL > d.deep ? pL0 : hL * uL, pR = hR > d.deep ? pR0 : hR * uR;
    float cL = fsqrt(d.g * fmaxf(hL, 0.f)), cR = fsqrt(d.g * fmaxf(hR, 0.f));
    float ap = fmaxf(fmaxf(uL + cL, uR + cR), 0.f);
    float am = fminf(fminf(uL - cL, uR - cR), 0.f);
    // g (h_f^2 - R_f^2) / 2 = g/2 (eta_f + min(H_f,0)) (eta_f + H_f + max(H_f,0))
    float Hn = fminf(Hf, 0.f), Hs2 = Hf + fmaxf(Hf, 0.f);
    float PL = 0.5f * d.g * (eL + Hn) * (eL + Hs2), PR = 0.5f * d.g * (eR + Hn) * (eR + Hs2);
    float FL = fmaf(pL, uL, PL), FR = fmaf(pR, uR, PR);
    // a+ - a- below 2^-100 m/s counts as a+ = a- = 0: its FP32 reciprocal
    // would overflow (a denormal momentum on a dry face gives such speeds)
    // and turn the weights into inf * 0.  Only faces with h_f <= 1e-61 m on
    // both sides fall in the gap, where both branches agree to O(g h_f^2).
    float den = ap - am;
    bool wet = den > 0x1p-100f;
    float w = wet ? rcp(den) : 0.f;
    const float apw = ap * w;
    float al = wet ? apw : 0.5f;
    float ga = am * apw;
    // alpha F_L + (1 - alpha) F_R as F_R + alpha (F_L - F_R): one operation
    // less, and exactly F_R where the two physical fluxes are equal (a lake
    // at rest)
    const float dp = pL - pR;
    F3 r;
    r.e = fmaf(al, dp, fmaf(ga, eR - eL, pR));
    r.p = fmaf(al, FL - FR, fmaf(ga, -dp, FR));
    r.q = r.e * (r.e >= 0.f ? vL : vR);
    return r;
}

// The same flux, bit for bit (up to the sign of a zero), where the face
// depth and the water depth on both sides exceed Dom::deep: h* = h, the face
// is below the datum (min(H_f,0) = 0) and a+ - a- >= 2 sqrt(g h) > 0, so the
// desingularisation, the dry-face weights and the datum terms drop out: 38
// instead of 66 vector instructions, beside the five transcendental ones.
template <class D>
__device__ __forceinline__ F3 cu_flux_deep(float eL, float pL, float qL, float eR, float pR, float qR, float Hf,
                                           const D &d)
{
    const float hL = eL + Hf, hR = eR + Hf;
    const float rL = rcp(hL), rR = rcp(hR);
    const float uL = pL * rL, vL = qL * rL, uR = pR * rR, vR = qR * rR;
    const float cL = fsqrt(d.g * hL), cR = fsqrt(d.g * hR);
    const float ap = fmaxf(fmaxf(uL + cL, uR + cR), 0.f);
    const float am = fminf(fminf(uL - cL, uR - cR), 0.f);
    const float H2 = Hf + Hf;
    const float PL = 0.5f * d.g * eL * (eL + H2), PR = 0.5f * d.g * eR * (eR + H2);
    const float FL = fmaf(pL, uL, PL), FR = fmaf(pR, uR, PR);
    const float al = ap * rcp(ap - am);
    const float ga = am * al;
    const float dp = pL - pR;
    F3 r;
    r.e = fmaf(al, dp, fmaf(ga, eR - eL, pR));
    r.p = fmaf(al, FL - FR, fmaf(ga, -dp, FR));
    r.q = r.e * (r.e >= 0.f ? vL : vR);
    return r;
}

// What a row of faces has beside plain deep water, uniform over the wave:
// DEEP: every face that touches water is deep in the sense of cu_flux_deep;
// LAND: some cell is land.  The kernels decide once per row and then run
// straight-line code for both directions: decided at every use (twenty
// branches a row instead of seven), stage 2 took 7 % longer where two waves
// share a SIMD (2600 x 900 coast in 24-row bands: 56.0 against 52.4 us) and 4 %
// where they fill it (2048 x 2048 in 12-row bands: 41.0 against 39.4).
//
// Face with the land rule: a face touching land carries the reflective-wall
// flux of its wet side; a face between two land cells carries nothing.  landL
// and landR are the lanes whose left (lower) and right (upper) cell is land;
// without any the selects leave every value as it is.
template <bool DEEP, bool LAND, class D>
__device__ __forceinline__ F3 face_flux(float eL, float pL, float qL, float eR, float pR, float qR,
                                        uint64_t landL, uint64_t landR, float Hf, const D &d)
{
    if (LAND) {
        const bool lL = in_mask(landL), lR = in_mask(landR);
        const float e2R = lR ? eL : eR, p2R = lR ? -pL : pR, q2R = lR ? qL : qR;
        const float e2L = lL ? eR : eL, p2L = lL ? -pR : pL, q2L = lL ? qR : qL;
        eL = e2L; pL = p2L; qL = q2L;
        eR = e2R; pR = p2R; qR = q2R;
    }
    F3 r = DEEP ? cu_flux_deep(eL, pL, qL, eR, pR, qR, Hf, d) : cu_flux(eL, pL, qL, eR, pR, qR, Hf, d);
    if (LAND && in_mask(landL & landR)) r.e = r.p = r.q = 0.f;
    return r;
}

// bathymetry source times 2 dx / g (x) or 2 dy / g (y): (h^E + h^W)(H_E - H_W)
// minus (R_E^2 - R_W^2), R = max(H, 0), matching the pressure flux of
// cu_flux.  With h = eta + H and H^2 - max(H,0)^2 = min(H,0)^2 this is
//   (eta^E + eta^W)(H_E - H_W) + min(H_E,0)^2 - min(H_W,0)^2,
// one formula for wet and dry faces with no cancellation of large terms;
// the caller scales it by g / (2 dx) or g / (2 dy).
// Below the datum (DEEP) the last two terms are zero.
template <bool DEEP>
__device__ __forceinline__ float bathy_source(float eE, float eW, float HE, float HW)
{
    if (DEEP) return (eE + eW) * (HE - HW);
    float mE = fminf(HE, 0.f), mW = fminf(HW, 0.f);
    float dry = fmaf(mE, mE, -(mW * mW));
    return fmaf(eE + eW, HE - HW, dry);
}

// bed shear stress coefficient S >= 0, the source being -S (hu, hv), from the
// cell's reciprocal desingularised depth ri = 1/h*
template <class D>
__device__ __forceinline__ float friction_coeff(int law, const D &d, float ri, float hu, float hv)
{
    const float ra = fabsf(ri), coeff = d.fric_c;
    if (law <= FR_LINEAR) return law == FR_NONE ? 0.f : coeff * ra;
    const float speed = fsqrt(hu * hu + hv * hv) * ra;
    if (law == FR_QUADRATIC) return coeff * speed * ra * ra;
    // Manning: g n^2 |u| / a^(4/3) = g n^2 |u| ra^(4/3)
    const float ra43 = __builtin_amdgcn_exp2f((4.0f / 3.0f) * __builtin_amdgcn_logf(ra));
    return coeff * speed * ra43;
}

// Wet-dry fix of eq. KxE_adjust of a cell's face values ep, em = eta +/- rho:
// a face value below the bottom (eta_f + H_f < 0) is set to the bottom and
// the other face takes 2 eta - eta_f, keeping the cell average; first the
// face on the + side, then the one on the - side.  As max/min: raising
// the + face to -H_+ is a max, and then the - face (2 eta - that) is the
// min of itself and 2 eta + H_+ -- exact when the fix applies, and equal
// to the unfixed value otherwise (up to one rounding when the two are
// within an ulp).
__device__ __forceinline__ void positivity_fix(float e, float Hp, float Hm, float &ep, float &em)
{
    ep = fmaxf(ep, -Hp);
    em = fminf(em, fmaf(2.f, e, Hp));
    em = fmaxf(em, -Hm);
    ep = fminf(ep, fmaf(2.f, e, Hm));
}

// One row of the sliding window (per lane: column i).
struct Row {
    float e, u, v, f;      // state and Coriolis parameter (NaN: land)
    float cx, cy;          // Coriolis terms of the reconstruction (f v, -f u)
    float Hw, He, Hs, Hn, Hb;
    float ri;              // 1 / h* of the cell
    uint64_t land;         // lanes whose cell is land
    uint64_t shallown;     // lanes whose north-west corner depth is not deep
    uint64_t shallow;      // water lanes with a face or water depth that is not deep (Dom::deep)
    uint64_t shallowy;     // output lanes whose water at the north or south face is not deep
    float dmL, dmU, dmV;   // y backward differences (this row minus the row below)
    float tmL, tmU, tmV;   // the same times 2 theta
    float eN, eS, uN, vN;  // north/south face values once the row was the middle row
};

// face depths, mean depth, land flag and Coriolis terms of a row from its
// four corner depths (south corners cs*, north corners cn*); the south face
// depth hs is the north face depth of the row below, 0.5 (cs0 + cs1)
template <bool PROJ, class D>
__device__ __forceinline__ void row_terms(Row &R, float cs0, float cs1, float cn0, float cn1, float hs, float th,
                                          const D &d)
{
    R.Hw = 0.5f * (cs0 + cn0);
    R.He = 0.5f * (cs1 + cn1);
    R.Hs = hs;
    R.Hn = 0.5f * (cn0 + cn1);
    R.Hb = 0.25f * ((cs0 + cn0) + (cs1 + cn1));
    const float h = R.e + R.Hb;
    R.land = __builtin_amdgcn_ballot_w64(isnan(R.f));
    // every face depth is the mean of two corner depths, and a cell's east
    // corners are the west ones of the next lane (lane 63's are not covered;
    // no output depends on its faces).  A depth that is not a number counts
    // as shallow
    const uint64_t north = __builtin_amdgcn_ballot_w64(!(cn0 > d.deep));
    const uint64_t corners = north | R.shallow;  // R.shallow: south on entry
    R.shallow = (corners | right_in(corners) | __builtin_amdgcn_ballot_w64(!(h > d.deep))) & ~R.land;
    R.shallown = north;
    const float ri = rcp(desing(h, d));
    R.ri = ri;
    float uu = R.u * ri, vv = R.v * ri;
    if (PROJ) {
        float c = __cosf(th), s = __sinf(th);
        float ue = c * uu - s * vv, vn = s * uu + c * vv;
        R.cx = R.f * (c * vn - s * ue);
        R.cy = R.f * (-s * vn - c * ue);
    } else {
        R.cx = R.f * vv;
        R.cy = -R.f * uu;
    }
}

// backward differences along y of row C against the row B below it; the
// K-type difference of eq. Kbackwards in its y form (L = g(eta + U))
template <class D>
__device__ __forceinline__ void y_diff(Row &C, const Row &B, const D &d)
{
    C.dmL = C.e - B.e - d.ky * (B.cy + C.cy);
    C.dmU = C.u - B.u;
    C.dmV = C.v - B.v;
    C.tmL = d.theta2 * C.dmL;
    C.tmU = d.theta2 * C.dmU;
    C.tmV = d.theta2 * C.dmV;
}

// limited y-slopes and N/S face values of row B (eq. hE in its N/S form);
// stores the N values, eS and the lanes that need the wet-dry fix in B and
// returns the S momenta for the face below B.  out: the output lanes of the
// tile, the only ones whose y-fluxes are used.
template <class D>
__device__ __forceinline__ void y_faces(Row &B, const Row &C, uint64_t landA, uint64_t out, const D &d, float &uS,
                                        float &vS)
{
    // twice the limited slopes (limited2)
    float sL = limited2(B.tmL, B.dmL + C.dmL, C.tmL);
    float sU = limited2(B.tmU, B.dmU + C.dmU, C.tmU);
    float sV = limited2(B.tmV, B.dmV + C.dmV, C.tmV);
    // first order next to land
    if (in_mask(landA | C.land)) sL = sU = sV = 0.f;
    const float rho = 0.25f * sL + d.ky * B.cy;
    B.eN = B.e + rho;
    B.eS = B.e - rho;
    // lanes of deep water at both faces: the wet-dry fix leaves them as they are
    const float low = fminf(B.eN + B.Hn, B.eS + B.Hs);
    B.shallowy = (B.shallow | (__builtin_amdgcn_ballot_w64(!(low > d.deep)) & ~B.land)) & out;
    B.uN = B.u + 0.25f * sU;
    B.vN = B.v + 0.25f * sV;
    uS = B.u - 0.25f * sU;
    vS = B.v - 0.25f * sV;
}

// flux through the face between row A (below, its N values) and row B
// (above, its S values): normal momentum hv, transverse hu
template <bool DEEP, bool LAND, class D>
__device__ __forceinline__ F3 y_flux(const Row &A, const Row &B, float uS, float vS, const D &d)
{
    return face_flux<DEEP, LAND>(A.eN, A.vN, A.uN, B.eS, vS, uS, A.land, B.land, B.Hs, d);
}

enum {
    kTileEdge = 1,    // writes ghost cells (output cells within two cells of a side)
    kTileFrs = 2,     // has output cells in a relaxation zone
    kTileFriction = 2 // shift of the friction law
};
struct TileCtx {
    int i, o;        // column of this lane, output row
    int lane, x0;    // lane and its strip's first output column
    bool out_lane;   // lane owns an output cell
    uint64_t out;    // the lanes that do
    uint64_t xneed;  // the lanes whose x-faces an output cell depends on (one more on each side)
    float dt, wx, wy;
    int kind;        // what the tile's rows do beside the update: bits below
    int fca, fcb;    // ghost columns that copy this lane's cells (frame_copy_cols)
    int wk;          // wind-field snapshot interval and weight at the stage time
    float ws;
};

// Wind at 10 m from its own grid at cell (i, o): samples at the centres of a
// w10nx x w10ny partition of the domain, bilinear in space (clamped at the
// edges, as a texture fetch with linear filtering) and linear in time between
// the snapshots around the stage time (eq. windstress_interpol); then the
// stress of Large and Pond, rho_a/rho_w C_D |W| W with C_D = 1.2e-3 below
// 11 m/s and (0.49 + 0.065 |W|) 1e-3 above, as the kinematic source.
template <class D>
__device__ __forceinline__ void w10_stress(const D &d, const TileCtx &c, float &sx, float &sy)
{
    float gx = fminf(fmaxf(((float)c.i + 0.5f) * d.w10sx - 0.5f, 0.f), (float)(d.w10nx - 1));
    float gy = fminf(fmaxf(((float)c.o + 0.5f) * d.w10sy - 0.5f, 0.f), (float)(d.w10ny - 1));
    const int i0 = (int)gx, j0 = (int)gy;
    const int i1 = min(i0 + 1, d.w10nx - 1), j1 = min(j0 + 1, d.w10ny - 1);
    const float fx = gx - (float)i0, fy = gy - (float)j0;
    const uint32_t plane = (uint32_t)d.w10nx * (uint32_t)d.w10ny * 2u;
    const float *Wa = d.w10 + (uint32_t)c.wk * plane;
    const float *Wb = d.w10n > 1 ? Wa + plane : Wa;
    float W[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        auto at = [&](const float *P, int i, int j) { return P[((uint32_t)j * (uint32_t)d.w10nx + (uint32_t)i) * 2u + q]; };
        float a = (1.f - fy) * ((1.f - fx) * at(Wa, i0, j0) + fx * at(Wa, i1, j0)) +
                  fy * ((1.f - fx) * at(Wa, i0, j1) + fx * at(Wa, i1, j1));
        float b = (1.f - fy) * ((1.f - fx) * at(Wb, i0, j0) + fx * at(Wb, i1, j0)) +
                  fy * ((1.f - fx) * at(Wb, i0, j1) + fx * at(Wb, i1, j1));
        W[q] = (1.f - c.ws) * a + c.ws * b;
    }
    if (d.w10_kind) {  // a stress field, interpolated as it is
        sx = d.w10q * W[0];
        sy = d.w10q * W[1];
        return;
    }
    const float sp = fsqrt(W[0] * W[0] + W[1] * W[1]);
    const float cd = sp < 11.f ? 1.2e-3f : (0.49f + 0.065f * sp) * 1e-3f;
    const float k = d.w10q * cd * sp;
    sx = k * W[0];
    sy = k * W[1];
}

// Boundary state around the relaxation zones of a tile at the stage time,
// interpolated once per tile (once per 64 rows) by the whole wave and kept in
// LDS: along a west or east side it depends on the row, along a south or north
// side on the column.  (Loaded row by row where the update uses them, two
// dependent global loads a row made the zone tiles the last ones of every
// launch: stage 2 of the 2600 x 900 coast took 37.6 us nested on all sides
// and 28.8 us with walls.)
constexpr int kFrsRows = 64;
struct FrsTable {
    float x[2][kFrsRows][3];  // W, E: rows row0 .. row0 + 63
    float y[2][kWave][3];     // S, N: the strip's columns
    float alpha[kMaxFrs];
    double bs;                // weight and interval of the boundary snapshots
    int bk, row0;
};

__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// external (eta, hu, hv) at perimeter entry idx
__device__ __forceinline__ void boundary_state(DomK &d, int bk, double t, int idx, float (&q)[3])
{
    const uint32_t P = (uint32_t)d.P;
    const float *pa = d.bnd + (uint32_t)bk * 3u * P + (uint32_t)idx;
    const float *pb = d.nb > 1 ? pa + 3u * P : pa;
#pragma unroll
    for (int k = 0; k < 3; ++k) q[k] = (float)((1.0 - t) * (double)pa[k * P] + t * (double)pb[k * P]);
}

// rows row0 .. of the west and east tables (tiles are within a zone of those
// sides or not as a whole strip); by all lanes of one wave
__device__ __forceinline__ void frs_fill_rows(DomK &d, FrsTable &f, int x0, int row0, int lane)
{
    const int y = row0 + lane;
    if (y < d.ny) {
        if (d.bc[0] == BC_NESTED && x0 < d.frs_w) boundary_state(d, f.bk, f.bs, y, f.x[0][lane]);
        if (d.bc[1] == BC_NESTED && x0 + kStrip > d.nx - d.frs_w) boundary_state(d, f.bk, f.bs, d.ny + y, f.x[1][lane]);
    }
    if (lane == 0) f.row0 = row0;
}

// the whole table of a tile that starts at row y0
__device__ __forceinline__ void frs_fill(DomK &d, FrsTable &f, double tau, int x0, int y0, int y1, int i, int lane)
{
    int bk;
    double bs;
    time_weights(d.nb, d.bnd_t, tau, bk, bs);
    if (lane == 0) { f.bk = bk; f.bs = bs; }
    if (lane < kMaxFrs) f.alpha[lane] = d.frs_alpha[lane];
    if (i >= 0 && i < d.nx) {
        if (d.bc[2] == BC_NESTED && y0 < d.frs_w) boundary_state(d, bk, bs, 2 * d.ny + i, f.y[0][lane]);
        if (d.bc[3] == BC_NESTED && y1 > d.ny - d.frs_w) boundary_state(d, bk, bs, 2 * d.ny + d.nx + i, f.y[1][lane]);
    }
    wave_fence();
    frs_fill_rows(d, f, x0, y0, lane);
    wave_fence();
}

// Ghost cells of the state this stage writes (Q* in stage 1, Q^{n+1} in
// stage 2) for the stage that reads it next, by edge tiles: the wall and
// periodic copies of a water cell's new values (frame_copy_cols / _rows;
// the lane's target columns are fixed for the tile, the row targets are
// uniform), stored from the registers that hold them.  A land cell keeps
// its state, and its ghosts their values.
template <int STAGE>
__device__ __forceinline__ void write_frame_copies(DomK &d, const TileCtx &c, float e, float u, float v)
{
    float *__restrict__ E = STAGE == 1 ? d.eta1 : d.eta;
    float *__restrict__ U = STAGE == 1 ? d.hu1 : d.hu;
    float *__restrict__ V = STAGE == 1 ? d.hv1 : d.hv;
    auto put = [&](int x, int y, float uu, float vv) {
        const uint32_t o = cell_off(d, y, x);
        st(E, o, e);
        st(U, o, uu);
        st(V, o, vv);
    };
    if (c.fca != kNoFrame) put(c.fca, c.o, d.bc[0] == BC_WALL ? -u : u, v);
    if (c.fcb != kNoFrame) put(c.fcb, c.o, d.bc[1] == BC_WALL ? -u : u, v);
    int ra, rb;
    frame_copy_rows(d, c.o, ra, rb);
    if (ra != kNoFrame) put(c.i, ra, u, d.bc[2] == BC_WALL ? -v : v);
    if (rb != kNoFrame) put(c.i, rb, u, d.bc[3] == BC_WALL ? -v : v);
}

// Nested ghosts take the boundary data at the reading stage's time (the
// interpolation of the boundary loads), independent of the state: written by
// the tiles next to a nested side, the rows of a west or east side side by
// side over the lanes.
template <int STAGE>
__device__ __forceinline__ void write_frame_nested(DomK &d, double tau, int x0, int y0, int y1, int lane)
{
    float *__restrict__ E = STAGE == 1 ? d.eta1 : d.eta;
    float *__restrict__ U = STAGE == 1 ? d.hu1 : d.hu;
    float *__restrict__ V = STAGE == 1 ? d.hv1 : d.hv;
    const int nx = d.nx, ny = d.ny;
    int bk;
    double t;
    time_weights(d.nb, d.bnd_t, tau, bk, t);
    auto put = [&](int idx, int xa, int ya, int xb, int yb) {
        float q[3];
        boundary_state(d, bk, t, idx, q);
        const uint32_t oa = cell_off(d, ya, xa), ob = cell_off(d, yb, xb);
        st(E, oa, q[0]); st(U, oa, q[1]); st(V, oa, q[2]);
        st(E, ob, q[0]); st(U, ob, q[1]); st(V, ob, q[2]);
    };
    const bool w = d.bc[0] == BC_NESTED && x0 == 0;
    const bool e = d.bc[1] == BC_NESTED && x0 + kStrip >= nx;
    if (w || e) {
        for (int y = y0 + lane; y < y1; y += kWave) {
            if (w) put(y, -1, y, -2, y);
            if (e) put(ny + y, nx, y, nx + 1, y);
        }
    }
    const int x = x0 - kHalo + lane;
    if (lane >= kHalo && lane < kWave - kHalo && x < nx) {
        if (d.bc[2] == BC_NESTED && y0 == 0) put(2 * ny + x, x, -1, x, -2);
        if (d.bc[3] == BC_NESTED && y1 == ny) put(2 * ny + nx + x, x, ny, x, ny + 1);
    }
}

// lanes of a wave that stored a non-finite state, or a water depth below
// -kappa (ballot masks, the same in every lane)
struct BadLanes {
    uint64_t nonfinite, negative;
};

// limited x-slopes and E/W face values of row A, before the wet-dry fix
struct XFaces {
    float eE, eW, uE, uW, vE, vW;
    uint64_t shallow;  // lanes that need the fix, of those an output cell depends on
};

template <class D>
__device__ __forceinline__ XFaces x_faces(const Row &A, const TileCtx &c, const D &d)
{
    const float th2 = d.theta2;
    float eL = from_left(A.e), cxL = from_left(A.cx);
    float uL = from_left(A.u), vL = from_left(A.v);
    float dmK = A.e - eL - d.kx * (cxL + A.cx);
    float dmU = A.u - uL, dmV = A.v - vL;
    // twice the limited slopes (limited2)
    float sK = limited2_x(dmK, th2);
    float sUx = limited2_x(dmU, th2);
    float sVx = limited2_x(dmV, th2);
    // first order next to land
    if (in_mask(left_in(A.land) | right_in(A.land))) sK = sUx = sVx = 0.f;
    const float rx = 0.25f * sK + d.kx * A.cx;
    XFaces x;
    x.eE = A.e + rx;
    x.eW = A.e - rx;
    const float low = fminf(x.eE + A.He, x.eW + A.Hw);
    x.shallow = (A.shallow | (__builtin_amdgcn_ballot_w64(!(low > d.deep)) & ~A.land)) & c.xneed;
    x.uE = A.u + 0.25f * sUx;
    x.uW = A.u - 0.25f * sUx;
    x.vE = A.v + 0.25f * sVx;
    x.vW = A.v - 0.25f * sVx;
    return x;
}

// what row A's update takes from its faces: the differences of the x-fluxes
// (east minus west) and the bathymetry sources of both directions
struct RowFlux {
    float dFe, dFp, dFq, bx, by;
};

template <bool DEEP, bool LAND, class D>
__device__ __forceinline__ RowFlux x_flux(const Row &A, XFaces &x, const D &d)
{
    if (!DEEP) positivity_fix(A.e, A.He, A.Hw, x.eE, x.eW);
    const F3 F = face_flux<DEEP, LAND>(x.eE, x.uE, x.vE, from_right(x.eW), from_right(x.uW), from_right(x.vW), A.land,
                                       right_in(A.land), A.He, d);
    RowFlux r;
    r.dFe = F.e - from_left(F.e);
    r.dFp = F.p - from_left(F.p);
    r.dFq = F.q - from_left(F.q);
    r.bx = bathy_source<DEEP>(x.eE, x.eW, A.He, A.Hw);
    r.by = bathy_source<DEEP>(A.eN, A.eS, A.Hn, A.Hs);
    return r;
}

// x- and y-fluxes of one step of the row loop: the flux through the north
// face of row A (its south one is known) and row A's x-part
template <bool DEEP, bool LAND, class D>
__device__ __forceinline__ void row_fluxes(const Row &A, Row &B, XFaces &x, float uS, float vS, const D &d, F3 &Gn,
                                           RowFlux &r)
{
    if (!DEEP) positivity_fix(B.e, B.Hn, B.Hs, B.eN, B.eS);
    Gn = y_flux<DEEP, LAND>(A, B, uS, vS, d);
    r = x_flux<DEEP, LAND>(A, x, d);
}

// The update of eq. rk2_semiimp of row A and (stage 2) the flow relaxation
// and CFL reduction.
template <int STAGE, bool PROJ, bool W10, bool COMP, class D>
__device__ __forceinline__ void finish_row(const Row &A, const F3 &Gs, const F3 &Gn, const RowFlux &rf,
                                           const TileCtx &c, float e0, float u0, float v0, const Lo &lo, DomK *dk,
                                           const FrsTable &ft,
                                           const D &d, float &wmax_loc, BadLanes &bad)
{
    // every lane computes; only output lanes over water store (no early exit,
    // so the x and y work of neighbouring rows can be interleaved)
    const uint64_t stored = c.out & ~A.land;
    const bool store = in_mask(stored);

    float Cx, Cy;
    if (PROJ) {
        float ang = store ? ld(d.north, cell_off(d, c.o, c.i)) : 0.f;
        float cc = __cosf(ang), ss = __sinf(ang);
        float hue = cc * A.u - ss * A.v, hvn = ss * A.u + cc * A.v;
        Cx = A.f * (cc * hvn - ss * hue);
        Cy = A.f * (-ss * hvn - cc * hue);
    } else {
        Cx = A.f * A.v;
        Cy = -A.f * A.u;
    }
    float wx = c.wx, wy = c.wy;
    if (W10 && d.w10n > 0) {
        float sx, sy;
        w10_stress(d, c, sx, sy);
        wx += sx;
        wy += sy;
    }
    float Me = -rf.dFe * d.rdx - (Gn.e - Gs.e) * d.rdy;
    float Mu = -rf.dFp * d.rdx - (Gn.q - Gs.q) * d.rdy + rf.bx * d.grdx2 +
               Cx + wx;
    float Mv = -rf.dFq * d.rdx - (Gn.p - Gs.p) * d.rdy + rf.by * d.grdy2 +
               Cy + wy;
    const uint32_t oo = cell_off(d, c.o, c.i);
    const float dt = c.dt;
    const int kind = here(c.kind);
    float S = friction_coeff(kind >> kTileFriction, d, A.ri, A.u, A.v);
    if (STAGE == 1) {
        float den = rcp(1.f + dt * S);
        if (COMP) {
            // compensated: the increment of each field, added to the stored
            // value plus its rounding error without losing the new error
            float le, lu, lv;
            const float en = two_sum(A.e, dt * Me + lo_value(lo.e0), le);
            const float un = two_sum(A.u, (dt * Mu - dt * S * A.u) * den + lo_value(lo.u0), lu);
            const float vn = two_sum(A.v, (dt * Mv - dt * S * A.v) * den + lo_value(lo.v0), lv);
            if (store) {
                st(d.eta1, oo, en);
                st(d.hu1, oo, un);
                st(d.hv1, oo, vn);
                st_lo(d.eta1_lo, oo, le);
                st_lo(d.hu1_lo, oo, lu);
                st_lo(d.hv1_lo, oo, lv);
                if (unlikely(kind & kTileEdge)) write_frame_copies<1>(cold(dk), c, en, un, vn);
            }
        } else {
            float en = A.e + dt * Me;
            float un = (A.u + dt * Mu) * den;
            float vn = (A.v + dt * Mv) * den;
            if (store) {
                st(d.eta1, oo, en);
                st(d.hu1, oo, un);
                st(d.hv1, oo, vn);
                if (unlikely(kind & kTileEdge)) write_frame_copies<1>(cold(dk), c, en, un, vn);
            }
        }
    } else {
        float den = rcp(1.f + 0.5f * dt * S);
        float en, un, vn, le = 0.f, lu = 0.f, lv = 0.f;
        if (COMP) {
            // Q^{n+1} = Q^n + (Q* - Q^n + dt M(Q*))/2 (momenta with the
            // friction factor), the differences taken with both errors
            const float de = (A.e - e0) + (lo_value(lo.e1) - lo_value(lo.e0));
            const float du = (A.u - u0) + (lo_value(lo.u1) - lo_value(lo.u0));
            const float dv = (A.v - v0) + (lo_value(lo.v1) - lo_value(lo.v0));
            en = two_sum(e0, 0.5f * (de + dt * Me) + lo_value(lo.e0), le);
            un = two_sum(u0, (0.5f * (du + dt * Mu) - 0.5f * dt * S * u0) * den + lo_value(lo.u0), lu);
            vn = two_sum(v0, (0.5f * (dv + dt * Mv) - 0.5f * dt * S * v0) * den + lo_value(lo.v0), lv);
        } else {
            en = 0.5f * (e0 + (A.e + dt * Me));
            un = 0.5f * (u0 + (A.u + dt * Mu)) * den;
            vn = 0.5f * (v0 + (A.v + dt * Mv)) * den;
        }
        if (unlikely(kind & kTileFrs)) {
          DomK &dc = cold(dk);
          int best, dd;  // the nearest nested side (ties W, E, S, N)
          frs_side(dc, c.i, c.o, best, dd);
          if (c.out_lane && best >= 0 && dd < dc.frs_w) {
            const float al = ft.alpha[dd];
            const float *q = best < 2 ? ft.x[best][c.o - ft.row0] : ft.y[best - 2][c.lane];
            const float ex[3] = {q[0], q[1], q[2]};
            if (COMP) {
                en = two_sum(en, le + al * ((ex[0] - en) - le), le);
                un = two_sum(un, lu + al * ((ex[1] - un) - lu), lu);
                vn = two_sum(vn, lv + al * ((ex[2] - vn) - lv), lv);
            } else {
                en = (1.f - al) * en + al * ex[0];
                un = (1.f - al) * un + al * ex[1];
                vn = (1.f - al) * vn + al * ex[2];
            }
          }
        }
        if (store) {
            const uint32_t so = local_off(oo);
            st(d.eta, so, en);
            st(d.hu, so, un);
            st(d.hv, so, vn);
            if (COMP) {
                st_lo(d.eta_lo, so, le);
                st_lo(d.hu_lo, so, lu);
                st_lo(d.hv_lo, so, lv);
            }
            if (unlikely(kind & kTileEdge)) write_frame_copies<2>(cold(dk), c, en, un, vn);
        }

        // eq. cfl on the new state.  bit 0 of the flags: a non-finite state;
        // bit 1: a water depth below -kappa (the scheme keeps h >= 0 under
        // its CFL bound, so this means breakdown); both as lane masks
        const float h = en + A.Hb;
        bad.negative |= stored & __builtin_amdgcn_ballot_w64(h < -d.kappa);
        const float ri = rcp(desing(h, d));
        const float cw = fsqrt(d.g * fmaxf(h, 0.f));
        // with square cells the larger speed is taken first: the same value,
        // bit for bit, rounding being monotone, as long as the product is
        // rounded before the sum as in the other form and in cfl_kernel (the
        // outer fabsf keeps the two from fusing)
        float w;
        if (likely(d.rdx == d.rdy)) w = (fabsf(fmaxf(fabsf(un), fabsf(vn)) * ri) + cw) * d.rdx;
        else w = fmaxf((fabsf(un * ri) + cw) * d.rdx, (fabsf(vn * ri) + cw) * d.rdy);
        wmax_loc = store ? fmaxf(wmax_loc, w) : wmax_loc;
        bad.nonfinite |= stored & (__builtin_amdgcn_ballot_w64(!isfinite(en)) | __builtin_amdgcn_ballot_w64(!isfinite(un)) |
                                   __builtin_amdgcn_ballot_w64(!isfinite(vn)));
    }
}

// the stored rounding errors of the own cell
template <int STAGE, bool COMP, class D>
__device__ __forceinline__ Lo load_lo(const D &d, const TileCtx &c)
{
    Lo lo{0u, 0u, 0u, 0u, 0u, 0u};
    if (COMP) {
        const uint32_t oo = cell_off(d, c.o, c.i);
        lo.e0 = ld_lo(d.eta_lo, oo);
        lo.u0 = ld_lo(d.hu_lo, oo);
        lo.v0 = ld_lo(d.hv_lo, oo);
        if (STAGE == 2) {
            lo.e1 = ld_lo(d.eta1_lo, oo);
            lo.u1 = ld_lo(d.hu1_lo, oo);
            lo.v1 = ld_lo(d.hv1_lo, oo);
        }
    }
    return lo;
}

// ---- one tile: a wavefront's 64 columns over rows y0..y1-1 ------------------
// The window of three rows rotates by unrolling (no register moves, no
// per-row branches) and the next row is prefetched while the current one is
// processed.  Every load is a plain 32-bit offset into a framed plane: the
// ghost cells sit in the frame (filled by the stage that wrote the state),
// so edge tiles load exactly as interior ones.  frs: the tile has output
// cells inside a relaxation zone; edge: it has output cells within two
// cells of a side, whose values it also writes into the frame afterwards.
struct RawRow {
    float e, u, v, f, cn0, cn1, th;
};

template <bool PROJ, class D>
__device__ __forceinline__ RawRow load_row(const D &d, const float *__restrict__ E, const float *__restrict__ U,
                                           const float *__restrict__ V, int il, int r)
{
    RawRow w;
    const uint32_t off = cell_off(d, r, il);
    const uint32_t cof = corner_off(d, r + 1, il);
    w.e = ld(E, off);
    w.u = ld(U, off);
    w.v = ld(V, off);
    w.f = ld(d.f, off);
    w.cn0 = ld(d.Hc, cof);
    w.cn1 = ld(d.Hc, cof + 1);
    w.th = PROJ ? ld(d.north, off) : 0.f;
    return w;
}

// Makes the compiler wait for a row's loads at this point (an empty asm that
// reads them).
__device__ __forceinline__ void arrived(const RawRow &r)
{
    asm volatile("" ::"v"(r.e), "v"(r.u), "v"(r.v), "v"(r.f), "v"(r.cn0), "v"(r.cn1), "v"(r.th));
}

// the first row of a tile and its south corners, issued before the tile's
// other preparations
struct TileStart {
    RawRow row;
    float cs0, cs1;
};

template <int STAGE, bool PROJ, class D>
__device__ __forceinline__ TileStart load_start(const D &d, int il, int r)
{
    TileStart s;
    s.row = load_row<PROJ>(d, STAGE == 1 ? d.eta : d.eta1, STAGE == 1 ? d.hu : d.hu1, STAGE == 1 ? d.hv : d.hv1, il, r);
    const uint32_t cof = corner_off(d, r, il);
    s.cs0 = ld(d.Hc, cof);
    s.cs1 = ld(d.Hc, cof + 1);
    return s;
}

template <int STAGE, bool PROJ, bool W10, bool COMP, class D>
__device__ __forceinline__ void run_tile(const D &d, DomK *dk, FrsTable &ft, TileCtx c, const TileStart &start, int y0,
                                         int y1,
                                         float &wmax_loc, BadLanes &bad)
{
    const float *__restrict__ E = STAGE == 1 ? d.eta : d.eta1;
    const float *__restrict__ U = STAGE == 1 ? d.hu : d.hu1;
    const float *__restrict__ V = STAGE == 1 ? d.hv : d.hv1;
    const int il = c.i;
    float cs0 = start.cs0, cs1 = start.cs1;  // south corners of the row loaded next
    const int klast = y1 + 1;
    RawRow nxt = start.row;

    // B: the row below C, whose north face depth is C's south one
    auto load = [&](Row &C, const Row &B, int k) {
        RawRow cur = nxt;
        // unconditional (the last row reloads itself), so that the memory
        // counter is the same on every path and a wait for this row's own
        // loads never has to drain the prefetch of the next one
        nxt = load_row<PROJ>(d, E, U, V, il, min(k + 1, klast));
        C.e = cur.e; C.u = cur.u; C.v = cur.v; C.f = cur.f;
        C.shallow = B.shallown;
        row_terms<PROJ>(C, cs0, cs1, cur.cn0, cur.cn1, B.Hn, cur.th, d);
        cs0 = cur.cn0;
        cs1 = cur.cn1;
    };

    Row R0, R1, R2;
    float uS, vS;
    R2.Hn = 0.5f * (cs0 + cs1);  // the face below the first row
    R2.shallown = __builtin_amdgcn_ballot_w64(!(cs0 > d.deep));
    load(R0, R2, y0 - 2);
    load(R1, R0, y0 - 1);
    y_diff(R1, R0, d);
    load(R2, R1, y0);
    y_diff(R2, R1, d);
    y_faces(R1, R2, R0.land, c.out, d, uS, vS);
    if (R1.shallowy != 0) positivity_fix(R1.e, R1.Hn, R1.Hs, R1.eN, R1.eS);
    load(R0, R2, y0 + 1);
    y_diff(R0, R2, d);
    y_faces(R2, R0, R1.land, c.out, d, uS, vS);
    if (R2.shallowy != 0) positivity_fix(R2.e, R2.Hn, R2.Hs, R2.eN, R2.eS);
    F3 Gs = (R1.shallowy | R2.shallowy) == 0 ? y_flux<true, true>(R1, R2, uS, vS, d)
                                             : y_flux<false, true>(R1, R2, uS, vS, d);

    // steady state: A = row k-2 (output), B = row k-1, C = row k
    auto step = [&](Row &A, Row &B, Row &C, int k) {
        c.o = k - 2;
        float e0 = 0.f, u0 = 0.f, v0 = 0.f;
        if (STAGE == 2) {
            const uint32_t oq = cell_off(d, c.o, c.i);
            e0 = ld(d.eta, oq);
            u0 = ld(d.hu, oq);
            v0 = ld(d.hv, oq);
        }
        const Lo lo = load_lo<STAGE, COMP>(d, c);
        load(C, B, k);
        y_diff(C, B, d);
        float us, vs;
        y_faces(B, C, A.land, c.out, d, us, vs);
        XFaces x = x_faces(A, c, d);
        F3 Gn;
        RowFlux rf;
        if (likely((A.shallowy | B.shallowy | x.shallow) == 0)) {
            if (likely((A.land | B.land) == 0)) row_fluxes<true, false>(A, B, x, us, vs, d, Gn, rf);
            else row_fluxes<true, true>(A, B, x, us, vs, d, Gn, rf);
        } else {
            row_fluxes<false, true>(A, B, x, us, vs, d, Gn, rf);
        }
        // The next row's loads are waited for here, before the stores.  Loads
        // and stores share one in-order counter, and the stores are behind
        // branches: a wait after them has to assume that none was issued, and
        // so drains those that were (1 to 3 % of stage 1).
        arrived(nxt);
        if (STAGE == 2 && unlikely(c.kind & kTileFrs) && c.o - y0 >= kFrsRows && (c.o - y0) % kFrsRows == 0) {
            wave_fence();
            frs_fill_rows(cold(dk), ft, c.x0, c.o, c.lane);
            wave_fence();
        }
        // a row whose output cells are all land has nothing to update
        if ((c.out & ~A.land) != 0)
            finish_row<STAGE, PROJ, W10, COMP>(A, Gs, Gn, rf, c, e0, u0, v0, lo, dk, ft, d, wmax_loc, bad);
        Gs = Gn;
    };
    for (int k = y0 + 2;;) {
        step(R2, R0, R1, k);
        if (++k > klast) break;
        step(R0, R1, R2, k);
        if (++k > klast) break;
        step(R1, R2, R0, k);
        if (++k > klast) break;
    }
}

// ---------------------------------------------------------------------------
// time step of one domain (the same in both stage kernels of a step and in
// every wave): dt from the CFL accumulator of the step's parity (eq. cfl) or a
// given dt, clamped to land on t_end, or the step skipped once t_end is reached
// ---------------------------------------------------------------------------
struct StepTime {
    double tn, dtd;
    double tnext;       // time at the start of the next step
    double hold, tupd;  // dt update policy state after this step
    uint32_t wbits;
    bool skip, last;
};

template <class D>
__device__ __forceinline__ StepTime step_time(const D &d, int parity, double dt_fixed, int lane)
{
    const Ctrl *ctrl = d.ctrl;
    StepTime s;
    s.tn = ctrl->t[parity];
    s.wbits = read_wmax(ctrl, parity, lane);
    const double te = ctrl->t_end;
    s.dtd = dt_fixed > 0.0 ? dt_fixed : (double)(d.courant_q / __uint_as_float(s.wbits));
    // dt update policy: keep the dt of the last update until the update time
    // is reached, then take the CFL dt and move the update time on by one
    // interval (to one interval past t^n if that is not enough)
    s.hold = ctrl->dt_hold[parity];
    s.tupd = ctrl->t_upd[parity];
    if (dt_fixed <= 0.0 && d.dt_interval > 0.0) {
        if (s.hold > 0.0 && s.tn < s.tupd) {
            s.dtd = s.hold;
        } else {
            s.hold = s.dtd;
            s.tupd += d.dt_interval;
            if (s.tupd <= s.tn) s.tupd = s.tn + d.dt_interval;
        }
    }
    s.skip = false;
    s.last = false;
    if (te > 0.0) {
        if (s.tn >= te) s.skip = true;
        else if (s.dtd >= te - s.tn) { s.dtd = te - s.tn; s.last = true; }
    }
    s.tnext = s.last ? te : s.tn + s.dtd;
    return s;
}

// The same step as stage 1 published it (advance_ctrl), read by stage 2: no
// reduction over the 64 slots, and no division.
template <class D>
__device__ __forceinline__ StepTime step_published(const D &d, int parity)
{
    const Ctrl *ctrl = d.ctrl;
    StepTime s;
    s.tn = ctrl->t[parity];
    s.dtd = ctrl->dt_step;
    s.tnext = ctrl->t[parity ^ 1];
    s.skip = ctrl->t_end > 0.0 && s.tn >= ctrl->t_end;
    return s;
}

// Done by one wavefront per domain in stage 1: the slots of the next parity
// are cleared for stage 2 to accumulate into (or, for a step past t_end, get
// the current maximum), and the next time is published.
__device__ __forceinline__ void advance_ctrl(Ctrl *ctrl, const StepTime &s, int parity, int lane)
{
    if (lane < kCflSlots) ctrl->wslot[parity ^ 1][lane][0] = s.skip ? s.wbits : 0u;
    if (lane == 0) {
        // a skipped step keeps the policy state; a step clamped to t_end
        // records the dt it would have taken
        ctrl->dt_hold[parity ^ 1] = s.skip ? ctrl->dt_hold[parity] : s.hold;
        ctrl->t_upd[parity ^ 1] = s.skip ? ctrl->t_upd[parity] : s.tupd;
        if (s.skip) {
            ctrl->t[parity ^ 1] = s.tn;
        } else {
            ctrl->t[parity ^ 1] = s.tnext;
            ctrl->dt_step = s.dtd;
            ctrl->dt_last = (float)s.dtd;
            ctrl->steps += 1;
        }
    }
}

// One tile (wavefront) of one stage:
//   STAGE 1: Q* = (Q^n + dt M(Q^n)) / (1 + dt S(Q^n))               (momenta)
//   STAGE 2: Q^{n+1} = (Q^n + Q* + dt M(Q*)) / 2 / (1 + dt/2 S(Q*))  (momenta)
//            then flow relaxation (eq. frs) and the CFL reduction for the
//            next step (eq. cfl)
// eq. rk2_semiimp; M is eq. sw_semidiscrete with the sources of eq. swe.
template <int STAGE, bool PROJ, bool W10, bool COMP, class D, class T_>
__device__ __forceinline__ void process_tile(const D &d, DomK *dk, FrsTable &ft, const T_ &T, int tile, int parity, double dt_fixed,
                                             bool advance, int lane)
{
    const int nx = d.nx, ny = d.ny;
    int strip, y0, y1;
    tile_place(T, tile, ny, strip, y0, y1);
    const int x0 = strip * kStrip;
    TileCtx c;
    c.i = x0 - kHalo + lane;
    c.lane = lane;
    c.x0 = x0;
    c.o = y0;
    c.out_lane = lane >= kHalo && lane < kWave - kHalo && c.i < nx;
    c.out = __builtin_amdgcn_ballot_w64(c.out_lane);
    c.xneed = c.out | left_in(c.out) | right_in(c.out);
    const TileStart start = load_start<STAGE, PROJ>(d, c.i, y0 - kHalo);
    const WindStart wind = load_wind(d);

    const StepTime st = STAGE == 1 ? step_time(d, parity, dt_fixed, lane) : step_published(d, parity);
    if (STAGE == 1 && advance) advance_ctrl(d.ctrl, st, parity, lane);
    if (st.skip) return;
    const double tau = STAGE == 1 ? st.tn : st.tn + st.dtd;
    c.dt = (float)st.dtd;
    wind_at(d, tau, wind, c.wx, c.wy);
    c.wk = 0;
    c.ws = 0.f;
    if (d.w10n > 0) {
        double s;
        time_weights(d.w10n, d.w10_t, tau, c.wk, s, &wind.t10);
        c.ws = (float)s;
    }

    // edge: some output cell lies within two cells of a side (its values go
    // into the frame too).  frs: some output cell lies within the relaxation
    // zone of a nested side.
    const bool edge = x0 < kHalo || x0 + kStrip > nx - kHalo || y0 < kHalo || y1 > ny - kHalo;
    const int W = d.frs_w;
    bool frs = false;
    if (W > 0) {
        frs |= d.bc[0] == BC_NESTED && x0 < W;
        frs |= d.bc[1] == BC_NESTED && x0 + kStrip > nx - W;
        frs |= d.bc[2] == BC_NESTED && y0 < W;
        frs |= d.bc[3] == BC_NESTED && y1 > ny - W;
    }
    c.kind = __builtin_amdgcn_readfirstlane((edge ? kTileEdge : 0) | (frs ? kTileFrs : 0) |
                                            d.friction << kTileFriction);
    frame_copy_cols(d, c.i, c.fca, c.fcb);
    float wmax_loc = 0.f;
    BadLanes bad{0, 0};
    // one row loop for every tile (a second variant of it in the same kernel
    // raised the register count of both by ~25 VGPRs): the relaxation zone
    // and the frame writes are uniform branches
    // nested frame cells are written for the time of the stage that reads
    // them: stage 2 of this step, or stage 1 of the next
    if (edge && d.nb > 0)
        write_frame_nested<STAGE>(cold(dk), STAGE == 1 ? st.tn + st.dtd : st.tnext, x0, y0, y1, lane);
    if (STAGE == 2 && frs) frs_fill(cold(dk), ft, tau, x0, y0, y1, c.i, lane);
    run_tile<STAGE, PROJ, W10, COMP>(d, dk, ft, c, start, y0, y1, wmax_loc, bad);

    if (STAGE == 2) {
        // at least +0 and no NaN, so its bits are ordered as it is
        const uint32_t wbits = wave_max(__float_as_uint(wmax_loc));
        const uint32_t fl = (bad.nonfinite ? 1u : 0u) | (bad.negative ? 2u : 0u);
        if (lane == 0) {
            atomicMax(&d.ctrl->wslot[parity ^ 1][tile & (kCflSlots - 1)][0], wbits);
            if (fl) atomicOr(&d.ctrl->flags, fl);
        }
    }
}

// ---------------------------------------------------------------------------
// single-domain stage kernel: one wavefront per tile
// ---------------------------------------------------------------------------
template <int STAGE, bool PROJ, bool W10, bool COMP>
__global__ __launch_bounds__(kWave * kWavesPerBlock) void stage_kernel(Dom d, Tiling T, int parity,
                                                                      double dt_fixed)
{
    const int lane = threadIdx.x & (kWave - 1);
    // the same in every lane of the wave: read as a scalar, so that the tile's
    // rows and columns, and with them the row offsets, are scalar values
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    // tile of this wave: head blocks before tail blocks, each part grouped
    // per XCD (neighbouring tiles, which share halo rows, meet in one L2)
    const int b = blockIdx.x;
    const int tile = block_tile(T, b, wid);

    if (tile < 0) return;
    // the domain block is the first kernel argument
    DomK *dk = (DomK *)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ FrsTable ft[kWavesPerBlock];
    process_tile<STAGE, PROJ, W10, COMP>(d, dk, ft[wid], T, tile, parity, dt_fixed, b == 0 && wid == 0, lane);
}

// ---------------------------------------------------------------------------
// ensemble stage kernel: many domains of uneven sizes in one launch.  The work
// items (member, tile) lie in one list, the tall bands of all members before
// the short ones that end the launch; a wave takes `chunk` consecutive items,
// and blocks are grouped per XCD like a single domain's.  The hardware hands
// out the blocks: a persistent grid that drew its items from device queues
// paid an atomic and two more dependent loads before every item, dealt
// neighbouring tiles to different XCDs and ran 16-row bands whatever the size
// (compensated state, us a step, before and now: 3 members of 0.25 M cells
// together 70 and 16, 12 of 3.8 M 137 and 84, 20 of 6.2 M 215 and 145, 48 of
// 13.3 M 434 and 383; float32 state 316 and 259).  Every member has its own
// parameters, time, dt slot and CFL accumulator.
// ---------------------------------------------------------------------------
template <int STAGE, bool PROJ, bool W10, bool COMP>
__global__ __launch_bounds__(kWave * kWavesPerBlock) __attribute__((amdgpu_waves_per_eu((PROJ || W10) ? 1 : 4)))
void ensemble_kernel(const EnsMember *__restrict__ mem, const EnsItem *__restrict__ items, const EnsCtrl *ec, int parity,
                     int chunk)
{
    // member table, items and counts do not change while the kernel runs:
    // through the constant address space they are scalar loads
    using MemberK = const __attribute__((address_space(4))) EnsMember;
    using ItemK = const __attribute__((address_space(4))) EnsItem;
    using CtrlK = const __attribute__((address_space(4))) EnsCtrl;
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    __shared__ FrsTable ft[kWavesPerBlock];
    const CtrlK &C = *(CtrlK *)(uintptr_t)ec;
    const int b = blockIdx.x, n1 = C.nblk1;
    const int at = b < n1 ? xcd_group(b, n1, 0) : n1 + xcd_group(b - n1, (int)gridDim.x - n1, 0);
    const int64_t first = ((int64_t)at * kWavesPerBlock + wid) * chunk;
    for (int64_t j = first; j < first + chunk && j < C.nitems; ++j) {
        const ItemK &it = ((ItemK *)(uintptr_t)items)[j];
        const int tile = it.tile;
        MemberK &M = ((MemberK *)(uintptr_t)mem)[it.member];
        process_tile<STAGE, PROJ, W10, COMP>(M.d, &M.d, ft[wid], M.T, tile, parity ^ M.pflip, 0.0, tile == 0, lane);
    }
}

// ---------------------------------------------------------------------------
// CFL reduction of a given state into the slots of parity `slot` (used at init and
// after a state change); one thread per cell.
// ---------------------------------------------------------------------------
__global__ void cfl_kernel(Dom d, int slot)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    int j = blockIdx.y;
    float w = 0.f;
    int bad = 0;
    if (i < d.nx && j < d.ny) {
        const size_t o = cell_off(d, j, i);
        if (!isnan(d.f[o])) {
            const float *H0 = d.Hc + corner_off(d, j, 0), *H1 = H0 + d.cpitch;
            float Hb = 0.25f * ((H0[i] + H1[i]) + (H0[i + 1] + H1[i + 1]));
            float e = d.eta[o], u = d.hu[o], v = d.hv[o];
            float h = e + Hb;
            float ri = rcp(desing(h, d));
            float c = fsqrt(d.g * fmaxf(h, 0.f));
            w = fmaxf((fabsf(u * ri) + c) * d.rdx, (fabsf(v * ri) + c) * d.rdy);
            if (!(isfinite(e) && isfinite(u) && isfinite(v))) bad |= 1;
            if (h < -d.kappa) bad |= 2;
        }
    }
    w = wave_max_any(w);
    const uint32_t fl = (__ballot(bad & 1) ? 1u : 0u) | (__ballot(bad & 2) ? 2u : 0u);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        int k = (blockIdx.x + blockIdx.y * gridDim.x + (threadIdx.x / kWave)) & (kCflSlots - 1);
        atomicMax(&d.ctrl->wslot[slot][k][0], __float_as_uint(w));
        if (fl) atomicOr(&d.ctrl->flags, fl);
    }
}

// ---------------------------------------------------------------------------
// Frames filled on the host side of the library's calls (init, a new state,
// new boundary data): the static planes (f, north angle, corner depths), and
// the frame of Q^n for the time of the step of a parity.  Afterwards the
// stage kernels keep the state frames current.  Every source is an interior
// cell or corner (col_map / row_map / map_corner), every target a frame cell,
// so no thread reads what another writes.
// ---------------------------------------------------------------------------
__global__ void frame_static_kernel(Dom d)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    const int ncell = frame_cells(d);
    float *f = const_cast<float *>(d.f), *north = const_cast<float *>(d.north), *Hc = const_cast<float *>(d.Hc);
    if (k < ncell) {
        int x, y;
        frame_cell(d, k, x, y);
        const GhostSrc g = ghost_src(d, col_map(d, x), x, y);
        float fv, th = 0.f;
        if (g.side >= 0) {
            const uint32_t q = (uint32_t)g.layer * (uint32_t)d.P + (uint32_t)g.idx;
            fv = d.fghost[q];
            if (north) th = d.nghost[q];
        } else {
            fv = flip_sign(f[g.off], (g.flip << 2) & kSign);
            if (north) th = north[g.off];
        }
        const uint32_t o = cell_off(d, y, x);
        f[o] = fv;
        if (north) north[o] = th;
    } else if (k < ncell + frame_corners(d)) {
        int x, y;
        frame_corner(d, k - ncell, x, y);
        const int cx = map_corner(x, d.nx, d.bc[0], d.bc[1]), cy = map_corner(y, d.ny, d.bc[2], d.bc[3]);
        Hc[corner_off(d, y, x)] = Hc[corner_off(d, cy, cx)];
    }
}

__global__ void frame_state_kernel(Dom d, int parity)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    int bk = 0;
    double t = 0.0;
    if (d.nb > 0) time_weights(d.nb, d.bnd_t, d.ctrl->t[parity], bk, t);  // by whole waves
    if (k >= frame_cells(d)) return;
    int x, y;
    frame_cell(d, k, x, y);
    const GhostSrc g = ghost_src(d, col_map(d, x), x, y);
    float e = 0.f, u = 0.f, v = 0.f;
    if (g.side >= 0) {
        if (d.nb > 0) {  // the interpolation of the stage kernels' boundary loads
            const uint32_t P = (uint32_t)d.P;
            const float *pa = d.bnd + (uint32_t)bk * 3u * P + (uint32_t)g.idx;
            const float *pb = d.nb > 1 ? pa + 3u * P : pa;
            e = (float)((1.0 - t) * (double)pa[0] + t * (double)pb[0]);
            u = (float)((1.0 - t) * (double)pa[P] + t * (double)pb[P]);
            v = (float)((1.0 - t) * (double)pa[2u * P] + t * (double)pb[2u * P]);
        }
    } else {
        e = d.eta[g.off];
        u = flip_sign(d.hu[g.off], g.flip & kSign);
        v = flip_sign(d.hv[g.off], (g.flip << 1) & kSign);
    }
    const uint32_t o = cell_off(d, y, x);
    d.eta[o] = e;
    d.hu[o] = u;
    d.hv[o] = v;
}

// control block set-up: time, CFL slot cleared, flags cleared
__global__ void ctrl_reset_kernel(Ctrl *c, double t, int slot)
{
    if (blockIdx.x == 0 && threadIdx.x < kCflSlots) {
        c->wslot[0][threadIdx.x][0] = 0u;
        c->wslot[1][threadIdx.x][0] = 0u;
        if (threadIdx.x == 0) {
            c->t[slot] = t;
            c->t[slot ^ 1] = t;
            c->flags = 0u;
            c->dt_last = 0.f;
            c->t_end = 0.0;
            c->dt_hold[0] = c->dt_hold[1] = 0.0;
            c->t_upd[0] = c->t_upd[1] = t;
        }
    }
}

// dt update policy restarted at the current time of the given parity
__global__ void ctrl_policy_reset_kernel(Ctrl *c, int parity)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        c->dt_hold[0] = c->dt_hold[1] = 0.0;
        c->t_upd[0] = c->t_upd[1] = c->t[parity];
    }
}

__global__ void ctrl_set_t_end_kernel(Ctrl *c, double te)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) c->t_end = te;
}

// ---------------------------------------------------------------------------
// float64 diagnostics: per-block partial sums in a fixed order, then one
// block adds the partials in order (deterministic).
// ---------------------------------------------------------------------------
constexpr int kDiagThreads = 256;

__global__ __launch_bounds__(kDiagThreads) void diag_partial_kernel(Dom d)
{
    __shared__ double sm[2][kDiagThreads];
    const int j = blockIdx.x;  // one block per row
    double m = 0.0, en = 0.0;
    const double area = d.dx64 * d.dy64;
    for (int i = threadIdx.x; i < d.nx; i += kDiagThreads) {
        const size_t o = cell_off(d, j, i);
        if (isnan(d.f[o])) continue;
        const float *H0 = d.Hc + corner_off(d, j, 0), *H1 = H0 + d.cpitch;
        double Hb = 0.25 * ((double)H0[i] + (double)H0[i + 1] + (double)H1[i] + (double)H1[i + 1]);
        double e = d.eta[o], u = d.hu[o], v = d.hv[o];
        double h = e + Hb;
        double a = fabs(h), kap = d.kappa64;
        double hs = fmax(a, fmin(h * h / (2.0 * kap) + 0.5 * kap, kap));
        hs = h < 0.0 ? -hs : hs;
        m += h * area;
        en += (0.5 * (u * u + v * v) / hs + 0.5 * d.g64 * e * e) * area;
    }
    sm[0][threadIdx.x] = m;
    sm[1][threadIdx.x] = en;
    __syncthreads();
    for (int s = kDiagThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sm[0][threadIdx.x] += sm[0][threadIdx.x + s];
            sm[1][threadIdx.x] += sm[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        d.partials[2 * j] = sm[0][0];
        d.partials[2 * j + 1] = sm[1][0];
    }
}

__global__ __launch_bounds__(kDiagThreads) void diag_final_kernel(Dom d)
{
    __shared__ double sm[2][kDiagThreads];
    double m = 0.0, en = 0.0;
    for (int j = threadIdx.x; j < d.ny; j += kDiagThreads) {
        m += d.partials[2 * j];
        en += d.partials[2 * j + 1];
    }
    sm[0][threadIdx.x] = m;
    sm[1][threadIdx.x] = en;
    __syncthreads();
    for (int s = kDiagThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sm[0][threadIdx.x] += sm[0][threadIdx.x + s];
            sm[1][threadIdx.x] += sm[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        d.ctrl->mass = sm[0][0];
        d.ctrl->energy = sm[1][0];
    }
}

// ---------------------------------------------------------------------------
// launch wrappers (host side)
// ---------------------------------------------------------------------------
// Kernel variants: stage (1, 2) x literal north projection x gridded wind x
// compensated state.  The wind-field and compensated-state code is compiled
// only into their own variants (it would otherwise raise the register count
// of every launch).
template <int S, bool P, bool W, bool C>
hipError_t launch_stage_v(const Dom &d, const Tiling &T, int parity, double dt_fixed, hipStream_t s, hipEvent_t ev0,
                          hipEvent_t ev1)
{
    dim3 grid(T.nblocks), block(kWave * kWavesPerBlock);
    if (ev0) hipExtLaunchKernelGGL(stage_kernel<S, P, W, C>, grid, block, 0, s, ev0, ev1, 0, d, T, parity, dt_fixed);
    else stage_kernel<S, P, W, C><<<grid, block, 0, s>>>(d, T, parity, dt_fixed);
    return hipGetLastError();
}

template <int S, bool P>
hipError_t launch_stage_pc(bool w, bool c, const Dom &d, const Tiling &T, int parity, double dt_fixed,
                           hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    if (c) return w ? launch_stage_v<S, P, true, true>(d, T, parity, dt_fixed, s, ev0, ev1)
                    : launch_stage_v<S, P, false, true>(d, T, parity, dt_fixed, s, ev0, ev1);
    return w ? launch_stage_v<S, P, true, false>(d, T, parity, dt_fixed, s, ev0, ev1)
             : launch_stage_v<S, P, false, false>(d, T, parity, dt_fixed, s, ev0, ev1);
}

hipError_t launch_stage(int stage, bool proj, const Dom &d, const Tiling &T, int parity, double dt_fixed,
                        hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    const bool w = d.w10n > 0, c = d.eta_lo != nullptr;
    if (stage == 1) return proj ? launch_stage_pc<1, true>(w, c, d, T, parity, dt_fixed, s, ev0, ev1)
                                : launch_stage_pc<1, false>(w, c, d, T, parity, dt_fixed, s, ev0, ev1);
    return proj ? launch_stage_pc<2, true>(w, c, d, T, parity, dt_fixed, s, ev0, ev1)
                : launch_stage_pc<2, false>(w, c, d, T, parity, dt_fixed, s, ev0, ev1);
}

// waves per SIMD that one stage kernel variant can keep resident, from its
// register usage (512 VGPRs per SIMD lane on gfx950, 8-register granules)
int waves_of(const void *f)
{
    hipFuncAttributes a{};
    if (hipFuncGetAttributes(&a, f) != hipSuccess || a.numRegs <= 0) return 3;
    int regs = (a.numRegs + 7) / 8 * 8;
    int w = 512 / regs;
    return w < 1 ? 1 : (w > 8 ? 8 : w);
}

int stage_waves_per_simd(int stage, bool proj, bool comp)
{
    const void *f;
    if (stage == 1) f = proj ? (comp ? (const void *)stage_kernel<1, true, false, true> : (const void *)stage_kernel<1, true, false, false>)
                             : (comp ? (const void *)stage_kernel<1, false, false, true> : (const void *)stage_kernel<1, false, false, false>);
    else f = proj ? (comp ? (const void *)stage_kernel<2, true, false, true> : (const void *)stage_kernel<2, true, false, false>)
                  : (comp ? (const void *)stage_kernel<2, false, false, true> : (const void *)stage_kernel<2, false, false, false>);
    return waves_of(f);
}

template <int S, bool P, bool W, bool C>
hipError_t launch_ensemble_v(const EnsMember *mem, const EnsItem *items, EnsCtrl *ec, int parity, int chunk,
                             int nblocks, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    dim3 grid(nblocks), block(kWave * kWavesPerBlock);
    if (ev0)
        hipExtLaunchKernelGGL(ensemble_kernel<S, P, W, C>, grid, block, 0, s, ev0, ev1, 0, mem, items, ec, parity, chunk);
    else ensemble_kernel<S, P, W, C><<<grid, block, 0, s>>>(mem, items, ec, parity, chunk);
    return hipGetLastError();
}

template <int S, bool P>
hipError_t launch_ensemble_pc(bool w, bool c, const EnsMember *mem, const EnsItem *items, EnsCtrl *ec, int parity,
                              int chunk, int nblocks, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1)
{
    if (c) return w ? launch_ensemble_v<S, P, true, true>(mem, items, ec, parity, chunk, nblocks, s, ev0, ev1)
                    : launch_ensemble_v<S, P, false, true>(mem, items, ec, parity, chunk, nblocks, s, ev0, ev1);
    return w ? launch_ensemble_v<S, P, true, false>(mem, items, ec, parity, chunk, nblocks, s, ev0, ev1)
             : launch_ensemble_v<S, P, false, false>(mem, items, ec, parity, chunk, nblocks, s, ev0, ev1);
}

hipError_t launch_ensemble(int stage, bool proj, bool w10, bool comp, const EnsMember *mem, const EnsItem *items,
                           EnsCtrl *ec, int parity, int chunk, int nblocks, hipStream_t s, hipEvent_t ev0,
                           hipEvent_t ev1)
{
    if (stage == 1)
        return proj ? launch_ensemble_pc<1, true>(w10, comp, mem, items, ec, parity, chunk, nblocks, s, ev0, ev1)
                    : launch_ensemble_pc<1, false>(w10, comp, mem, items, ec, parity, chunk, nblocks, s, ev0, ev1);
    return proj ? launch_ensemble_pc<2, true>(w10, comp, mem, items, ec, parity, chunk, nblocks, s, ev0, ev1)
                : launch_ensemble_pc<2, false>(w10, comp, mem, items, ec, parity, chunk, nblocks, s, ev0, ev1);
}

hipError_t launch_cfl(const Dom &d, int slot, hipStream_t s)
{
    dim3 grid((d.nx + 255) / 256, d.ny), block(256);
    cfl_kernel<<<grid, block, 0, s>>>(d, slot);
    return hipGetLastError();
}

hipError_t launch_frame_static(const Dom &d, hipStream_t s)
{
    const int n = frame_cells(d) + frame_corners(d);
    hipLaunchKernelGGL(frame_static_kernel, dim3((n + 255) / 256), dim3(256), 0, s, d);
    return hipGetLastError();
}

hipError_t launch_frame_state(const Dom &d, int parity, hipStream_t s)
{
    const int n = frame_cells(d);
    hipLaunchKernelGGL(frame_state_kernel, dim3((n + 255) / 256), dim3(256), 0, s, d, parity);
    return hipGetLastError();
}

hipError_t launch_ctrl_reset(Ctrl *c, double t, int slot, hipStream_t s)
{
    ctrl_reset_kernel<<<1, 64, 0, s>>>(c, t, slot);
    return hipGetLastError();
}

hipError_t launch_policy_reset(Ctrl *c, int parity, hipStream_t s)
{
    ctrl_policy_reset_kernel<<<1, 64, 0, s>>>(c, parity);
    return hipGetLastError();
}

hipError_t launch_set_t_end(Ctrl *c, double te, hipStream_t s)
{
    ctrl_set_t_end_kernel<<<1, 64, 0, s>>>(c, te);
    return hipGetLastError();
}

hipError_t launch_diagnostics(const Dom &d, hipStream_t s)
{
    diag_partial_kernel<<<d.ny, kDiagThreads, 0, s>>>(d);
    diag_final_kernel<<<1, kDiagThreads, 0, s>>>(d);
    return hipGetLastError();
}

}  // namespace swe
