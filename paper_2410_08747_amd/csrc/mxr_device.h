// mxr_device.h -- per-ray device code for gfx950: counter-based RNG, ray
// state in registers, the component models and the voxel traversal.
//
// One lane carries one ray from the source to the end of the component list
// (paper, section 2.2: rays are independent; every per-ray intermediate is
// local).  Component parameters live in a small device block read with
// wave-uniform (scalar) loads; the only shared writable state is the monitor
// histograms, updated with FP64 atomics (paper, section 2.2.2: the monitor
// arrays are the one structure threads must share).
//
// The library is compiled with -ffp-contract=off: every expression rounds as
// written, so wherever a formula is the same as in an independent
// implementation the two agree bit for bit; FMA is spelled out only in the
// traversal's inner loop.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mxr.h"
#include "mxr_tiles.h"

namespace mxr {

// The device's constant address space, for tables that no kernel writes
// while they are read (in the host pass, where kernel bodies are only
// parsed, it is the ordinary one).
#if defined(__HIP_DEVICE_COMPILE__)
#define MXR_CONSTANT __attribute__((address_space(4)))
#else
#define MXR_CONSTANT
#endif

// The same address, which the compiler takes for another: the constants behind
// it are loaded again where they are used next instead of being held, and
// spilled into vector lanes, in scalar registers.
template <class T>
__device__ __forceinline__ const MXR_CONSTANT T *again(const MXR_CONSTANT T *p) {
    asm volatile("" : "+s"(p));
    return p;
}

constexpr double kHc = 12.398419843320026;  // keV * Angstrom (CODATA 2018)
constexpr double kPi = 3.14159265358979323846;
constexpr double kTwoPi = 2.0 * 3.14159265358979323846;
// log 2 in two parts: its first 32 bits and the rest
constexpr double kLog2Hi = 0x1.62e42fee00000p-1, kLog2Lo = 0x1.a39ef35793c76p-33;
constexpr double kInf = __builtin_huge_val();

enum RayStatus : int32_t { kAlive = 0, kExited = 1, kAbsorbed = 2 };

// Device copy of one component: the caller's parameters plus constants the
// host derives once (aux), the first uniform index it draws, and for a
// monitor its tally slot.
struct DevComp {
    uint32_t type, flags, draw0, slot;
    double pos[3];
    double rot[9];
    double par[16];
    double aux[16];
    const void *data0;
    const void *data1;
    uint64_t n0, n1;
    uint32_t dims[4];
};

struct DevInstr {
    uint32_t ncomp;
    int32_t phantom;  // index of the phantom component or -1
    uint32_t n_mat, n_ebin;
    DevComp c[MXR_MAX_COMPONENTS];
    // the phantom's attenuation table as the kernels stage it in LDS: mu / 10
    // (per mm), energy-major (row e holds every material), n_ebin x n_mat.
    // (After the components, which keep their 16-byte alignment.)
    const double *mu_em;
    // the phantom's brick map: per brick of 4^3 voxels (x fastest, edge bricks
    // cut off by the volume) its material, or 255 if it holds several
    const uint8_t *bricks;
};

struct TallyPtrs {
    unsigned long long *count[MXR_MAX_DETECTORS];
    double *sum_w[MXR_MAX_DETECTORS];
    double *sum_w2[MXR_MAX_DETECTORS];
};

// Proposal mixture of a cone-beam source, prepared on the host from the
// caller's 8 x (pi, mu[3], sigma[3]) table: per component the normal
// distribution function (P) and its upper tail (Q) at the box edges, in
// standard units, the box masses pi_k Z_k, and the prefactor of the
// component's own truncated density, 1 / (sigma_u sigma_v sigma_E
// (2 pi)^(3/2) F_k) with F_k its box mass without pi_k (0 for an empty
// component).
struct PropTable {
    double kcoef[8];
    double mu[8][3], sigma[8][3], inv_sigma[8][3];
    double Pa[8][3], Pb[8][3], Qa[8][3], Qb[8][3];
    double mass[8];
    double norm;       // sum_k pi_k Z_k
    double alpha;      // share of the plain source in the mixture
    double t2;         // tan^2 of the cone half-angle
    double inv_omega;  // 1 / solid angle of the cone
    double lo[3], hi[3];
};

// Where a hit-collecting run writes the rays that reach a monitor.
struct HitSink {
    float *ctx;                  // n x 6
    double *y;                   // n x 3: u = dx/dz, v = dy/dz (source frame), E
    double *w;                   // n
    int64_t *bin;                // n
    unsigned long long *count;   // rows written (may exceed capacity: then truncated)
    uint64_t capacity;
    float c[6];                  // context of this run
};

// Divisors of a stratified range of n rays over G x G cells, prepared on the
// host: ray i of the range lies in cell floor(i G^2 / n), and a cell holds
// c0 = floor(n / G^2) or c0 + 1 rays (r = n mod G^2 of the cells hold one
// more), so the cell factor (n / G^2) / count takes one of the two values f0
// and f1, each the same division the factor is defined by.  rn, rG and rG2
// are 1/n, 1/G and 1/G^2 rounded, for the quotient estimates.
struct StratDiv {
    uint64_t n, G2, c0, r;
    uint32_t G, pad;
    double rn, rG, rG2, f0, f1;
};

// The tiles of a launch of the image kernels: 256 << rounds rays each, the
// ranges' tiles one after the other.
struct TilePlan {
    uint64_t first_tile, tiles;  // of this launch, of the whole run
    uint32_t rounds, ranges;
    // the work-group's private histogram: 2^lx x 2^ly pixels of lds_ne energy
    // bins (0: none)
    uint32_t lx, ly, lds_ne;
    uint32_t cull;               // the one range is a whole stratified cone: tiles that miss the monitor end at once
    TileRange r[9];
};

struct RunArgs {
    const DevInstr *ins;
    uint64_t first, n, n_total, seed;
    uint64_t G, G2;  // strata per side used, and its square
    StratDiv sd;     // the same strata's divisors
    uint32_t word3;  // purpose << 24 | job
    uint32_t blocks_per_xcd;
    uint32_t compact_rounds;  // compacting kernel: 64-ray rounds per wave
    uint32_t xcd_order;       // tiles per XCD: 0 the x-th eighth of the range, 1 launch order, 2 runs of 64 tiles
    TallyPtrs tally;
    double *ledger;
    const uint64_t *ids;  // trace mode: ray ids
    mxr_ray_soa dump;     // trace mode: outputs
    const PropTable *prop;  // proposal of the cone-beam source, or null
    // proposal runs: branch b (plain, then components 0..7) takes ray ids
    // [pb[b], pb[b+1]) (pb[0] = 0 is implicit: pb here holds the 9 upper
    // bounds), stratified over psd[b].G^2 cells; pc[b] = its share of the rays
    uint64_t pb[9];
    StratDiv psd[9];
    double pc[9];
    HitSink hits;  // hit-collecting runs
    TilePlan tp;   // tiled launches (the image kernels)
};

// ------------------------------------------------------------- Philox ----
// Philox4x32-10 (Salmon et al., SC'11).  The 32x32->64 products map to
// v_mad_u64_u32, the two exclusive ors of a word to one v_bitop3_b32.
struct Philox {
    uint32_t k0, k1, c1, c2, c3;

    __device__ __forceinline__ void block(uint32_t j, uint32_t out[4]) const {
        uint32_t x0 = j, x1 = c1, x2 = c2, x3 = c3, a = k0, b = k1;
        // the round keys are added up (in scalar registers) for each block: kept
        // for a whole kernel they end up in lanes of a vector register
#pragma unroll
        for (int r = 0; r < 10; ++r) {
            uint64_t pa = (uint64_t)0xD2511F53u * x0;
            uint64_t pb = (uint64_t)0xCD9E8D57u * x2;
            const uint32_t y0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), x1, a, 0x96);
            const uint32_t y2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), x3, b, 0x96);
            x1 = (uint32_t)pb;
            x3 = (uint32_t)pa;
            x0 = y0;
            x2 = y2;
            a += 0x9E3779B9u;
            b += 0xBB67AE85u;
        }
        out[0] = x0; out[1] = x1; out[2] = x2; out[3] = x3;
    }
};

// ((w >> 12) + 1/2) 2^-52 of the 64-bit word w: 1 + (w >> 12) 2^-52 by its bits,
// less 1 - 2^-53 (exact: the result has 53 bits).
__device__ __forceinline__ double u01(uint32_t lo, uint32_t hi) {
    const uint64_t w = ((uint64_t)hi << 32) | lo;
    return __longlong_as_double((long long)((w >> 12) | 0x3FF0000000000000ull)) - 0x1.fffffffffffffp-1;
}

// Uniforms of one ray, produced two at a time on demand.
struct Stream {
    Philox ph;
    int blk;
    uint32_t w[4];

    __device__ __forceinline__ void init(uint64_t seed, uint64_t ray, uint32_t word3) {
        ph.k0 = (uint32_t)seed;
        ph.k1 = (uint32_t)(seed >> 32);
        ph.c1 = (uint32_t)ray;
        ph.c2 = (uint32_t)(ray >> 32);
        ph.c3 = word3;
        blk = -1;
    }
    __device__ __forceinline__ double u(int index) {
        int b = index >> 1;
        if (b != blk) {
            ph.block((uint32_t)b, w);
            blk = b;
        }
        return (index & 1) ? u01(w[2], w[3]) : u01(w[0], w[1]);
    }
};

// ---------------------------------------------------------------- ray ----
struct Ray {
    double r[3], d[3];
    double E, w;
};

__device__ __forceinline__ void to_local(const DevComp &c, const Ray &ray, double q[3], double dl[3]) {
    double v0 = ray.r[0] - c.pos[0], v1 = ray.r[1] - c.pos[1], v2 = ray.r[2] - c.pos[2];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double *R = c.rot + 3 * i;
        q[i] = R[0] * v0 + R[1] * v1 + R[2] * v2;
        dl[i] = R[0] * ray.d[0] + R[1] * ray.d[1] + R[2] * ray.d[2];
    }
}

__device__ __forceinline__ void to_lab(const DevComp &c, const double q[3], const double dl[3], Ray &ray) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ray.r[i] = c.rot[i] * q[0] + c.rot[3 + i] * q[1] + c.rot[6 + i] * q[2] + c.pos[i];
        ray.d[i] = c.rot[i] * dl[0] + c.rot[3 + i] * dl[1] + c.rot[6 + i] * dl[2];
    }
}

// A ray leaving the component's origin: position pos, direction R dl (what
// to_lab gives for q = 0, since R 0 + pos = pos for a finite rotation).
__device__ __forceinline__ void from_origin(const DevComp &c, const double dl[3], Ray &ray) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ray.r[i] = c.pos[i];
        ray.d[i] = c.rot[i] * dl[0] + c.rot[3 + i] * dl[1] + c.rot[6 + i] * dl[2];
    }
}

__device__ __forceinline__ bool plane_z0(double q[3], const double dl[3]) {
    if (!(dl[2] > 0.0)) return false;
    double t = -q[2] / dl[2];
    if (!(t >= 0.0)) return false;
    q[0] = q[0] + t * dl[0];
    q[1] = q[1] + t * dl[1];
    q[2] = 0.0;
    return true;
}

// ------------------------------------------- functions of known ranges ----
// The library's sqrt, log, sincos and division take any argument: scaling of
// subnormals, reductions of huge angles, infinities.  Where the range is known
// (uniforms, unit vectors, values near 1) the forms below leave that out, at the
// same accuracy (about an ulp of the exact result).  Instructions for 64 rays of
// the lens instrument 1609 -> 1220 and of the beamline 2000 -> 1620, both bound
// by VALU issue: 1e8 rays 4.45 -> 3.26 ms and 5.04 -> 4.20 ms.  (A polynomial
// asin for the mirror and the crystals gave the beamline less than 1 %.)

// 1 / d, d positive or negative and normal with a normal reciprocal: two Newton
// steps from the hardware's estimate (about 23 bits).
__device__ __forceinline__ double rcp_normal(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
}
// a / d from r = rcp_normal(d), corrected by its remainder: the rounded quotient.
__device__ __forceinline__ double div_normal(double a, double d, double r) {
    const double q = a * r;
    return fma(fma(-d, q, a), r, q);
}
// sqrt(x), x normal and positive: one coupled Newton step for the root and
// half its reciprocal, then the root's remainder.
__device__ __forceinline__ double sqrt_normal(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}

// sqrt(x) of a finite x >= 0, and 1 / sqrt(x) of a normal one (a second step for
// the reciprocal).
__device__ __forceinline__ double sqrt_finite(double x) {
    const double r = sqrt_normal(x);
    return x > 0.0 ? r : 0.0;
}
__device__ __forceinline__ double rsqrt_normal(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    h = fma(h, fma(-g, h, 0.5), h);
    return h + h;
}

// log(u), 0 < u < 1 normal, by the published reduction to [sqrt(1/2), sqrt 2) and
// the atanh series (W. J. Cody and W. Waite, Software Manual for the Elementary
// Functions, 1980, which also splits log 2; the last additions in the order of
// fdlibm's log, Sun Microsystems, 1993): u = 2^k m, f = m - 1 (exact), s = f / (2 + f), log(1 + f) = 2 atanh(s) = f - f^2/2 + s (f^2/2 + R)
// with the series R = 2 (s^2/3 + s^4/5 + ...) (|s| < 0.172: the first term left
// out is below 2e-18), added smallest first to k log 2 in two parts (the first
// of 32 bits, so that its multiples are exact).
__device__ __forceinline__ double log_unit(double u) {
    double m = __builtin_amdgcn_frexp_mant(u);
    int k = __builtin_amdgcn_frexp_exp(u);
    const bool low = m < 0.70710678118654752;
    m = low ? m + m : m;
    k = low ? k - 1 : k;
    const double f = m - 1.0, s = f * rcp_normal(2.0 + f), z = s * s, half = 0.5 * (f * f), kd = (double)k;
    double R = 2.0 / 21.0;
    R = fma(z, R, 2.0 / 19.0);
    R = fma(z, R, 2.0 / 17.0);
    R = fma(z, R, 2.0 / 15.0);
    R = fma(z, R, 2.0 / 13.0);
    R = fma(z, R, 2.0 / 11.0);
    R = fma(z, R, 2.0 / 9.0);
    R = fma(z, R, 2.0 / 7.0);
    R = fma(z, R, 2.0 / 5.0);
    R = fma(z, R, 2.0 / 3.0);
    const double lo = fma(kd, kLog2Lo, s * fma(z, R, half));
    return fma(kd, kLog2Hi, -((half - lo) - f));
}

// sin y and cos y for |y| <= pi/4 from their Maclaurin series through y^17
// and y^18 (the first omitted terms, y^19/19! and y^20/20!, are below 1e-19
// there), evaluated by Horner's rule in fused multiply-adds.
__device__ __forceinline__ void sincos_quarter(double y, double &sn, double &cs) {
    const double y2 = y * y;
    double p = -1.0 / 355687428096000.0;
    p = fma(y2, p, 1.0 / 1307674368000.0);
    p = fma(y2, p, -1.0 / 6227020800.0);
    p = fma(y2, p, 1.0 / 39916800.0);
    p = fma(y2, p, -1.0 / 362880.0);
    p = fma(y2, p, 1.0 / 5040.0);
    p = fma(y2, p, -1.0 / 120.0);
    p = fma(y2, p, 1.0 / 6.0);
    sn = fma(-(y * y2), p, y);
    double q = 1.0 / 6402373705728000.0;
    q = fma(y2, q, -1.0 / 20922789888000.0);
    q = fma(y2, q, 1.0 / 87178291200.0);
    q = fma(y2, q, -1.0 / 479001600.0);
    q = fma(y2, q, 1.0 / 3628800.0);
    q = fma(y2, q, -1.0 / 40320.0);
    q = fma(y2, q, 1.0 / 720.0);
    q = fma(y2, q, -1.0 / 24.0);
    q = fma(y2, q, 0.5);
    cs = fma(-y2, q, 1.0);
}

// sin and cos of 2 pi u, 0 <= u < 1: the nearest quarter turn taken off exactly.
__device__ __forceinline__ void sincos_turn(double u, double &sn, double &cs) {
    const double k = rint(4.0 * u);
    double a, b;
    sincos_quarter(kTwoPi * fma(k, -0.25, u), a, b);
    const int n = (int)k;
    const double c0 = n & 1 ? b : a, c1 = n & 1 ? a : b;
    sn = n & 2 ? -c0 : c0;
    cs = (n + 1) & 2 ? -c1 : c1;
}

// ------------------------------------------------------------ sources ----
// Square emitter, cone uniform in solid angle: with s = sqrt(U) sin(a/2) =
// sin(theta/2), sin(theta) = 2 s sqrt(1 - s^2) and cos(theta) = 1 - 2 s^2,
// free of the cancellation of 1 - cos at small angles.
__device__ __forceinline__ void src_rect_cone(const DevComp &c, Stream &s, Ray &ray) {
    double q[3], dl[3];
    q[0] = (s.u(0) - 0.5) * c.par[0];
    q[1] = (s.u(1) - 0.5) * c.par[1];
    q[2] = 0.0;
    double sh = sqrt_normal(s.u(2)) * c.aux[0];
    double ch = sqrt(1.0 - sh * sh);
    double sinp, cosp;
    sincos_turn(s.u(3), sinp, cosp);
    double st = 2.0 * sh * ch;
    dl[0] = st * cosp;
    dl[1] = st * sinp;
    dl[2] = 1.0 - 2.0 * (sh * sh);
    ray.E = c.par[3] + c.aux[1] * s.u(4);
    ray.w = 1.0;
    to_lab(c, q, dl, ray);
}

// Tube spectrum (section 3.4's source: Kramers continuum plus two Gaussian
// lines), per keV and normalised; the constant divisors come as host-side
// reciprocals and quotients: aux[4] = 1/sigma, aux[5] = 1/(sigma sqrt(2 pi)),
// aux[6] = continuum weight / continuum integral.
__device__ __forceinline__ double spectrum(const DevComp &c, double E) {
    double z1 = (E - c.par[5]) * c.aux[4];
    double z2 = (E - c.par[7]) * c.aux[4];
    double g1 = exp(-0.5 * z1 * z1) * c.aux[5];
    double g2 = exp(-0.5 * z2 * z2) * c.aux[5];
    return c.aux[6] * ((c.par[3] - E) / E) + c.par[6] * g1 + c.par[8] * g2;
}

// The same as div_est for 32 bits.
__device__ __forceinline__ uint32_t div_est32(uint32_t x, uint32_t d, double rd, uint32_t q_max) {
    uint32_t q = (uint32_t)((double)x * rd);
    q = q > q_max ? q_max : q;
    const uint32_t p = q * d;
    if (p > x) q -= 1;
    else if (x - p >= d) q += 1;
    return q;
}

// Cell (cx, cy) of ray i of a stratified range and its factor (n / G^2) /
// count.  cell = floor(i G^2 / n) < G^2 <= 2^32; the count is c0 plus the
// difference of ceil(j r / G^2) at the cell's two ends (its first ray is
// ceil(cell n / G^2) = cell c0 + ceil(cell r / G^2)).
struct StratCell {
    uint32_t cx, cy;
    double factor;
};
__device__ __forceinline__ StratCell strat_cell(const StratDiv &s, uint64_t i) {
    const uint64_t cell = div_est(i * s.G2, s.n, s.rn, s.G2 - 1);
    const uint32_t cy = div_est32((uint32_t)cell, s.G, s.rG, s.G - 1);
    const uint32_t cx = (uint32_t)cell - cy * s.G;
    uint64_t count = s.c0;
    if (s.r != 0)
        count += div_est((cell + 1) * s.r + s.G2 - 1, s.G2, s.rG2, s.G2 - 1) -
                 div_est(cell * s.r + s.G2 - 1, s.G2, s.rG2, s.G2 - 1);
    return {cx, cy, count == s.c0 ? s.f0 : s.f1};
}

// Concentric map of (ca, cb) in [-1, 1]^2 onto the unit disk: radius rad
// and the angle's sine and cosine.  The angle is (pi/4) x with x = cb/ca,
// or pi/2 - (pi/4) x with x = ca/cb, |x| <= 1; both come from sin and cos
// of y = (pi/4) x (swapped for the second form).
__device__ __forceinline__ void concentric(double ca, double cb, double &rad, double &sa, double &cs) {
    double y = 0.0;
    bool swap = false;
    if (ca == 0.0 && cb == 0.0) {
        rad = 0.0;
    } else if (fabs(ca) > fabs(cb)) {
        rad = ca;
        y = (kPi / 4.0) * div_normal(cb, ca, rcp_normal(ca));
    } else {
        rad = cb;
        y = (kPi / 4.0) * div_normal(ca, cb, rcp_normal(cb));
        swap = true;
    }
    double sn, cn;
    sincos_quarter(y, sn, cn);
    sa = swap ? cn : sn;
    cs = swap ? sn : cn;
}

// Cone-beam point source, stratified: ray r lies in cell floor(r G^2 / N);
// the cell's square is mapped to the unit disk by the concentric map and the
// disk radius rho to the cone by sin(theta/2) = rho sin(alpha/2).  Then
// (dx, dy) = sin(theta) (px, py) / rho = 2 sin(alpha/2) cos(theta/2) (px, py).
// In two parts: the direction (returning the cell's weight factor), and the
// energy and weight, which a ray that ends before them never needs.
__device__ __forceinline__ double cone_direction(const DevComp &c, Stream &s, Ray &ray, uint64_t ray_id,
                                                 const RunArgs &a) {
    const StratCell sc = strat_cell(a.sd, ray_id);
    double u = ((double)sc.cx + s.u(0)) * a.sd.rG;
    double v = ((double)sc.cy + s.u(1)) * a.sd.rG;
    double ca = 2.0 * u - 1.0, cb = 2.0 * v - 1.0;
    double rad, sa, cs;
    concentric(ca, cb, rad, sa, cs);
    double px = rad * cs, py = rad * sa;
    double sh = fabs(rad) * c.aux[0];
    double ch = sqrt(1.0 - sh * sh);
    double k = 2.0 * c.aux[0] * ch;
    double dl[3] = {k * px, k * py, 1.0 - 2.0 * (sh * sh)};
    from_origin(c, dl, ray);
    return sc.factor;
}
__device__ __forceinline__ void cone_energy(const DevComp &c, Stream &s, Ray &ray, double factor) {
    ray.E = c.par[1] + c.aux[1] * s.u(2);
    ray.w = (c.aux[1] * spectrum(c, ray.E)) * factor;
}
__device__ __forceinline__ void src_cone_beam(const DevComp &c, Stream &s, Ray &ray, uint64_t ray_id,
                                              const RunArgs &a) {
    const double factor = cone_direction(c, s, ray, ray_id, a);
    cone_energy(c, s, ray, factor);
}

// Standard normal truncated to [za, zb] by inversion: the point leaving
// mass U of the interval below it, written as a lower-tail probability
// Pa + U (Pb - Pa) when that is at most 1/2 and as the upper-tail
// probability Qb + (1 - U)(Qa - Qb) otherwise, so that no probability near 1
// is inverted.  Phi^-1(p) = -sqrt(2) erfcinv(2p).
__device__ __forceinline__ double trunc_normal(double Pa, double Pb, double Qa, double Qb, double U) {
    const double pl = Pa + U * (Pb - Pa);
    const bool low = pl <= 0.5;
    // one inversion for both sides: a wave's energies fall on either
    const double z = 1.4142135623730951 * erfcinv(2.0 * (low ? pl : Qb + (1.0 - U) * (Qa - Qb)));
    return low ? -z : z;
}

// Cone-beam point source drawing y = (u, v, E), u = dx/dz, v = dy/dz, from
// the proposal as a stratified deterministic mixture: the run's ray ids are
// split into contiguous ranges, one per branch (the plain source, then the 8
// truncated-normal components, sized by alpha and the box masses); within its
// range a ray's first two uniforms are stratified over G x G cells like the
// plain source, so the rays of a wave leave in neighbouring directions.  The
// plain branch maps the pair to the cone (concentric map), a component
// inverts a truncated normal per coordinate (E from the third uniform).  The
// weight is p(y) over the realised mixture density sum_b (n_b / n) q_b(y)
// (balance heuristic: unbiased for any split) times the cell factor.  A draw
// outside the cone gets weight 0 and the source returns false.
__device__ __forceinline__ bool src_cone_proposal(const DevComp &c, const PropTable *__restrict__ P, Stream &s,
                                                  Ray &ray, uint64_t ray_id, const RunArgs &a) {
    int branch = -1;
    uint64_t start = 0;
    if (ray_id >= a.pb[0]) {
        for (int k = 0; k < 8; ++k) {
            if (ray_id < a.pb[k + 1]) {
                branch = k;
                start = a.pb[k];
                break;
            }
        }
    }
    const StratDiv &sd = a.psd[branch + 1];
    const StratCell sc = strat_cell(sd, ray_id - start);
    const double factor = sc.factor;
    const double su = ((double)sc.cx + s.u(0)) * sd.rG;
    const double sv = ((double)sc.cy + s.u(1)) * sd.rG;
    double y[3];
    if (branch < 0) {
        double ca = 2.0 * su - 1.0, cb = 2.0 * sv - 1.0;
        double rad, sa, cs;
        concentric(ca, cb, rad, sa, cs);
        double sh = fabs(rad) * c.aux[0];
        double ch = sqrt(1.0 - sh * sh);
        double k = 2.0 * c.aux[0] * ch;
        double dz = 1.0 - 2.0 * (sh * sh);
        y[0] = (k * (rad * cs)) / dz;
        y[1] = (k * (rad * sa)) / dz;
        y[2] = c.par[1] + c.aux[1] * s.u(2);
    } else {
        const double U[3] = {su, sv, s.u(2)};
        for (int d = 0; d < 3; ++d) {
            double z = trunc_normal(P->Pa[branch][d], P->Pb[branch][d], P->Qa[branch][d], P->Qb[branch][d], U[d]);
            y[d] = P->mu[branch][d] + P->sigma[branch][d] * z;
        }
    }
    const double r2 = y[0] * y[0] + y[1] * y[1];
    const bool in_cone = r2 <= P->t2 && y[2] >= P->lo[2] && y[2] <= P->hi[2];
    const bool in_box = y[0] >= P->lo[0] && y[0] <= P->hi[0] && y[1] >= P->lo[1] && y[1] <= P->hi[1] &&
                        y[2] >= P->lo[2] && y[2] <= P->hi[2];
    // the Jacobian (1 + r2)^(-3/2) of the map from (u, v) to directions, from
    // the square root the direction needs anyway (pow would cost ~200
    // instructions per ray; the two forms differ by a few units in the last
    // place)
    const double w2 = 1.0 + r2;
    const double n = sqrt_normal(w2), w3 = w2 * n;
    const double J = div_normal(1.0, w3, rcp_normal(w3));
    double q = in_cone ? a.pc[0] * (J * P->inv_omega * c.aux[7]) : 0.0;
    if (in_box) {
        for (int k = 0; k < 8; ++k) {
            if (a.pc[k + 1] == 0.0) continue;
            double zu = (y[0] - P->mu[k][0]) * P->inv_sigma[k][0];
            double zv = (y[1] - P->mu[k][1]) * P->inv_sigma[k][1];
            double ze = (y[2] - P->mu[k][2]) * P->inv_sigma[k][2];
            q += a.pc[k + 1] * (P->kcoef[k] * exp(-0.5 * (zu * zu + zv * zv + ze * ze)));
        }
    }
    const double p_phys = in_cone ? spectrum(c, y[2]) * J * P->inv_omega : 0.0;
    const double rn = rcp_normal(n);
    double dl[3] = {div_normal(y[0], n, rn), div_normal(y[1], n, rn), div_normal(1.0, n, rn)};
    ray.E = y[2];
    ray.w = p_phys > 0.0 ? (p_phys / q) * factor : 0.0;
    from_origin(c, dl, ray);
    return p_phys > 0.0;
}

// tan(x): for |x| < 2^-7 the Maclaurin series x + x^3/3 + 2x^5/15 +
// 17x^7/315 + 62x^9/2835 (the first omitted term is below 1e-23 of x there),
// else the library tan.  Beam divergences are micro- to milliradians, so a
// wave normally skips the library call and its argument reduction.
__device__ __forceinline__ double tan_small(double x) {
    if (fabs(x) < 0.0078125) {
        const double x2 = x * x;
        const double p = 1.0 / 3.0 + x2 * (2.0 / 15.0 + x2 * (17.0 / 315.0 + x2 * (62.0 / 2835.0)));
        return x + x * (x2 * p);
    }
    return tan(x);
}

__device__ __forceinline__ void src_gaussian(const DevComp &c, Stream &s, Ray &ray) {
    double r1 = sqrt_normal(-2.0 * log_unit(s.u(0)));
    double s1, c1, s2, c2;
    sincos_turn(s.u(1), s1, c1);
    double r2 = sqrt_normal(-2.0 * log_unit(s.u(2)));
    sincos_turn(s.u(3), s2, c2);
    double q[3], dl[3];
    q[0] = c.par[0] * (r1 * c1);
    q[1] = c.par[1] * (r1 * s1);
    q[2] = 0.0;
    double tx = tan_small(c.par[2] * (r2 * c2));
    double ty = tan_small(c.par[3] * (r2 * s2));
    // (at most 1e18, where tan ends: nrm and its reciprocal are normal)
    const double nrm = sqrt_normal(tx * tx + ty * ty + 1.0), rn = rcp_normal(nrm);
    dl[0] = div_normal(tx, nrm, rn);
    dl[1] = div_normal(ty, nrm, rn);
    dl[2] = div_normal(1.0, nrm, rn);
    ray.E = c.par[4] * ((1.0 - c.par[5]) + 2.0 * c.par[5] * s.u(4));
    ray.w = 1.0;
    to_lab(c, q, dl, ray);
}

// ---------------------------------------------------------- apertures ----
__device__ __forceinline__ bool comp_slit(const DevComp &c, Ray &ray) {
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    if (!plane_z0(q, dl)) return false;
    if (c.flags & 1u) {
        if (!(q[0] * q[0] + q[1] * q[1] <= c.aux[2])) return false;
    } else {
        if (!(fabs(q[0]) <= c.aux[0] && fabs(q[1]) <= c.aux[1])) return false;
    }
    to_lab(c, q, dl, ray);
    return true;
}

__device__ __forceinline__ void comp_box(const DevComp &c, Ray &ray) {
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    double a_in = 0.0, a_out = kInf;
    bool miss = false;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double h = c.par[i];
        if (dl[i] == 0.0) {
            if (!(q[i] > -h && q[i] < h)) miss = true;
        } else {
            double inv = 1.0 / dl[i];
            double a0 = (-h - q[i]) * inv, a1 = (h - q[i]) * inv;
            double lo = a0 < a1 ? a0 : a1, hi = a0 < a1 ? a1 : a0;
            if (lo > a_in) a_in = lo;
            if (hi < a_out) a_out = hi;
        }
    }
    double L = (!miss && a_out > a_in) ? a_out - a_in : 0.0;
    double E = ray.E;
    double mu = c.par[3] / (E * E * E) + c.par[4];
    ray.w = ray.w * exp(-(mu * L) / 10.0);
}

// --------------------------------------------------------------- lens ----
// Compound refractive lens (section 3.2): N identical bi-concave parabolic
// lenses; lens k (centre c_k = (k - (N-1)/2) p on the local z axis) holds
// material between z = c_k - w/2 - rho^2/2R and z = c_k + w/2 + rho^2/2R
// inside the aperture radius.  Per surface: the intersection quadratic's
// root nearest -C/B in the stable form C / q', the aperture test, the unit
// normal into the next medium, and Snell's law in vector form with the
// normal coefficient sqrt(k) - eta cos_i written as
// (1 - eta^2) / (sqrt(k) + eta cos_i) (no cancellation; 1 - eta^2 comes
// in closed form from delta).  The path inside the material is summed and
// the weight attenuated once.  S = -1 front surface, +1 back surface.
template <int S>
__device__ __forceinline__ bool lens_surface(double q[3], double dl[3], double z0, double inv_R, double inv_2R,
                                             double ra2, double eta, double one_m_eta2, double &t_out) {
    const double A = (double)(-S) * ((dl[0] * dl[0] + dl[1] * dl[1]) * inv_2R);
    const double B = dl[2] - (double)S * ((q[0] * dl[0] + q[1] * dl[1]) * inv_R);
    const double C = (q[2] - z0) - (double)S * ((q[0] * q[0] + q[1] * q[1]) * inv_2R);
    const double disc = B * B - 4.0 * A * C;
    if (!(disc >= 0.0)) return false;
    const double qq = -0.5 * (B + copysign(sqrt_finite(disc), B));
    if (qq == 0.0) return false;
    const double t = div_normal(C, qq, rcp_normal(qq));
    if (!(t >= 0.0)) return false;
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = q[i] + t * dl[i];
    if (q[0] * q[0] + q[1] * q[1] > ra2) return false;
    const double g0 = (double)(-S) * (q[0] * inv_R), g1 = (double)(-S) * (q[1] * inv_R);
    const double inv_gn = rsqrt_normal(g0 * g0 + g1 * g1 + 1.0);
    const double m0 = g0 * inv_gn, m1 = g1 * inv_gn, m2 = inv_gn;
    const double cos_i = dl[0] * m0 + dl[1] * m1 + dl[2] * m2;
    if (!(cos_i > 0.0)) return false;
    const double k = 1.0 - eta * eta * (1.0 - cos_i * cos_i);
    if (!(k >= 0.0)) return false;
    const double den = sqrt_finite(k) + eta * cos_i;
    const double gc = div_normal(one_m_eta2, den, rcp_normal(den));
    dl[0] = eta * dl[0] + gc * m0;
    dl[1] = eta * dl[1] + gc * m1;
    dl[2] = eta * dl[2] + gc * m2;
    t_out = t;
    return true;
}

// aux: 0 1/R, 1 1/(2R), 2 aperture radius^2
__device__ __forceinline__ bool comp_lens(const DevComp &c, Ray &ray) {
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    const double inv_R = c.aux[0], inv_2R = c.aux[1], ra2 = c.aux[2];
    const double w = c.par[2], pitch = c.par[3];
    const int N = (int)c.par[1];
    const double E = ray.E;
    const double er = c.par[6] / E;
    const double delta = c.par[5] * (er * er);
    const double mu = c.par[7] / (E * E * E) + c.par[8];
    const double eta_in = 1.0 / (1.0 - delta), eta_out = 1.0 - delta;
    const double ome_in = -delta * (2.0 - delta) / ((1.0 - delta) * (1.0 - delta));
    const double ome_out = delta * (2.0 - delta);
    const double half_n1 = 0.5 * (double)(N - 1);
    double L = 0.0, t;
    for (int k = 0; k < N; ++k) {
        const double ck = ((double)k - half_n1) * pitch;
        if (!lens_surface<-1>(q, dl, ck - 0.5 * w, inv_R, inv_2R, ra2, eta_in, ome_in, t)) return false;
        if (!lens_surface<1>(q, dl, ck + 0.5 * w, inv_R, inv_2R, ra2, eta_out, ome_out, t)) return false;
        L = L + t;
    }
    ray.w = ray.w * exp(-(mu * L) / 10.0);
    to_lab(c, q, dl, ray);
    return true;
}

// ------------------------------------------------------------ phantom ----
// Exact radiological path through the voxel grid.
//
// The ray is walked along its dominant axis D (largest |d|): every step
// crosses one D plane; with cubic voxels and |d_A|, |d_B| <= |d_D| at most
// one plane of each other axis lies between two D planes, so those rarer
// crossings are taken in a branch that coherent waves mostly skip.  Every
// crossing parameter is a fixed function of the exact plane coordinate
// (fma(plane, inv, -q inv), or (plane - q) inv, with inv = 1/d and q fixed
// per ray and axis), so a plane's alpha is the same number in whatever order
// the planes are visited and in the set-up that finds the first plane
// (negative directions are mirrored so every axis steps by +v, which
// leaves both forms unchanged).  The optical depth is accumulated per material run:
// segment lengths between crossings telescope, so a run of voxels of one
// material adds mu * (alpha_end - alpha_start) -- the same sum of
// mu * length as segment by segment, up to rounding -- and the mu table is
// read only where the material changes.  Voxels are read with buffer loads
// (hardware range check: an out-of-range offset reads 0 instead of
// faulting).  The walk is bounded by nx + ny + nz + 3 steps.
#ifndef MXR_WALK_ROUND
#define MXR_WALK_ROUND 4
#endif
#ifndef MXR_LOCATE_ROUND
#define MXR_LOCATE_ROUND 3
#endif
constexpr int kWalkRound = MXR_WALK_ROUND;      // crossings per round of loads
constexpr int kLocateRound = MXR_LOCATE_ROUND;  // the same for the locate walks

struct PhantomGeo {
    const uint8_t *vol;
    uint32_t nvox;
    int n[3];
    double v, rv;  // voxel edge and its reciprocal
    double corner[3];
    // the occupied box: every voxel outside the planes blo[i] .. bhi[i] holds
    // material bg; box = false when every voxel does
    double blo[3], bhi[3];
    uint32_t bg;
    bool box;
};

__device__ __forceinline__ PhantomGeo phantom_geo(const DevComp &c) {
    PhantomGeo g;
    g.vol = (const uint8_t *)c.data0;
    g.n[0] = (int)c.dims[0];
    g.n[1] = (int)c.dims[1];
    g.n[2] = (int)c.dims[2];
    g.v = c.par[0];
    g.rv = c.aux[6];
    g.corner[0] = c.aux[0];
    g.corner[1] = c.aux[1];
    g.corner[2] = c.aux[2];
    g.nvox = (uint32_t)c.n0;
    for (int i = 0; i < 3; ++i) {
        g.blo[i] = c.aux[8 + i];
        g.bhi[i] = c.aux[11 + i];
    }
    g.bg = (uint32_t)c.aux[14];
    g.box = c.aux[15] != 0.0;
    return g;
}

// The loaded byte goes through an empty asm so that it stays a plain 32-bit
// value: the compiler otherwise narrows the walk's materials to 16 bits and
// masks the loads with extra instructions.
__device__ __forceinline__ uint32_t load_voxel(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    uint32_t m = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, off, 0, 0);
    asm("" : "+v"(m));
    return m;
}

template <class T>
__device__ __forceinline__ T pick3(int k, T a0, T a1, T a2) {
    return k == 0 ? a0 : (k == 1 ? a1 : a2);
}

// alpha of the plane at coordinate P on an axis with start q, reciprocal
// direction inv and offset nq = -q inv.  ONE_ROUNDING: fma(P, inv, nq), one
// instruction, one rounding after the exact product; otherwise
// (P - q) * inv, the reference definition's rounding.  The walks that
// locate interaction points keep the latter: a scattering chain feeds each
// located point into the next walk, so it stays on the reference's
// roundings, while a plain optical depth only sums the crossings' alphas.
template <bool ONE_ROUNDING>
__device__ __forceinline__ double plane_alpha(double P, double q, double inv, double nq) {
    if constexpr (ONE_ROUNDING) return fma(P, inv, nq);
    else return (P - q) * inv;
}

// Per-axis walk state, one entry per axis; roles D, A, B pick from it with
// selects (registers cannot be indexed by a per-lane value).
struct AxisSet {
    double P[3], q[3], nq[3], inv[3], c[3];  // c: corner, mirrored (-corner) for negative directions
    int k[3], doff[3];
};

// Minimum of two doubles that are never NaN, as the one VALU instruction
// v_min_f64.  The ternary a < b ? a : b compiles to a compare and two
// selects, and fmin() adds canonicalising instructions for operands the
// compiler cannot prove canonical; the walk's alphas are finite or +inf and
// positive, so a tie returns the same number either way.
__device__ __forceinline__ double min_f64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ double max_f64(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The divergent event's updates, written so that each new value takes the
// register of the value it replaces (tied operands).  The uniform D step
// leaves the A and B state untouched; with in-place updates on the other
// path the two paths meet without register copies (the compiler otherwise
// gives the new values fresh registers and copies the old ones on the
// uniform path, five to six moves per event).  Same arithmetic as
// P = fma(f, v, P), a = fma(P, inv, nq) and m = min(a, b).
__device__ __forceinline__ void step_in_place(double &P, double f, double v) {
    asm("v_fma_f64 %0, %1, %2, %0" : "+v"(P) : "v"(f), "s"(v));
}
__device__ __forceinline__ void alpha_in_place(double &a, double P, double inv, double nq) {
    asm("v_fma_f64 %0, %1, %2, %3" : "+v"(a) : "v"(P), "v"(inv), "v"(nq));
}
__device__ __forceinline__ void min_in_place(double &m, double a, double b) {
    asm("v_min_f64 %0, %1, %2" : "+v"(m) : "v"(a), "v"(b));
}

// clamp(x, 0, hi) for hi >= 0 as one v_med3_i32, and a * b + c on the low
// 24 bits of a and b as one full-rate v_mad_u32_u24.  Written out because
// the compiler emits max + min for the first and folds the second into a
// 64-bit multiply-add.  hi and a are wave-uniform here (the phantom's
// dimensions) and stay in scalar registers.
__device__ __forceinline__ int clamp0_i32(int x, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(x), "s"(hi));
    return r;
}
__device__ __forceinline__ uint32_t mad_u24(int a, int b, int c) {
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "s"(a), "v"(b), "v"(c));
    return r;
}

// The walk in rounds of K crossings ("events").  Each event is the nearest
// of the next D, A and B crossings (D first on ties with the others, A before
// B); its alpha is computed from the plane coordinate, so it is the same
// number the merged order of all crossings would see.  The nearer of the A
// and B crossings is kept (mAB), so one compare tells whether a lane's next
// event is a D step.  When no lane of the wave has an A or B crossing next,
// the event is a D step for the whole wave (the common case).  Otherwise
// every lane steps one axis without branching: each axis's plane advances
// by a factor of 1 or 0 times v (an exact fma), and all three alphas are
// recomputed from their planes, which leaves the two unchanged ones bit for
// bit as they were.  An axis the ray runs parallel to has inv = 0 and
// nq = +inf, so its alpha is +inf and it never steps.  The K voxel loads of
// a round are issued together and then folded into the material runs in
// order.  Events are not clipped to the exit: a lane past its exit keeps
// stepping, and the fold clips each closing alpha to a_out, so runs past the
// exit have zero length and add nothing (their voxels are read through the
// range-checked buffer).
//
// LOCATE: also find where the running optical depth reaches tau_star.  Within
// a material run mu is constant, so the point is checked when a run closes:
// a_start + (tau_star - tau_before) / mu in the first attenuating run whose
// closing depth reaches tau_star (hit.found); hit.last_end / last_m keep the
// end and material of the last attenuating run for a tau_star that rounding
// leaves beyond the total.  A wave leaves the walk once every lane has found
// its point or passed its exit.
struct WalkHit {
    double s = 0.0, last_end = 0.0;
    uint32_t m = 0, last_m = 0;
    bool found = false;
};

// Close the material run [a_start, tc] of material m (attenuation mu) onto
// the optical depth tau; LOCATE: and check it for the depth tau_star.
template <bool LOCATE>
__device__ __forceinline__ void close_run(double tc, double mu, uint32_t m, double &tau, double a_start,
                                          double tau_star, WalkHit *hit) {
    const double closed = fma(mu, tc - a_start, tau);
    if constexpr (LOCATE) {
        if (mu > 0.0 && tc > a_start) {
            if (!hit->found && closed >= tau_star) {
                hit->found = true;
                hit->s = a_start + (tau_star - tau) / mu;
                hit->m = m;
            }
            hit->last_end = tc;
            hit->last_m = m;
        }
    }
    tau = closed;
}

// a_vol <= a_in: the path enters the volume at a_vol and the walk at a_in,
// the first voxel (off) lying just past a_in; before it the path runs in
// material bg (bg < 0: a_vol = a_in).  The walk stops once every lane's events
// reach a_stop <= a_out; runs still close at a_out.
template <bool EXACT, int K, bool LOCATE = false>
__device__ __forceinline__ double siddon_walk(const PhantomGeo &g, const AxisSet &S, int D, int A, int B,
                                              uint32_t off, double a_vol, double a_in, double a_stop, double a_out,
                                              int bg, const double *__restrict__ mu_row, double tau_star = 0.0,
                                              WalkHit *hit = nullptr) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)g.vol, (short)0, (int)g.nvox, 0x00020000);
    const double v = g.v;
    double PD = pick3(D, S.P[0], S.P[1], S.P[2]), PA = pick3(A, S.P[0], S.P[1], S.P[2]);
    double PB = pick3(B, S.P[0], S.P[1], S.P[2]);
    constexpr bool ONE = !LOCATE;
    const double nD = pick3(D, S.nq[0], S.nq[1], S.nq[2]);
    const double nA = pick3(A, S.nq[0], S.nq[1], S.nq[2]), nB = pick3(B, S.nq[0], S.nq[1], S.nq[2]);
    const double qD = pick3(D, S.q[0], S.q[1], S.q[2]);
    const double qA = pick3(A, S.q[0], S.q[1], S.q[2]), qB = pick3(B, S.q[0], S.q[1], S.q[2]);
    const double iD = pick3(D, S.inv[0], S.inv[1], S.inv[2]);
    const double iA = pick3(A, S.inv[0], S.inv[1], S.inv[2]), iB = pick3(B, S.inv[0], S.inv[1], S.inv[2]);
    int kD = pick3(D, S.k[0], S.k[1], S.k[2]), kA = pick3(A, S.k[0], S.k[1], S.k[2]);
    int kB = pick3(B, S.k[0], S.k[1], S.k[2]);
    const int oD = pick3(D, S.doff[0], S.doff[1], S.doff[2]), oA = pick3(A, S.doff[0], S.doff[1], S.doff[2]);
    const int oB = pick3(B, S.doff[0], S.doff[1], S.doff[2]);
    const int dA = oA - oD, dB = oB - oD;  // offset change of an A or B step in place of the D step
    // plane k of a mirrored axis sits at -corner + k v
    const double cD = pick3(D, S.c[0], S.c[1], S.c[2]);
    const double cA = pick3(A, S.c[0], S.c[1], S.c[2]), cB = pick3(B, S.c[0], S.c[1], S.c[2]);
    double aD = plane_alpha<ONE>(PD, qD, iD, nD);
    double aA = plane_alpha<ONE>(PA, qA, iA, nA);
    double aB = plane_alpha<ONE>(PB, qB, iB, nB);
    double mAB = min_f64(aA, aB);

    uint32_t run_m = load_voxel(rs, off);
    double a_start = a_vol, tau = 0.0;
    if (bg >= 0 && run_m != (uint32_t)bg) {
        // the background run ends where the walk enters its first voxel
        close_run<LOCATE>(a_in, mu_row[bg], (uint32_t)bg, tau, a_vol, tau_star, hit);
        a_start = a_in;
    }
    const int max_rounds = __builtin_amdgcn_readfirstlane((g.n[0] + g.n[1] + g.n[2] + 3) / K + 2);
    for (int round = 0; round < max_rounds; ++round) {
        uint32_t o[K];
        double t[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool side = mAB < aD;
            t[j] = min_f64(aD, mAB);
            // every lane takes the D step; a lane whose next crossing is an
            // A or B plane takes that one instead: in an exec-masked block it
            // advances that plane, adds the stride difference and moves its
            // D plane back by v (exact), so the step leaves it in place
            off += (uint32_t)oD;
            if constexpr (EXACT) PD = PD + v;
            else ++kD;
            const uint64_t wside = __builtin_amdgcn_ballot_w64(side);
            if (LOCATE && wside != 0) {
                // the locate walks (scattering chains, whose kernel runs
                // short of registers): every lane advances each axis's plane
                // by a 0/1 factor times v (branch-free, no exec changes)
                const bool tA = side && aA <= aB;
                const bool tB = side && !tA;
                off += (uint32_t)(tA ? dA : (tB ? dB : 0));
                if constexpr (EXACT) {
                    PD = fma(side ? -1.0 : 0.0, v, PD);
                    PA = fma(tA ? 1.0 : 0.0, v, PA);
                    PB = fma(tB ? 1.0 : 0.0, v, PB);
                } else {
                    kD -= side;
                    kA += tA;
                    kB += tB;
                    PA = cA + (double)kA * v;
                    PB = cB + (double)kB * v;
                }
                aA = plane_alpha<ONE>(PA, qA, iA, nA);
                aB = plane_alpha<ONE>(PB, qB, iB, nB);
                mAB = min_f64(aA, aB);
            } else if (wside != 0) {
                // the A/B order as a lane mask straight from the compare, so
                // the wave can skip a block that none of its lanes takes
                const uint64_t wle = __builtin_amdgcn_fcmp(aA, aB, 5);  // FCMP_OLE: ordered <=
                const bool AfirstB = aA <= aB;
                if (__builtin_expect((wside & wle) != 0, 0)) {
                    if (side && AfirstB) {
                        off += (uint32_t)dA;
                        PA = EXACT ? PA + v : cA + (double)(++kA) * v;
                        aA = plane_alpha<ONE>(PA, qA, iA, nA);
                        if constexpr (EXACT) PD = PD - v;
                        else kD -= 1;
                    }
                }
                if (__builtin_expect((wside & ~wle) != 0, 0)) {
                    if (side && !AfirstB) {
                        off += (uint32_t)dB;
                        PB = EXACT ? PB + v : cB + (double)(++kB) * v;
                        aB = plane_alpha<ONE>(PB, qB, iB, nB);
                        if constexpr (EXACT) PD = PD - v;
                        else kD -= 1;
                    }
                }
                mAB = min_f64(aA, aB);
            }
            if constexpr (!EXACT) PD = cD + (double)kD * v;
            aD = plane_alpha<ONE>(PD, qD, iD, nD);
            o[j] = off;
        }
        uint32_t m[K];
#pragma unroll
        for (int j = 0; j < K; ++j) m[j] = load_voxel(rs, o[j]);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            // a material change closes the run (a wave with no change skips
            // the block on its empty execution mask)
            if (m[j] != run_m) {
                const double tc = min_f64(t[j], a_out);
                close_run<LOCATE>(tc, mu_row[run_m], run_m, tau, a_start, tau_star, hit);
                a_start = tc;
                run_m = m[j];
            }
        }
        // every lane is past its exit once its last event lies at or beyond a_out
        if constexpr (LOCATE) {
            if (__builtin_amdgcn_ballot_w64(t[K - 1] < a_out && !hit->found) == 0) break;
        } else {
            if (__builtin_amdgcn_ballot_w64(t[K - 1] < a_stop) == 0) break;
        }
    }
    close_run<LOCATE>(a_out, mu_row[run_m], run_m, tau, a_start, tau_star, hit);
    return tau;
}

// The path's stretch a_in .. a_out inside the volume (false: none) and its
// reciprocal directions (0 for an axis it runs parallel to).
__device__ __forceinline__ bool volume_chord(const PhantomGeo &g, const double q[3], const double dl[3], double inv[3],
                                             double &a_in, double &a_out) {
    a_in = 0.0;
    a_out = kInf;
    bool in = true;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double lo_p = g.corner[i];
        double hi_p = g.corner[i] + (double)g.n[i] * g.v;
        if (dl[i] == 0.0) {
            inv[i] = 0.0;
            if (!(q[i] > lo_p && q[i] < hi_p)) in = false;
        } else {
            inv[i] = 1.0 / dl[i];
            double a0 = (lo_p - q[i]) * inv[i], a1 = (hi_p - q[i]) * inv[i];
            double lo = a0 < a1 ? a0 : a1, hi = a0 < a1 ? a1 : a0;
            if (lo > a_in) a_in = lo;
            if (hi < a_out) a_out = hi;
        }
    }
    return in && a_out > a_in;
}

// EXACT: every plane coordinate corner + i v is reached exactly by adding v
// (true for dyadic voxel sizes such as 1 mm); decided once per instrument.
// BOX (optical depths only): the walk covers the path's stretch inside the
// occupied box.  Outside it every voxel holds the background material, so
// the run that enters the volume there stays open up to the box, and the
// box's faces are crossed at the alphas the full walk computes for those
// planes (fma(plane, inv, -q inv)): the same runs and sums, except that a
// path touching the box only along an edge or a face takes its background run
// in one piece (a zero-length run less, a rounding of the sum).
template <bool EXACT, bool LOCATE = false, bool BOX = false, int KW = kWalkRound>
__device__ __forceinline__ double siddon_tau(const PhantomGeo &g, const double q[3], const double dl[3],
                                             const double *__restrict__ mu_row, double tau_star = 0.0,
                                             WalkHit *hit = nullptr) {
    double inv[3], a_in, a_out;
    if (!volume_chord(g, q, dl, inv, a_in, a_out)) return 0.0;
    const double a_vol = a_in;
    double a_stop = a_out;
    int bg = -1;
    if constexpr (BOX && !LOCATE) {
        bool miss = !g.box;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (dl[i] == 0.0) {
                // the voxel slab the walk would keep (as in the set-up below)
                const double f = floor((q[i] - g.corner[i]) / g.v);
                const int idx = (int)fmin(fmax(f, 0.0), (double)(g.n[i] - 1));
                const int lo = (int)rint((g.blo[i] - g.corner[i]) * g.rv);
                const int hi = (int)rint((g.bhi[i] - g.corner[i]) * g.rv);
                if (idx < lo || idx >= hi) miss = true;
            } else {
                const double nq = -(q[i] * inv[i]);
                const double b0 = fma(g.blo[i], inv[i], nq), b1 = fma(g.bhi[i], inv[i], nq);
                a_in = fmax(a_in, fmin(b0, b1));
                a_stop = fmin(a_stop, fmax(b0, b1));
            }
        }
        if (miss || !(a_stop > a_in)) return fma(mu_row[g.bg], a_out - a_vol, 0.0);
        bg = (int)g.bg;
    }

    // Per axis: the voxel holding the start of the walk and the first plane
    // crossed after a_in.  Planes are mirrored for negative directions
    // (coordinate -x, plane index counted downwards), so that the next plane
    // is always reached by adding v; alpha keeps its value (with -P, -q and
    // -inv the product P inv and the difference (P - q) inv are the same
    // numbers, -q inv unchanged).  An axis the ray runs parallel to gets an
    // alpha of +inf: inv = 0 and nq = +inf for the one-rounding form, a
    // plane ahead of q and inv = +inf for the other.
    constexpr bool ONE = !LOCATE;
    int idx[3];
    AxisSet S;
    const int nx = g.n[0], nxy = g.n[0] * g.n[1];
    const int stride[3] = {1, nx, nxy};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int n = g.n[i];
        const double c = g.corner[i], v = g.v;
        if (dl[i] == 0.0) {
            double f = floor((q[i] - c) / v);
            idx[i] = (int)fmin(fmax(f, 0.0), (double)(n - 1));
            S.k[i] = 0;
            S.P[i] = ONE ? 0.0 : q[i] + 1.0;
            S.q[i] = q[i];
            S.nq[i] = kInf;
            S.inv[i] = ONE ? 0.0 : kInf;
            S.c[i] = c;
            S.doff[i] = 0;
            continue;
        }
        const double nq = -(q[i] * inv[i]);
        const double x_in = q[i] + a_in * dl[i];
        const double f = (x_in - c) * g.rv;  // an estimate: p is corrected below
        int p;
        if (dl[i] > 0.0) {
            // first plane p in [1, n] with alpha(p) > a_in
            p = (int)fmin(fmax(floor(f) + 1.0, 1.0), (double)n);
            if (p > 1 && plane_alpha<ONE>(c + (double)(p - 1) * v, q[i], inv[i], nq) > a_in) p -= 1;
            if (p < n && !(plane_alpha<ONE>(c + (double)p * v, q[i], inv[i], nq) > a_in)) p += 1;
            idx[i] = p - 1;
            S.k[i] = p;
            S.P[i] = c + (double)p * v;
            S.q[i] = q[i];
            S.nq[i] = nq;
            S.inv[i] = inv[i];
            S.c[i] = c;
            S.doff[i] = stride[i];
        } else {
            // last plane p in [0, n - 1] with alpha(p) > a_in, walked downwards
            p = (int)fmin(fmax(ceil(f) - 1.0, 0.0), (double)(n - 1));
            if (p < n - 1 && plane_alpha<ONE>(c + (double)(p + 1) * v, q[i], inv[i], nq) > a_in) p += 1;
            if (p > 0 && !(plane_alpha<ONE>(c + (double)p * v, q[i], inv[i], nq) > a_in)) p -= 1;
            idx[i] = p;
            // mirrored: plane index k = -p, coordinate -(c + p v), -q, -inv
            S.k[i] = -p;
            S.P[i] = -(c + (double)p * v);
            S.q[i] = -q[i];
            S.nq[i] = nq;
            S.inv[i] = -inv[i];
            S.c[i] = -c;
            S.doff[i] = -stride[i];
        }
    }
    // dominant axis (largest |d|, lowest index on ties) and the other two
    const double ax = fabs(dl[0]), ay = fabs(dl[1]), az = fabs(dl[2]);
    int D, A, B;
    if (ax >= ay && ax >= az) { D = 0; A = 1; B = 2; }
    else if (ay >= az) { D = 1; A = 0; B = 2; }
    else { D = 2; A = 0; B = 1; }
    const uint32_t off = (uint32_t)(idx[0] + nx * idx[1] + nxy * idx[2]);
    return siddon_walk<EXACT, LOCATE ? kLocateRound : KW, LOCATE>(g, S, D, A, B, off, a_vol, a_in, a_stop,
                                                                         a_out, bg, mu_row, tau_star, hit);
}

// ---------------------------------------------------- fixed-step model ----
// The paper's own way through the voxel sample (section 3.3): fixed steps of
// length h, each reading the voxel that holds its end position and
// attenuating over its length.  The chord is the exact walk's; step j covers
// [a_in + (j-1) h, min(a_in + j h, a_out)] (the last step is clipped at the
// exit) and reads the voxel at u_in + j (h d / v) in voxel units (one fused
// multiply-add per axis), taken unclipped and clamped into the volume.  Both numbers come from j directly,
// with no running sum, so the steps are independent: kStepRound voxel loads
// are issued per round.  The optical depth is summed per material run as in
// the exact walk.  jmax (volume diagonal / h + 2, from the host) bounds every
// loop; a voxel index is clamped per axis, so every load is in range.
constexpr int kStepRound = 4;

// One path's steps: length, sample position and advance in voxel units, and
// their count.
struct StepPath {
    double h, u0[3], du[3];
    int J;
};
// Set up a path (false: it misses the volume); inv = 1 / dl (0: parallel).
__device__ __forceinline__ bool step_path(const PhantomGeo &g, const double q[3], const double dl[3], double h, int jmax,
                                          double inv[3], double &a_in, double &a_out, StepPath &p) {
    if (!volume_chord(g, q, dl, inv, a_in, a_out)) return false;
    p.h = h;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p.u0[i] = ((q[i] + a_in * dl[i]) - g.corner[i]) / g.v;
        p.du[i] = (h * dl[i]) / g.v;
    }
    // this lane's step count: the first j with a_in + j h >= a_out
    // (a_in + j h is non-decreasing in j, so the fix-ups end at that j)
    p.J = (int)fmin(fmax(ceil((a_out - a_in) / h), 1.0), (double)jmax);
    while (p.J > 1 && !(a_in + (double)(p.J - 1) * h < a_out)) --p.J;
    while (p.J < jmax && a_in + (double)p.J * h < a_out) ++p.J;
    return true;
}

// Voxel of step j: truncation then clamping at 0 equals floor then clamping,
// for every value in int range.  The host admits the model only for ny nz <
// 2^24, so the offset takes two 24-bit multiply-adds (full rate) instead of
// 32-bit multiplies (quarter rate).
__device__ __forceinline__ uint32_t step_voxel(const StepPath &p, int j, int nx, int ny, int nz) {
    const double dj = (double)j;
    const int ix = clamp0_i32((int)fma(dj, p.du[0], p.u0[0]), nx - 1);
    const int iy = clamp0_i32((int)fma(dj, p.du[1], p.u0[1]), ny - 1);
    const int iz = clamp0_i32((int)fma(dj, p.du[2], p.u0[2]), nz - 1);
    return mad_u24(nx, mad_u24(ny, iz, iy), ix);
}

__device__ __forceinline__ double step_tau(const PhantomGeo &g, const double q[3], const double dl[3], double h,
                                           int jmax, const double *__restrict__ mu_row) {
    double inv[3], a_in, a_out;
    StepPath p;
    if (!step_path(g, q, dl, h, jmax, inv, a_in, a_out, p)) return 0.0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)g.vol, (short)0, (int)g.nvox, 0x00020000);
    uint32_t run_m = load_voxel(rs, step_voxel(p, 1, g.n[0], g.n[1], g.n[2]));
    double a_start = a_in, tau = 0.0;
    const int max_rounds = (jmax + kStepRound - 1) / kStepRound + 1;
    int j0 = 2;
    for (int round = 0; round < max_rounds; ++round, j0 += kStepRound) {
        if (__builtin_amdgcn_ballot_w64(j0 <= p.J) == 0) break;
        uint32_t m[kStepRound];
#pragma unroll
        for (int k = 0; k < kStepRound; ++k) m[k] = load_voxel(rs, step_voxel(p, j0 + k, g.n[0], g.n[1], g.n[2]));
#pragma unroll
        for (int k = 0; k < kStepRound; ++k) {
            // a step past this lane's last one starts at or beyond a_out:
            // clamped there, it closes the open run exactly as the final
            // term would and adds zero-length runs after it, so no per-step
            // j <= J test is needed
            if (m[k] != run_m) {
                const double a = min_f64(a_in + (double)(j0 + k - 1) * h, a_out);
                tau = fma(mu_row[run_m], a - a_start, tau);
                a_start = a;
                run_m = m[k];
            }
        }
    }
    return fma(mu_row[run_m], a_out - a_start, tau);
}

// ------------------------------------------------------- bundle walk ----
// Optical depths of a whole wave.  The strata send the 64 rays of a wave in
// nearly one direction, and almost everywhere the few voxels that the bundle
// covers in a layer across its dominant axis D hold one material: of the 256
// layers of the luggage phantom 2 to 11 hold a boundary inside the bundle and
// 3 to 7 more begin with a new material.  So the lanes look at layers, one
// each, and the rays then only
//   - close their run at a D plane where the whole bundle changes material,
//   - walk a stretch of mixed layers, event by event (stretch_walk).
// The lanes look twice: first at 64 layers of 4^3-voxel bricks, whose map
// (a brick's one material, or kMixed) was made with the instrument, then at
// the voxels of the layers whose bricks do not settle it, 64 layers at a
// time.  A look is the bundle's footprint in the layer -- from the smallest
// and largest of the rays' A and B coordinates at two D planes -- and whether
// what it covers agrees.
// All alphas are the event walk's own (plane_alpha of the same planes), and
// material runs close at the same crossings, so the sums are the same but
// for the order in which a run is split.
//
// Footprints are conservative: single-precision bounds in voxel units widened
// by kBundleSlack (coordinates stay below 2^12 for volumes of at most
// kBundleDim voxels an axis, so a bound's rounding is below 2^-9), clamped to
// the volume (a ray is outside the volume there and its run is clipped).  A
// footprint wider than kBrickWide bricks or kBundleWide voxels counts as
// mixed, and a bundle that is nowhere narrower than kBundleNarrow voxels, or
// has fewer than kBundleLayers layers to cross, is not looked at (a 64^3
// phantom with 36 occupied layers, 2e5 rays: 26.1 us with the looks, 21.9
// without; 3e6 rays 116 either way; a 128^3 one, 1e6 rays: 62 and 95 us).
//
// What bounds its kernel: VALU issue, 0.8 of the rate in the tiled image kernel,
// the source and the ray's share of the looks before the stretches.  A ray id a
// lane and without tiles, 1e9 rays through 256^3 voxels at 0 / 0.785 rad, event walk
// of every ray that reaches the monitor 33.3 / 48 ms, this 29.4 / 31.3 ms (in tiles
// 16.5 ms); 2e7 rays in wide strata (256^2) through 512^3: 3.2 -> 0.76 ms and 3.7 ->
// 1.0 ms.
constexpr float kBundleSlack = 0.0078125f, kBundleNarrow = 6.0f;
constexpr int kBundleDim = 2048, kBundleWide = 4, kBrickWide = 3;
constexpr int kBundleLayers = 64;
constexpr int kMixed = 255, kNoLayer = 254;  // codes of a layer beside its one material
constexpr int kBrick = 4;                    // voxels along a brick's edge
constexpr int kStretchRound = 4;  // crossings per round of a stretch's walk

// The least over the wave of each of eight values, in scalar registers.
// row_shr 1, 2, 4, 8 leave a row's least value in its last lane, row_bcast 15
// and 31 carry it on to lane 63; a lane without a source lane keeps its own.
// One instruction a step (the compiler's form of update_dpp and fminf takes
// four); eight chains side by side keep the two wait states between a write
// and a DPP read.
#define MXR_MIN8(step)                                 \
    "v_min_f32_dpp %0, %0, %0 " step "\n\t"            \
    "v_min_f32_dpp %1, %1, %1 " step "\n\t"            \
    "v_min_f32_dpp %2, %2, %2 " step "\n\t"            \
    "v_min_f32_dpp %3, %3, %3 " step "\n\t"            \
    "v_min_f32_dpp %4, %4, %4 " step "\n\t"            \
    "v_min_f32_dpp %5, %5, %5 " step "\n\t"            \
    "v_min_f32_dpp %6, %6, %6 " step "\n\t"            \
    "v_min_f32_dpp %7, %7, %7 " step "\n\t"
__device__ __forceinline__ void wave_min8(float x[8]) {
    asm("s_nop 1\n\t" MXR_MIN8("row_shr:1 row_mask:0xf bank_mask:0xf") MXR_MIN8("row_shr:2 row_mask:0xf bank_mask:0xf")
            MXR_MIN8("row_shr:4 row_mask:0xf bank_mask:0xf") MXR_MIN8("row_shr:8 row_mask:0xf bank_mask:0xf")
                MXR_MIN8("row_bcast:15 row_mask:0xf bank_mask:0xf") MXR_MIN8("row_bcast:31 row_mask:0xf bank_mask:0xf")
        "s_nop 1"
        : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[i]), 63));
}
#undef MXR_MIN8

// floor(x) as an integer, the lesser of two floats: one instruction each.
__device__ __forceinline__ int floor_i32(float x) {
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ float min_f32(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Open material run of a path: material m (attenuation mu, read when the run
// opens so that its close does not wait for it) since a_start, depth tau of
// the runs closed before it.
struct OpenRun {
    uint32_t m;
    double mu, a_start, tau;
};

// The same, looking for the depth tau_star on the way (see WalkHit).
struct FindRun : OpenRun {
    double tau_star;
    WalkHit hit;
};

// tau plus the depth of a run of length len >= 0.  A run of no length adds
// nothing, also in an opaque material (mu infinite): a path turns through the
// materials it meets behind the place where its run closed, or behind its end.
__device__ __forceinline__ double add_run(double mu, double len, double tau) {
    const int hi = len > 0.0 ? __double2hiint(mu) : 0;  // the low word alone is a finite number
    return fma(__hiloint2double(hi, __double2loint(mu)), len, tau);
}

// Close the run at t (clipped to the path's end, and never set back) and open
// one of material m.
template <class Run>
__device__ __forceinline__ void turn_run(Run &run, double t, double a_out, uint32_t m, const double *__restrict__ mu_row) {
    const double tc = max_f64(min_f64(t, a_out), run.a_start);
    if constexpr (sizeof(Run) > sizeof(OpenRun)) {
        if (tc > run.a_start) {  // as close_run
            const double tau = fma(run.mu, tc - run.a_start, run.tau);
            if (run.mu > 0.0) {
                if (!run.hit.found && tau >= run.tau_star) {
                    run.hit.found = true;
                    run.hit.s = run.a_start + (run.tau_star - run.tau) / run.mu;
                    run.hit.m = run.m;
                }
                run.hit.last_end = tc;
                run.hit.last_m = run.m;
            }
            run.tau = tau;
        }
    } else {
        run.tau = add_run(run.mu, tc - run.a_start, run.tau);
    }
    run.a_start = tc;
    run.m = m;
    run.mu = mu_row[m];
}

// One axis of a path across the volume, in the role of D, A or B: the
// lane's start, direction and reciprocal (direction 0: reciprocal 0).
struct Role {
    double q, d, inv;
};
// Its constants, the wave's: corner, voxel count and strides of the voxels
// and of the bricks.
struct RoleAxis {
    double c;
    int n, str, brick;
};
__device__ __forceinline__ RoleAxis role_axis(const MXR_CONSTANT DevComp *ph, int i) {
    const int nx = (int)ph->dims[0], ny = (int)ph->dims[1], nz = (int)ph->dims[2];
    const int bx = (nx + kBrick - 1) / kBrick, by = (ny + kBrick - 1) / kBrick;
    return {pick3(i, ph->aux[0], ph->aux[1], ph->aux[2]), pick3(i, nx, ny, nz), pick3(i, 1, nx, nx * ny),
            pick3(i, 1, bx, bx * by)};
}

// State of an axis at alpha as: the next plane ahead (coordinate mirrored by
// the sign of the direction), its index, and the voxel before it.  The plane
// comes from the position alone: one that lies within a rounding of as may be
// taken as passed or as ahead, which moves a run's end by that rounding.
struct RoleStep {
    double P, iv, nq, c;
    int k, idx, off;
};
__device__ __forceinline__ RoleStep role_at(const Role &r, const RoleAxis &x, double v, double rv, double as) {
    RoleStep s;
    const bool fwd = r.d > 0.0;
    const double f = ((r.q + as * r.d) - x.c) * rv;
    // forward: voxel floor(f), plane one above it; backward: plane ceil(f) - 1,
    // the voxel above that plane; along the axis: voxel floor(f), no plane
    const double g = r.d < 0.0 ? ceil(f) - 1.0 : floor(f);
    s.idx = (int)min_f64(max_f64(g, 0.0), (double)(x.n - 1));
    s.k = fwd ? s.idx + 1 : -s.idx;
    s.c = fwd ? x.c : -x.c;
    s.iv = fwd ? r.inv : -r.inv;
    s.nq = r.d == 0.0 ? kInf : -(r.q * r.inv);
    s.P = s.c + (double)s.k * v;
    s.off = r.d == 0.0 ? 0 : (fwd ? x.str : -x.str);
    return s;
}

// The event walk (see siddon_walk) of a stretch of layers, from as to ae: a
// path begins at the stretch's first plane, in the D layer behind it, or, if
// late, further on, in the layer its position gives.  Events past ae are
// events of the path all the same; the next stretch or change sees them again
// as runs of no length (turn_run never sets a run back).
template <bool EXACT, int K, class Run>
__device__ __forceinline__ void stretch_walk(const MXR_CONSTANT DevComp *ph, int axD, const Role &D, const Role &A,
                                             const Role &B, bool back, int layer, bool late, double as, double ae,
                                             double a_out, Run &run, const double *__restrict__ mu_row) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)ph->data0, (short)0, (int)ph->n0, 0x00020000);
    const RoleAxis xD = role_axis(ph, axD), xA = role_axis(ph, axD == 0 ? 1 : 0), xB = role_axis(ph, axD == 2 ? 1 : 2);
    constexpr bool ONE = sizeof(Run) == sizeof(OpenRun);  // as the event walk's alphas (see siddon_walk)
    const double v = ph->par[0], rv = ph->aux[6];
    const RoleStep a = role_at(A, xA, v, rv, as), b = role_at(B, xB, v, rv, as);
    if (late) layer = role_at(D, xD, v, rv, as).idx;
    const double cD = back ? -xD.c : xD.c, iD = back ? -D.inv : D.inv, nD = -(D.q * D.inv), qD = back ? -D.q : D.q;
    const double qA = A.d > 0.0 ? A.q : -A.q, qB = B.d > 0.0 ? B.q : -B.q;
    int kD = back ? -layer : layer + 1, kA = a.k, kB = b.k;
    double PD = cD + (double)kD * v, PA = a.P, PB = b.P;
    double aD = plane_alpha<ONE>(PD, qD, iD, nD);
    double aA = a.nq == kInf ? kInf : plane_alpha<ONE>(PA, qA, a.iv, a.nq), aB = b.nq == kInf ? kInf : plane_alpha<ONE>(PB, qB, b.iv, b.nq);
    double mAB = min_f64(aA, aB);
    const int oD = back ? -xD.str : xD.str, dA = a.off - oD, dB = b.off - oD;
    uint32_t off = (uint32_t)(layer * xD.str + a.idx * xA.str + b.idx * xB.str);
    uint32_t m0 = load_voxel(rs, off);
    bool first = true;
    const int max_rounds = (xD.n + xA.n + xB.n + 3) / K + 2;
    for (int round = 0; round < max_rounds; ++round) {
        uint32_t o[K];
        double t[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const bool side = mAB < aD;
            t[j] = min_f64(aD, mAB);
            off += (uint32_t)oD;
            if constexpr (EXACT) PD = PD + v;
            else ++kD;
            const uint64_t wside = __builtin_amdgcn_ballot_w64(side);
            if (wside != 0) {
                const uint64_t wle = __builtin_amdgcn_fcmp(aA, aB, 5);  // FCMP_OLE: ordered <=
                const bool AfirstB = aA <= aB;
                if (__builtin_expect((wside & wle) != 0, 0)) {
                    if (side && AfirstB) {
                        off += (uint32_t)dA;
                        PA = EXACT ? PA + v : a.c + (double)(++kA) * v;
                        aA = plane_alpha<ONE>(PA, qA, a.iv, a.nq);
                        if constexpr (EXACT) PD = PD - v;
                        else kD -= 1;
                    }
                }
                if (__builtin_expect((wside & ~wle) != 0, 0)) {
                    if (side && !AfirstB) {
                        off += (uint32_t)dB;
                        PB = EXACT ? PB + v : b.c + (double)(++kB) * v;
                        aB = plane_alpha<ONE>(PB, qB, b.iv, b.nq);
                        if constexpr (EXACT) PD = PD - v;
                        else kD -= 1;
                    }
                }
                mAB = min_f64(aA, aB);
            }
            if constexpr (!EXACT) PD = cD + (double)kD * v;
            aD = plane_alpha<ONE>(PD, qD, iD, nD);
            o[j] = off;
        }
        uint32_t m[K];
#pragma unroll
        for (int j = 0; j < K; ++j) m[j] = load_voxel(rs, o[j]);
        // the first voxel's material arrives with the first round's
        if (first && m0 != run.m) turn_run(run, as, a_out, m0, mu_row);
        first = false;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (m[j] != run.m) turn_run(run, t[j], a_out, m[j], mu_row);
        if (__builtin_amdgcn_ballot_w64(t[K - 1] < ae) == 0) break;
    }
}

// First step of a path whose sample lies behind the D plane number `plane`
// (u0, du: the path's D coordinate; end: the plane its paths leave the volume
// by, behind which the last step's sample is still read in the last layer).
__device__ __forceinline__ int step_at(int plane, bool back, int end, double u0, double du, int J) {
    if (plane == end) return J + 1;
    const double P = (double)plane;
    auto behind = [&](int j) {
        const double x = fma((double)j, du, u0);
        return back ? x < P : x >= P;
    };
    // the quotient is off by a few roundings of a number below 2^26
    int j = (int)fmin(fmax(ceil((P - u0) / du), 1.0), (double)(J + 1));
    if (j > 1 && behind(j - 1)) --j;
    else if (j <= J && !behind(j)) ++j;
    return j;
}

// The fixed steps js .. je - 1 of a path (see step_tau).  Steps past je and
// past the path's end do no harm, as in stretch_walk.
__device__ __forceinline__ void stretch_steps(const MXR_CONSTANT DevComp *ph, const StepPath &p, int js, int je,
                                              double a_in, double a_out, OpenRun &run, const double *__restrict__ mu_row) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)ph->data0, (short)0, (int)ph->n0, 0x00020000);
    const int nx = (int)ph->dims[0], ny = (int)ph->dims[1], nz = (int)ph->dims[2];
    for (int j0 = js; __builtin_amdgcn_ballot_w64(j0 < je) != 0; j0 += kStepRound) {
        uint32_t m[kStepRound];
#pragma unroll
        for (int k = 0; k < kStepRound; ++k) m[k] = load_voxel(rs, step_voxel(p, j0 + k, nx, ny, nz));
#pragma unroll
        for (int k = 0; k < kStepRound; ++k)
            if (m[k] != run.m) turn_run(run, a_in + (double)(j0 + k - 1) * p.h, a_out, m[k], mu_row);
    }
}

// Optical depth of one path by its steps, the sums of step_tau; only the steps in
// the occupied box's layers across the path's dominant axis look at voxels.
__device__ __forceinline__ double steps_tau(const MXR_CONSTANT DevComp *ph, const PhantomGeo &g, const double q[3],
                                            const double dl[3], const double *__restrict__ mu_row) {
    double inv[3], a_in, a_out;
    StepPath p;
    if (!step_path(g, q, dl, ph->par[3], (int)ph->aux[5], inv, a_in, a_out, p)) return 0.0;
    OpenRun run;
    run.m = g.bg, run.mu = mu_row[g.bg], run.a_start = a_in, run.tau = 0.0;
    if (g.box) {
        const double ax = fabs(dl[0]), ay = fabs(dl[1]), az = fabs(dl[2]);
        const int D = (ax >= ay && ax >= az) ? 0 : (ay >= az ? 1 : 2);
        const bool back = pick3(D, dl[0], dl[1], dl[2]) < 0.0;
        const double c = pick3(D, g.corner[0], g.corner[1], g.corner[2]);
        const int lo = (int)rint((pick3(D, g.blo[0], g.blo[1], g.blo[2]) - c) * g.rv);
        const int hi = (int)rint((pick3(D, g.bhi[0], g.bhi[1], g.bhi[2]) - c) * g.rv);
        const int end = back ? 0 : pick3(D, g.n[0], g.n[1], g.n[2]);
        const double u0 = pick3(D, p.u0[0], p.u0[1], p.u0[2]), du = pick3(D, p.du[0], p.du[1], p.du[2]);
        const int js = step_at(back ? hi : lo, back, end, u0, du, p.J), je = step_at(back ? lo : hi, back, end, u0, du, p.J);
        if (je > js) stretch_steps(ph, p, js, je, a_in, a_out, run, mu_row);
        if (run.m != g.bg) turn_run(run, a_in + (double)(je - 1) * p.h, a_out, g.bg, mu_row);
    }
    return add_run(run.mu, a_out - run.a_start, run.tau);
}

// Code of a footprint of (da + 1) x (db + 1) cells from offset o on, strides
// strA and strB: the four corners first, the cells between them where the
// corners agree (all loads in flight; offsets beyond the footprint fall on its
// edge).
template <int WIDE>
__device__ __forceinline__ int footprint_code(__amdgpu_buffer_rsrc_t rs, uint32_t o, int da, int db, int strA, int strB) {
    if (da >= WIDE || db >= WIDE) return kMixed;
    const uint32_t oa = (uint32_t)(da * strA), ob = (uint32_t)(db * strB);
    const uint32_t m00 = load_voxel(rs, o), m10 = load_voxel(rs, o + oa);
    const uint32_t m01 = load_voxel(rs, o + ob), m11 = load_voxel(rs, o + oa + ob);
    uint32_t diff = (m00 ^ m10) | (m00 ^ m01) | (m00 ^ m11);
    if (diff == 0 && (da > 1 || db > 1)) {
        const uint32_t oa1 = da > 0 ? (uint32_t)strA : 0u, ob1 = db > 0 ? (uint32_t)strB : 0u;
        const uint32_t c1 = load_voxel(rs, o + oa1), c2 = load_voxel(rs, o + ob1), c3 = load_voxel(rs, o + oa1 + ob1);
        const uint32_t c4 = load_voxel(rs, o + oa + ob1), c5 = load_voxel(rs, o + oa1 + ob);
        diff = (m00 ^ c1) | (m00 ^ c2) | (m00 ^ c3) | (m00 ^ c4) | (m00 ^ c5);
        if constexpr (WIDE > 3) {
            const uint32_t oa2 = da > 1 ? 2u * (uint32_t)strA : oa1, ob2 = db > 1 ? 2u * (uint32_t)strB : ob1;
            const uint32_t d1 = load_voxel(rs, o + oa2), d2 = load_voxel(rs, o + ob2), d3 = load_voxel(rs, o + oa2 + ob1);
            const uint32_t d4 = load_voxel(rs, o + oa1 + ob2), d5 = load_voxel(rs, o + oa2 + ob2);
            const uint32_t d6 = load_voxel(rs, o + oa + ob2), d7 = load_voxel(rs, o + oa2 + ob);
            diff |= (m00 ^ d1) | (m00 ^ d2) | (m00 ^ d3) | (m00 ^ d4) | (m00 ^ d5) | (m00 ^ d6) | (m00 ^ d7);
        }
    }
    return diff == 0 ? (int)m00 : kMixed;
}

// tau of every lane with in = true (its path enters the volume of the phantom
// ph at a_vol and leaves it at a_out, inv = 1 / dl); all 64 lanes of the wave
// call it together.
//
// STEP: the fixed-step model.  A layer whose footprint holds one material gives
// it to every step whose sample lies there (the sample's own rounding decides
// which, step_at), mixed layers are stepped through; the layer by which paths
// leave the volume covers what a step reaches behind it.  Samples are read
// inside the occupied box's layers by every path, also one that passes the box.
// 5e7 rays in steps of a third of a voxel through 256^3: every step of every
// ray that reaches the monitor 4.5 ms, this 1.3 ms.
template <bool EXACT, bool STEP = false, class Run = OpenRun>
__device__ __forceinline__ double bundle_tau(const MXR_CONSTANT DevComp *comp, const MXR_CONSTANT uint8_t *bricks,
                                             const double q[3], const double dl[3], const double inv[3], double a_vol,
                                             double a_out, bool in, const double *__restrict__ mu_row,
                                             const StepPath *sp = nullptr, double tau_star = 0.0, WalkHit *hit_out = nullptr) {
    constexpr bool ONE = sizeof(Run) == sizeof(OpenRun);  // as the event walk's alphas (see siddon_walk)
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    // the dominant axis, as in siddon_tau, and its direction
    const double ax = fabs(dl[0]), ay = fabs(dl[1]), az = fabs(dl[2]);
    const int ownD = (ax >= ay && ax >= az) ? 0 : (ay >= az ? 1 : 2);
    const int own = 2 * ownD + (pick3(ownD, dl[0], dl[1], dl[2]) < 0.0);
    const MXR_CONSTANT DevComp *const p0 = again(comp);
    const uint32_t bg = (uint32_t)p0->aux[14];
    Run run;
    run.m = bg, run.mu = mu_row[bg], run.a_start = a_vol, run.tau = 0.0;
    if constexpr (!ONE) run.tau_star = tau_star;
    // the path's part inside the occupied box, as in siddon_tau; outside it
    // the run of background stays open
    double a_box = a_vol, z_box = a_out;
    bool hit = in && p0->aux[15] != 0.0;
#pragma unroll
    for (int i = 0; i < (STEP ? 0 : 3); ++i) {
        const double lo = p0->aux[8 + i], hi = p0->aux[11 + i];
        const double nq = -(q[i] * inv[i]);
        const double b0 = plane_alpha<ONE>(lo, q[i], inv[i], nq), b1 = plane_alpha<ONE>(hi, q[i], inv[i], nq);
        if (dl[i] != 0.0) {
            a_box = max_f64(a_box, min_f64(b0, b1));
            z_box = min_f64(z_box, max_f64(b0, b1));
        } else {
            const double c = p0->aux[i], idx = fmin(fmax(floor((q[i] - c) / p0->par[0]), 0.0), (double)((int)p0->dims[i] - 1));
            hit = hit && idx >= rint((lo - c) * p0->aux[6]) && idx < rint((hi - c) * p0->aux[6]);
        }
    }
    if constexpr (!STEP) hit = hit && z_box > a_box;
    uint64_t live = __builtin_amdgcn_ballot_w64(hit);
    // the rays that share the first live one's axis and direction: nearly
    // always all of them
    while (live != 0) {
        const int side = __builtin_amdgcn_readlane(own, __builtin_ctzll(live));
        const bool part = hit && own == side;
        live &= ~__builtin_amdgcn_ballot_w64(part);
        const int iD = side >> 1, iA = iD == 0 ? 1 : 0, iB = iD == 2 ? 1 : 2;
        const bool back = (side & 1) != 0;
        auto role = [&](int i) {
            return Role{pick3(i, q[0], q[1], q[2]), pick3(i, dl[0], dl[1], dl[2]), pick3(i, inv[0], inv[1], inv[2])};
        };
        const Role D = role(iD), A = role(iA), B = role(iB);
        const MXR_CONSTANT DevComp *const ph = again(comp);
        const RoleAxis xD = role_axis(ph, iD);
        const double v = ph->par[0];
        // layers of bricks along D that hold the occupied box, and their
        // outer planes
        const double rv = ph->aux[6];
        const int Lo = __builtin_amdgcn_readfirstlane((int)rint((pick3(iD, ph->aux[8], ph->aux[9], ph->aux[10]) - xD.c) * rv));
        const int Hi = __builtin_amdgcn_readfirstlane((int)rint((pick3(iD, ph->aux[11], ph->aux[12], ph->aux[13]) - xD.c) * rv));
        const int bLo = Lo / kBrick, bHi = (Hi + kBrick - 1) / kBrick, NB = bHi - bLo;
        const int P0 = bLo * kBrick, P1 = bHi * kBrick < xD.n ? bHi * kBrick : xD.n;
        const double nD = -(D.q * D.inv);
        auto alpha_of = [&](int plane) { return plane_alpha<ONE>(xD.c + (double)plane * v, D.q, D.inv, nD); };
        // the bundle's span is bounded between two planes: those of the box's
        // layers; with fixed steps, by which a path's last sample lies up to its
        // reach behind the volume, the planes it enters by and the exit moved on
        // by that much (spans at two planes bound those between, not beyond)
        const int end = back ? 0 : xD.n;  // the plane by which paths leave the volume
        float F0 = (float)P0, F1 = (float)P1;
        double e0 = alpha_of(back && STEP ? P1 : P0), e1 = alpha_of(back && STEP ? P0 : P1);
        if constexpr (STEP) {
            if (back) F0 = (float)P1, F1 = (float)P0;
            if ((back ? P0 : P1) == end) {
                const double reach = p0->par[3] * rv * 1.001, beyond = back ? -reach : (double)end + reach;
                F1 = (float)beyond;
                e1 = plane_alpha<ONE>(xD.c + beyond * v, D.q, D.inv, nD);
            }
        }
        float m[8];
        {
            const double cA = pick3(iA, ph->aux[0], ph->aux[1], ph->aux[2]), cB = pick3(iB, ph->aux[0], ph->aux[1], ph->aux[2]);
            const float xA0 = (float)(((A.q - cA) + e0 * A.d) * rv), xA1 = (float)(((A.q - cA) + e1 * A.d) * rv);
            const float xB0 = (float)(((B.q - cB) + e0 * B.d) * rv), xB1 = (float)(((B.q - cB) + e1 * B.d) * rv);
            const float big = 1e30f;
            m[0] = part ? xA0 : big, m[1] = part ? xA1 : big, m[2] = part ? xB0 : big, m[3] = part ? xB1 : big;
            m[4] = part ? -xA0 : big, m[5] = part ? -xA1 : big, m[6] = part ? -xB0 : big, m[7] = part ? -xB1 : big;
        }
        wave_min8(m);
        const float perL = __builtin_amdgcn_rcpf(F1 - F0);
        const float A0 = m[0], A1 = (m[1] - A0) * perL, B0 = m[2], B1 = (m[3] - B0) * perL;
        const float mA0 = m[4], mA1 = (m[5] - mA0) * perL, mB0 = m[6], mB1 = (m[7] - mB0) * perL;
        // a bundle that stays wide, one in few layers, or one in a volume too
        // long for the bounds' precision walks all layers as one stretch
        const bool narrow = Hi - Lo >= kBundleLayers && (int)ph->dims[0] <= kBundleDim && (int)ph->dims[1] <= kBundleDim &&
                            (int)ph->dims[2] <= kBundleDim && fminf(-m[4] - m[0], -m[5] - m[1]) < kBundleNarrow &&
                            fminf(-m[6] - m[2], -m[7] - m[3]) < kBundleNarrow;
        // voxels [a0, a1] x [b0, b1] that the bundle covers between two planes
        int a0, a1, b0, b1;
        auto footprint = [&](int pa, int pb, int nA, int nB) {
            float fa = (float)pa - F0, fb = (float)pb - F0;
            if constexpr (STEP) {
                if (back) fa = pa == end ? F1 - F0 : fa;
                else fb = pb == end ? F1 - F0 : fb;
            }
            a0 = clamp0_i32(floor_i32(min_f32(fmaf(fa, A1, A0), fmaf(fb, A1, A0)) - kBundleSlack), nA - 1);
            a1 = clamp0_i32(floor_i32(kBundleSlack - min_f32(fmaf(fa, mA1, mA0), fmaf(fb, mA1, mA0))), nA - 1);
            b0 = clamp0_i32(floor_i32(min_f32(fmaf(fa, B1, B0), fmaf(fb, B1, B0)) - kBundleSlack), nB - 1);
            b1 = clamp0_i32(floor_i32(kBundleSlack - min_f32(fmaf(fa, mB1, mB0), fmaf(fb, mB1, mB0))), nB - 1);
        };
        // the material every ray is in, or kMixed, and the first plane of the
        // open stretch of mixed layers
        int prev = narrow ? (int)bg : kMixed, open = narrow ? -1 : (back ? P1 : P0);
        for (int base = narrow ? 0 : NB & ~63; base <= NB; base += 64) {
            // the layers of bricks, in travel order; behind the last one the
            // background
            const int t = base + lane;
            int code = (int)bg;
            const int bi = back ? bHi - 1 - t : bLo + t;
            if (narrow && t < NB) {
                const MXR_CONSTANT DevComp *const ph = again(comp);
                const RoleAxis xA = role_axis(ph, iA), xB = role_axis(ph, iB);
                const int all = role_axis(ph, 2).brick * (((int)ph->dims[2] + kBrick - 1) / kBrick);
                const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)bricks, (short)0, all, 0x00020000);
                const int pa = bi * kBrick;
                footprint(pa, pa + kBrick < xD.n ? pa + kBrick : xD.n, xA.n, xB.n);
                a0 /= kBrick, a1 /= kBrick, b0 /= kBrick, b1 /= kBrick;
                code = footprint_code<kBrickWide>(rb, (uint32_t)(bi * xD.brick + a0 * xA.brick + b0 * xB.brick), a1 - a0,
                                                  b1 - b0, xA.brick, xB.brick);
            }
            const int before = __builtin_amdgcn_update_dpp(prev, code, 0x138, 0xf, 0xf, false);  // wave_shr 1
            const uint64_t mixed = __builtin_amdgcn_ballot_w64(code == kMixed);
            uint64_t todo = narrow ? __builtin_amdgcn_ballot_w64((code == kMixed || code != before || t == NB) && t <= NB)
                                   : 1ull << (NB & 63);
            // the k-th mixed layer's number in lane k
            const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mixed >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mixed, 0u));
            const int count = __builtin_popcountll(mixed);
            const int slot = code == kMixed ? rank : count + lane - rank;
            const int nth = __builtin_amdgcn_ds_permute(4 * slot, bi);
            int k = 0, fine = kMixed, at = 0, shift = 0;
            uint32_t sub = 0;    // changes among the four layers of the mixed one at hand
            uint64_t turns = 0;  // voxel layers, of 16 mixed layers of bricks, that differ from the one before
            bool ended = false;
            while (true) {
                int c, plane;  // the next change: code and first plane of its layer
                if (sub != 0) {
                    const int u = __builtin_ctz(sub);
                    sub &= sub - 1;
                    c = __builtin_amdgcn_readlane(fine, shift + u);
                    const int pb = at * kBrick + kBrick < xD.n ? at * kBrick + kBrick : xD.n;
                    plane = back ? pb - u : at * kBrick + u;
                    if (c == kNoLayer) continue;
                } else {
                    if (todo == 0) break;
                    const int b = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    at = back ? bHi - 1 - (base + b) : bLo + base + b;
                    if ((mixed >> b) & 1) {
                        if ((k & 15) == 0) {
                            // look at the voxel layers of the next 16 mixed
                            // layers of bricks
                            const int kk = k + lane / kBrick, u = lane % kBrick;
                            const int lb = __builtin_amdgcn_ds_bpermute(4 * kk, nth);
                            const int lt = back ? bHi - 1 - lb : lb - bLo;
                            const int last = __builtin_amdgcn_ds_bpermute(4 * (lt - base), before);
                            const int pb = lb * kBrick + kBrick < xD.n ? lb * kBrick + kBrick : xD.n;
                            const int layer = back ? pb - 1 - u : lb * kBrick + u;
                            const int carry = __builtin_amdgcn_readlane(fine, 63);
                            fine = kNoLayer;
                            if (kk < count && layer >= lb * kBrick && layer < pb) {
                                const MXR_CONSTANT DevComp *const ph = again(comp);
                                const RoleAxis xA = role_axis(ph, iA), xB = role_axis(ph, iB);
                                const __amdgpu_buffer_rsrc_t rs =
                                    __builtin_amdgcn_make_buffer_rsrc((void *)ph->data0, (short)0, (int)ph->n0, 0x00020000);
                                footprint(layer, layer + 1, xA.n, xB.n);
                                fine = footprint_code<kBundleWide>(rs, (uint32_t)(layer * xD.str + a0 * xA.str + b0 * xB.str),
                                                                   a1 - a0, b1 - b0, xA.str, xB.str);
                            }
                            int ahead = __builtin_amdgcn_update_dpp(carry, fine, 0x138, 0xf, 0xf, false);  // wave_shr 1
                            if (u == 0 && last != kMixed) ahead = last;
                            turns = __builtin_amdgcn_ballot_w64(fine != ahead);
                        }
                        shift = (k & 15) * kBrick;
                        sub = (uint32_t)(turns >> shift) & 15u;
                        ++k;
                        continue;
                    }
                    c = __builtin_amdgcn_readlane(code, b);
                    ended = base + b == NB;
                    plane = ended ? (back ? P0 : P1) : (back ? (at * kBrick + kBrick < xD.n ? at * kBrick + kBrick : xD.n) : at * kBrick);
                }
                if (c == kMixed) {
                    open = open < 0 ? plane : open;
                    prev = kMixed;
                    continue;
                }
                if (open >= 0) {
                    // walk the stretch of mixed layers that ends here
                    if constexpr (STEP) {
                        const double u0 = pick3(iD, sp->u0[0], sp->u0[1], sp->u0[2]), du = pick3(iD, sp->du[0], sp->du[1], sp->du[2]);
                        const int js = step_at(open, back, end, u0, du, sp->J), je = step_at(plane, back, end, u0, du, sp->J);
                        if (part && je > js) stretch_steps(again(comp), *sp, js, je, a_vol, a_out, run, mu_row);
                    }
                    const double a0 = alpha_of(open), as = max_f64(a0, a_box), ae = min_f64(alpha_of(plane), z_box);
                    if (!STEP && part && ae > as)
                        stretch_walk<EXACT, kStretchRound, Run>(again(comp), iD, D, A, B, back, back ? open - 1 : open, as > a0, as,
                                                           ae, a_out, run, mu_row);
                    open = -1;
                }
                if (c != prev) {
                    // every ray enters material c at this plane, or (the
                    // background) has at the latest on leaving the box
                    if (part && run.m != (uint32_t)c) {
                        double t = 0.0;
                        if constexpr (STEP)
                            t = a_vol + (double)(step_at(plane, back, end, pick3(iD, sp->u0[0], sp->u0[1], sp->u0[2]),
                                                         pick3(iD, sp->du[0], sp->du[1], sp->du[2]), sp->J) - 1) * sp->h;
                        else
                            t = alpha_of(plane);
                        turn_run(run, t, z_box, (uint32_t)c, mu_row);
                    }
                    prev = c;
                }
            }
            if (ended) break;
        }
    }
    if constexpr (!ONE) {
        turn_run(run, a_out, a_out, run.m, mu_row);
        *hit_out = run.hit;
        return run.tau;
    }
    return add_run(run.mu, a_out - run.a_start, run.tau);
}

// ------------------------------------------------- scattering phantom ----
// Photons scattered exactly K times in the volume (section 3.3: the voxel
// sample models absorption and scattering), each interaction forced: on the
// chord ahead the total optical depth tau is taken by the exact walk, the
// depth tau* = -log(1 - u1 (1 - e^-tau)) is located by the same walk (in
// the material run where the running depth reaches tau*, at
// a_start + (tau* - tau_before) / mu), and the weight takes 1 - e^-tau,
// the scatter albedo
// (mu_R + mu_C) / mu_tot of the voxel's material and the angular factor;
// Rayleigh (Thomson law, no form factor) is chosen with probability
// mu_R / (mu_R + mu_C) (u2), Compton (Klein-Nishina, free electrons)
// otherwise, lowering E to E / (1 + k (1 - cos)).  Directions: uniform on
// the sphere (cos = 2 u3 - 1, phi = 2 pi u4 about the old direction, frame
// e1 = d x a / |d x a| with a = y unless |d_y| >= 1/2, then x, e2 = d x e1),
// weight 4 pi x the density per steradian; or, for the last interaction of
// an aimed phantom (flags bit 2), towards the point c + (2 u3 - 1) a +
// (2 u4 - 1) b of a target rectangle, weight = density / (dist^2 /
// (|n . d| 4 |a x b|)).  After the K-th interaction the walk to the exit
// attenuates at the final energy.  The total-attenuation channel is read
// from LDS (mu / 10 per mm, as for the plain phantom), the Rayleigh and
// Compton channels from the table in global memory at each interaction.
constexpr double kMeC2Kev = 510.99895;

// Klein-Nishina total cross section over 2 pi r_e^2
__device__ __forceinline__ double kn_f(double k) {
    const double l = log1p(2.0 * k);
    return ((1.0 + k) / (k * k)) * (2.0 * (1.0 + k) / (1.0 + 2.0 * k) - l / k) + l / (2.0 * k) -
           (1.0 + 3.0 * k) / ((1.0 + 2.0 * k) * (1.0 + 2.0 * k));
}

// Walk the chord from q along dl voxel by voxel (every plane crossing at
// alpha = (plane - q) / d with plane = corner + p v, as in the exact walk),
// summing mu * length segment by segment until the running optical depth
// reaches tau_star.  Returns true with the interaction distance s and the
// voxel's material (if rounding leaves tau_star beyond the last attenuating
// segment: the end of that segment); with tau_star = infinity it walks the
// whole chord and tau_out is the chord's optical depth.  False if the ray
// misses the volume.  Bounded by nx + ny + nz + 3 steps.
__device__ __forceinline__ bool siddon_locate(const PhantomGeo &g, const double q[3], const double dl[3],
                                              const double *__restrict__ mu_row, double tau_star, double &s_out,
                                              uint32_t &m_out, double &tau_out) {
    double inv[3], a_in = 0.0, a_out = kInf;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double lo_p = g.corner[i], hi_p = g.corner[i] + (double)g.n[i] * g.v;
        if (dl[i] == 0.0) {
            inv[i] = 0.0;
            if (!(q[i] > lo_p && q[i] < hi_p)) return false;
        } else {
            inv[i] = 1.0 / dl[i];
            const double a0 = (lo_p - q[i]) * inv[i], a1 = (hi_p - q[i]) * inv[i];
            const double lo = a0 < a1 ? a0 : a1, hi = a0 < a1 ? a1 : a0;
            if (lo > a_in) a_in = lo;
            if (hi < a_out) a_out = hi;
        }
    }
    if (!(a_out > a_in)) return false;
    int idx[3], p[3], st[3];
    double na[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int n = g.n[i];
        const double c = g.corner[i], v = g.v;
        if (dl[i] == 0.0) {
            const double f = floor((q[i] - c) / v);
            idx[i] = (int)fmin(fmax(f, 0.0), (double)(n - 1));
            p[i] = 0;
            st[i] = 0;
            na[i] = kInf;
            continue;
        }
        const double f = ((q[i] + a_in * dl[i]) - c) / v;
        if (dl[i] > 0.0) {
            int pp = (int)fmin(fmax(floor(f) + 1.0, 1.0), (double)n);
            if (pp > 1 && ((c + (double)(pp - 1) * v) - q[i]) * inv[i] > a_in) pp -= 1;
            if (pp < n && !(((c + (double)pp * v) - q[i]) * inv[i] > a_in)) pp += 1;
            idx[i] = pp - 1;
            p[i] = pp;
            st[i] = 1;
        } else {
            int pp = (int)fmin(fmax(ceil(f) - 1.0, 0.0), (double)(n - 1));
            if (pp < n - 1 && ((c + (double)(pp + 1) * v) - q[i]) * inv[i] > a_in) pp += 1;
            if (pp > 0 && !(((c + (double)pp * v) - q[i]) * inv[i] > a_in)) pp -= 1;
            idx[i] = pp;
            p[i] = pp;
            st[i] = -1;
        }
        na[i] = ((c + (double)p[i] * v) - q[i]) * inv[i];
    }
    // per-axis state in scalars (an array indexed by the crossing axis
    // would live in scratch memory)
    const int nx = g.n[0], nxy = g.n[0] * g.n[1];
    int i0 = idx[0], i1 = idx[1], i2 = idx[2];
    int p0 = p[0], p1 = p[1], p2 = p[2];
    double n0 = na[0], n1 = na[1], n2 = na[2];
    double a_prev = a_in, tc = 0.0, last_end = a_in;
    uint32_t last_m = 0;
    // the next voxel's load is issued before the current segment is summed
    // (its index does not depend on the material), hiding its latency
    uint32_t m = g.vol[i0 + nx * i1 + nxy * i2];
    const int max_steps = g.n[0] + g.n[1] + g.n[2] + 3;
    for (int step = 0; step < max_steps; ++step) {
        const int ax = (n1 < n0) ? ((n2 < n1) ? 2 : 1) : ((n2 < n0) ? 2 : 0);
        const double nmin = min_f64(n0, min_f64(n1, n2));  // the value of axis ax
        const double a_next = min_f64(nmin, a_out);
        const bool more = nmin < a_out;
        if (more) {
            // cross the plane: the next voxel along that axis (clamped)
            if (ax == 0) {
                i0 = clamp0_i32(i0 + st[0], g.n[0] - 1);
                p0 += st[0];
                n0 = ((g.corner[0] + (double)p0 * g.v) - q[0]) * inv[0];
            } else if (ax == 1) {
                i1 = clamp0_i32(i1 + st[1], g.n[1] - 1);
                p1 += st[1];
                n1 = ((g.corner[1] + (double)p1 * g.v) - q[1]) * inv[1];
            } else {
                i2 = clamp0_i32(i2 + st[2], g.n[2] - 1);
                p2 += st[2];
                n2 = ((g.corner[2] + (double)p2 * g.v) - q[2]) * inv[2];
            }
        }
        const uint32_t m_next = g.vol[i0 + nx * i1 + nxy * i2];
        const double mu = mu_row[m];
        if (mu > 0.0 && a_next > a_prev) {
            const double d = mu * (a_next - a_prev);
            last_m = m;
            last_end = a_next;
            if (tc + d >= tau_star) {
                s_out = a_prev + (tau_star - tc) / mu;
                m_out = m;
                tau_out = tc + d;
                return true;
            }
            tc = tc + d;
        }
        if (!more) break;
        m = m_next;
        a_prev = a_next;
    }
    s_out = last_end;
    m_out = last_m;
    tau_out = tc;
    return true;
}

// The scattering phantom component: par 4 = K; flags bit 2 aims the last
// interaction at the rectangle par 5..7 (centre), 8..10 and 11..13 (half
// axes), lab frame.  T: the three-channel table (1/cm) in global memory.
// The 2K + 1 walks (optical depth ahead, interaction point, ..., exit) run
// as passes of one loop (BUNDLE: the first two before it, by a full wave's
// bundle walk): the event walk in locate mode (tau_star infinite for
// the depth and exit passes) for the coherent chords, the voxel-by-voxel
// walk for the chords after an isotropic scatter.
template <bool EXACT, bool BUNDLE>
__device__ __forceinline__ bool comp_phantom_scatter(const DevComp &c, const DevInstr *ins, Stream &s, Ray &ray,
                                                     const double *mu_lds, uint32_t n_mat, uint32_t n_ebin) {
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    PhantomGeo g;
    g.vol = (const uint8_t *)c.data0;
    g.n[0] = (int)c.dims[0];
    g.n[1] = (int)c.dims[1];
    g.n[2] = (int)c.dims[2];
    g.v = c.par[0];
    g.rv = c.aux[6];
    g.corner[0] = c.aux[0];
    g.corner[1] = c.aux[1];
    g.corner[2] = c.aux[2];
    g.nvox = (uint32_t)c.n0;
    const double *__restrict__ T = (const double *)c.data1;
    const uint32_t plane = n_mat * n_ebin;
    const int K = (int)c.par[4];
    const bool aimed = (c.flags & 4u) != 0;
    double E = ray.E, w = ray.w, tau_star = kInf, pint = 0.0;
    int e = 0;
    WalkHit hit;
    // the primary chords of a full wave are walked as a bundle, both passes
    const bool bundle = BUNDLE && __builtin_amdgcn_ballot_w64(true) == ~0ull;
    if (bundle) {
        e = (int)fmin(fmax(floor((E - c.par[1]) * c.aux[3]), 0.0), (double)(n_ebin - 1));
        const double *mu_row = mu_lds + e * n_mat;
        double inv[3], a_in, a_out;
        bool in = volume_chord(g, q, dl, inv, a_in, a_out);
        const MXR_CONSTANT DevComp *const cc = (const MXR_CONSTANT DevComp *)&c;
        const MXR_CONSTANT uint8_t *const bricks = (const MXR_CONSTANT uint8_t *)ins->bricks;
        // (one copy of the walk, the first time for a depth that no path has)
        double tau = 0.0;
        for (int look = 0; look < 2; ++look) {
            hit = WalkHit();
            const double t = bundle_tau<EXACT, false, FindRun>(cc, bricks, q, dl, inv, a_in, a_out, in, mu_row, nullptr,
                                                               tau_star, &hit);
            if (look) break;
            tau = t;
            in = in && tau > 0.0;
            pint = -expm1(-tau);
            tau_star = -log1p(-s.u((int)c.draw0) * pint);
        }
        if (!in) return false;
    }
    for (int pass = bundle ? 1 : 0; pass <= 2 * K; ++pass) {
        const int k = pass >> 1;
        const bool locate = (pass & 1) != 0;
        if (!locate) {
            const double f = floor((E - c.par[1]) * c.aux[3]);
            e = (int)fmin(fmax(f, 0.0), (double)(n_ebin - 1));
            tau_star = kInf;
        }
        // chords along the primary or towards the target are coherent
        // across a wave and take the event walk; chords after an isotropic
        // scatter go voxel by voxel
        const bool coherent = k == 0 || (k == K && aimed);
        double tau = 0.0;
        if (bundle && pass == 1) {
        } else if (coherent) {
            hit = WalkHit();
            tau = siddon_tau<EXACT, true>(g, q, dl, mu_lds + e * n_mat, tau_star, &hit);
        } else {
            hit = WalkHit();
            double sl = 0.0;
            uint32_t ml = 0;
            if (siddon_locate(g, q, dl, mu_lds + e * n_mat, tau_star, sl, ml, tau)) {
                hit.found = sl >= 0.0 && tau_star < kInf;
                hit.s = sl;
                hit.m = ml;
                hit.last_end = sl;
                hit.last_m = ml;
            }
        }
        if (pass == 2 * K) {  // the exit walk
            ray.E = E;
            ray.w = w * exp(-tau);
            break;
        }
        if (!locate) {
            // optical depth ahead: draw the forced interaction depth
            if (!(tau > 0.0)) return false;
            pint = -expm1(-tau);
            tau_star = -log1p(-s.u((int)c.draw0 + 4 * k) * pint);
            continue;
        }
        const double sint = hit.found ? hit.s : hit.last_end;
        const uint32_t m = hit.found ? hit.m : hit.last_m;
#pragma unroll
        for (int i = 0; i < 3; ++i) q[i] = q[i] + sint * dl[i];
        const double mu_t = T[m * n_ebin + e];
        const double mu_r = T[plane + m * n_ebin + e];
        const double mu_c = T[2 * plane + m * n_ebin + e];
        if (!(mu_r + mu_c > 0.0)) return false;
        const double albedo = (mu_r + mu_c) / mu_t;
        const bool rayleigh = s.u((int)c.draw0 + 4 * k + 1) < mu_r / (mu_r + mu_c);
        double ct = 2.0 * s.u((int)c.draw0 + 4 * k + 2) - 1.0;
        const double phi = kTwoPi * s.u((int)c.draw0 + 4 * k + 3);
        double nd[3], dens_ratio = 4.0 * kPi;
        if (aimed && k == K - 1) {
            double tw[3], tl[3], ta[3], tb[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) tw[i] = c.par[5 + i] - c.pos[i];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                tl[i] = c.rot[3 * i] * tw[0] + c.rot[3 * i + 1] * tw[1] + c.rot[3 * i + 2] * tw[2];
                ta[i] = c.rot[3 * i] * c.par[8] + c.rot[3 * i + 1] * c.par[9] + c.rot[3 * i + 2] * c.par[10];
                tb[i] = c.rot[3 * i] * c.par[11] + c.rot[3 * i + 1] * c.par[12] + c.rot[3 * i + 2] * c.par[13];
            }
            const double sa = 2.0 * s.u((int)c.draw0 + 4 * k + 2) - 1.0;
            const double sb = 2.0 * s.u((int)c.draw0 + 4 * k + 3) - 1.0;
            double r[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) r[i] = (tl[i] + sa * ta[i] + sb * tb[i]) - q[i];
            const double dist2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
            const double dist = sqrt(dist2);
            const double nrm0 = ta[1] * tb[2] - ta[2] * tb[1], nrm1 = ta[2] * tb[0] - ta[0] * tb[2],
                         nrm2 = ta[0] * tb[1] - ta[1] * tb[0];
            const double area4 = sqrt(nrm0 * nrm0 + nrm1 * nrm1 + nrm2 * nrm2);
            if (!(dist > 0.0) || !(area4 > 0.0)) return false;
#pragma unroll
            for (int i = 0; i < 3; ++i) nd[i] = r[i] / dist;
            const double cosn = fabs(nd[0] * nrm0 + nd[1] * nrm1 + nd[2] * nrm2) / area4;
            if (!(cosn > 0.0)) return false;
            dens_ratio = (cosn * 4.0 * area4) / dist2;
            ct = dl[0] * nd[0] + dl[1] * nd[1] + dl[2] * nd[2];
        } else {
            double a0 = 0.0, a1 = 1.0;
            if (!(fabs(dl[1]) < 0.5)) {
                a0 = 1.0;
                a1 = 0.0;
            }
            // e1 = d x a with a = (a0, a1, 0)
            double e1[3] = {dl[1] * 0.0 - dl[2] * a1, dl[2] * a0 - dl[0] * 0.0, dl[0] * a1 - dl[1] * a0};
            const double n1 = sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) e1[i] = e1[i] / n1;
            const double e2[3] = {dl[1] * e1[2] - dl[2] * e1[1], dl[2] * e1[0] - dl[0] * e1[2],
                                  dl[0] * e1[1] - dl[1] * e1[0]};
            const double sn = sqrt(1.0 - ct * ct);
            double sp, cp;
            sincos(phi, &sp, &cp);
#pragma unroll
            for (int i = 0; i < 3; ++i) nd[i] = ct * dl[i] + sn * (cp * e1[i] + sp * e2[i]);
        }
        const double st2 = 1.0 - ct * ct;
        double dens;
        if (rayleigh) {
            dens = 3.0 * (1.0 + ct * ct) / (16.0 * kPi);
        } else {
            const double kk = E / kMeC2Kev;
            const double rho = 1.0 / (1.0 + kk * (1.0 - ct));
            dens = rho * rho * (rho + 1.0 / rho - st2) / (4.0 * kPi * kn_f(kk));
            E = rho * E;
        }
        w = w * (pint * albedo * (dens * dens_ratio));
#pragma unroll
        for (int i = 0; i < 3; ++i) dl[i] = nd[i];
    }
    to_lab(c, q, dl, ray);
    return true;
}

// ------------------------------------------------------------- mirror ----
__device__ __forceinline__ bool comp_mirror(const DevComp &c, Ray &ray) {
    // aux: 0 Cy, 1 Cz, 2 uy, 3 uz, 4 vy, 5 vz, 6 1/a^2, 7 1/b^2,
    //      8 sin t0, 9 cos t0, 10 length/2, 11 width/2, 12 node step
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    const double Cy = c.aux[0], Cz = c.aux[1], uy = c.aux[2], uz = c.aux[3], vy = c.aux[4], vz = c.aux[5];
    const double ia2 = c.aux[6], ib2 = c.aux[7];
    double gy = q[1] - Cy, gz = q[2] - Cz;
    double s0 = gy * uy + gz * uz, n0 = gy * vy + gz * vz;
    double ds = dl[1] * uy + dl[2] * uz, dn = dl[1] * vy + dl[2] * vz;
    double A = ds * ds * ia2 + dn * dn * ib2;
    double B = 2.0 * (s0 * ds * ia2 + n0 * dn * ib2);
    double C = s0 * s0 * ia2 + n0 * n0 * ib2 - 1.0;
    double disc = B * B - 4.0 * A * C;
    if (!(disc >= 0.0)) return false;
    double t = (-B + sqrt(disc)) / (2.0 * A);
    if (!(t > 0.0)) return false;
    double X[3] = {q[0] + t * dl[0], q[1] + t * dl[1], q[2] + t * dl[2]};
    double along = X[1] * c.aux[8] + X[2] * c.aux[9];
    if (!(fabs(X[0]) <= c.aux[11] && fabs(along) <= c.aux[10])) return false;
    double hy = X[1] - Cy, hz = X[2] - Cz;
    double hs = (hy * uy + hz * uz) * ia2, hn = (hy * vy + hz * vz) * ib2;
    double N1 = hs * uy + hn * vy, N2 = hs * uz + hn * vz;
    double nn = sqrt(0.0 * 0.0 + N1 * N1 + N2 * N2);
    N1 = N1 / nn;
    N2 = N2 / nn;
    double dd = dl[0] * 0.0 + dl[1] * N1 + dl[2] * N2;
    if (dd > 0.0) {
        N1 = -N1;
        N2 = -N2;
        dd = -dd;
    }
    double theta = asin(-dd);
    const double *tab = (const double *)c.data0;
    const int64_t nt = (int64_t)c.n0;
    double R = 0.0;
    double uu = theta / c.aux[12];
    if (uu <= (double)(nt - 1)) {
        int64_t k = (int64_t)floor(uu);
        if (k > nt - 2) k = nt - 2;
        double f = uu - (double)k;
        R = tab[k] * (1.0 - f) + tab[k + 1] * f;
    }
    double out[3] = {dl[0] - 2.0 * dd * 0.0, dl[1] - 2.0 * dd * N1, dl[2] - 2.0 * dd * N2};
    ray.w = ray.w * R;
    to_lab(c, X, out, ray);
    return true;
}

// --------------------------------------------------------- crystals ----
__device__ __forceinline__ double darwin(double x) {
    double ax = fabs(x);
    if (ax <= 1.0) return 1.0;
    double den = ax + sqrt(ax * ax - 1.0);
    return 1.0 / (den * den);
}

__device__ __forceinline__ bool bragg(double q[3], double dl[3], const double P[3], const double N[3],
                                      double th_b, double half_w, double &R) {
    double dn = dl[0] * N[0] + dl[1] * N[1] + dl[2] * N[2];
    if (!(dn < 0.0)) return false;
    double rel0 = q[0] - P[0], rel1 = q[1] - P[1], rel2 = q[2] - P[2];
    double t = -(rel0 * N[0] + rel1 * N[1] + rel2 * N[2]) / dn;
    if (!(t >= 0.0)) return false;
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = q[i] + t * dl[i];
    double th_in = asin(-dn);
    R = darwin((th_in - th_b) / half_w);
#pragma unroll
    for (int i = 0; i < 3; ++i) dl[i] = dl[i] - 2.0 * dn * N[i];
    return true;
}

__device__ __forceinline__ bool comp_dcm(const DevComp &c, Ray &ray) {
    // aux: 0..2 n1, 3..5 n2 = -n1, 6..8 crystal-2 point, 9 2d, 10 width/2
    double q[3], dl[3], R1, R2;
    to_local(c, ray, q, dl);
    const double P1[3] = {0.0, 0.0, 0.0};
    const double th_b = asin(kHc / (c.aux[9] * ray.E));  // both crystals' Bragg angle
    if (!bragg(q, dl, P1, c.aux + 0, th_b, c.aux[10], R1)) return false;
    if (!bragg(q, dl, c.aux + 6, c.aux + 3, th_b, c.aux[10], R2)) return false;
    ray.w = ray.w * R1;
    ray.w = ray.w * R2;
    to_lab(c, q, dl, ray);
    return true;
}

// ------------------------------------------------------------- powder ----
__device__ __forceinline__ bool comp_powder(const DevComp &c, Stream &s, Ray &ray) {
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    if (!plane_z0(q, dl)) return false;
    if (!(fabs(q[0]) <= c.aux[0] && fabs(q[1]) <= c.aux[1])) return false;
    const double *dsp = (const double *)c.data0;
    const int64_t nd = (int64_t)c.n0;
    int64_t j = (int64_t)floor((double)nd * s.u((int)c.draw0));
    if (j > nd - 1) j = nd - 1;
    double lambda = kHc / ray.E;
    double sarg = lambda / (2.0 * dsp[j]);
    if (!(sarg <= 1.0)) return false;
    double e1x = -dl[2], e1z = dl[0];
    double n1 = sqrt(e1x * e1x + 0.0 * 0.0 + e1z * e1z);
    e1x = e1x / n1;
    e1z = e1z / n1;
    const double e1y = 0.0;
    double e2x = dl[1] * e1z - dl[2] * e1y;
    double e2y = dl[2] * e1x - dl[0] * e1z;
    double e2z = dl[0] * e1y - dl[1] * e1x;
    // the cone angle 2 asin(sarg) by its sine and cosine (1 - sarg is exact where
    // 1 - sarg^2 would cancel, near backscattering)
    const double st = 2.0 * sarg * sqrt((1.0 - sarg) * (1.0 + sarg)), ct = 1.0 - 2.0 * (sarg * sarg);
    double se, ce;
    sincos_turn(s.u((int)c.draw0 + 1), se, ce);
    double out[3] = {ct * dl[0] + st * (ce * e1x + se * e2x), ct * dl[1] + st * (ce * e1y + se * e2y),
                     ct * dl[2] + st * (ce * e1z + se * e2z)};
    to_lab(c, q, out, ray);
    return true;
}

// ----------------------------------------------------------- monitors ----
__device__ __forceinline__ int64_t bin_of(double x, double lo, double scale, uint32_t n) {
    double f = floor((x - lo) * scale);
    if (!(f >= 0.0 && f < (double)n)) return -1;
    return (int64_t)f;
}

// Pixel (ix, iy) in which a ray reaches the monitor's plane (false: it misses
// the pixels or cannot reach the plane), and the energy (or wavelength) bin:
// comp_detector in two parts, on the same numbers.
__device__ __forceinline__ bool detector_pixel(const DevComp &c, const Ray &ray, uint32_t &ix, uint32_t &iy) {
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    if (!plane_z0(q, dl)) return false;
    const int64_t bx = bin_of(q[0], c.par[0], c.aux[0], c.dims[0]);
    const int64_t by = bin_of(q[1], c.par[2], c.aux[1], c.dims[1]);
    ix = (uint32_t)bx;
    iy = (uint32_t)by;
    return bx >= 0 && by >= 0;
}

// Whether every ray of the cone-beam source src whose place (ca, cb) in the
// source's square lies within (ha, hb) of (ca0, cb0) misses the monitor's
// pixels (no component between them deflects).  The concentric map moves a
// point by at most 1.4 times what its argument moves (its Jacobian's largest
// singular value is 1.383), the map of the disk onto the cone by at most
// 2 s / cos(alpha/2), s = sin(alpha/2), and a rotation's rows bound the rest;
// the rays' places on the plane then lie in a box around the middle one's.
__device__ __forceinline__ bool bundle_misses(const DevComp &src, const DevComp &det, double ca0, double cb0, double ha,
                                              double hb) {
    double rad, sa, cs;
    concentric(ca0, cb0, rad, sa, cs);
    const double s = src.aux[0], c2 = 1.0 - s * s;
    if (!(c2 > 1e-6)) return false;
    const double sh = fabs(rad) * s, k = 2.0 * s * sqrt(1.0 - sh * sh);
    const double dir[3] = {k * (rad * cs), k * (rad * sa), 1.0 - 2.0 * (sh * sh)};
    const double eps = (2.0 * s / sqrt(c2)) * (1.4 * sqrt(ha * ha + hb * hb)) + 1e-12;
    Ray ray;
    from_origin(src, dir, ray);
    double q[3], dl[3], err[3];
    to_local(det, ray, q, dl);
    double src_norm = 0.0;
    for (int i = 0; i < 9; ++i) src_norm = src_norm + src.rot[i] * src.rot[i];
    for (int i = 0; i < 3; ++i) {
        const double *R = det.rot + 3 * i;
        err[i] = sqrt((R[0] * R[0] + R[1] * R[1] + R[2] * R[2]) * src_norm) * eps;
    }
    if (dl[2] + err[2] <= 0.0 || q[2] > 0.0) return true;  // none reaches the plane moving forward
    const double low = dl[2] - err[2];
    if (!(low > 0.0)) return false;
    for (int i = 0; i < 2; ++i) {
        const double ratio = dl[i] / dl[2];
        const double off = fabs(q[2]) * ((err[i] + fabs(ratio) * err[2]) / low);
        const double x = q[i] - q[2] * ratio, slack = off + 1e-9 * (fabs(q[i]) + fabs(x) + off);
        if (x + slack < det.par[2 * i] || x - slack > det.par[2 * i + 1]) return true;
    }
    return false;
}
__device__ __forceinline__ int64_t detector_energy_bin(const DevComp &c, double E) {
    return bin_of((c.flags & 1u) ? kHc / E : E, c.par[4], c.aux[2], c.dims[2]);
}

// returns false if the ray cannot reach the plane; bin = -1 outside
__device__ __forceinline__ bool comp_detector(const DevComp &c, Ray &ray, int64_t &bin) {
    // aux: 0 nx/(xmax-xmin), 1 ny/(ymax-ymin), 2 ne/(emax-emin)
    double q[3], dl[3];
    to_local(c, ray, q, dl);
    if (!plane_z0(q, dl)) return false;
    double ev = (c.flags & 1u) ? kHc / ray.E : ray.E;
    int64_t ix = bin_of(q[0], c.par[0], c.aux[0], c.dims[0]);
    int64_t iy = bin_of(q[1], c.par[2], c.aux[1], c.dims[1]);
    int64_t ie = bin_of(ev, c.par[4], c.aux[2], c.dims[2]);
    bin = (ix >= 0 && iy >= 0 && ie >= 0) ? (iy * (int64_t)c.dims[0] + ix) * (int64_t)c.dims[2] + ie : -1;
    to_lab(c, q, dl, ray);
    return true;
}

}  // namespace mxr
