// HIP kernels of the DiffUS fan-beam renderer for MI355X (gfx950, CDNA4).
//
// Method: arXiv 2508.06768.  Per ray, Eq. 1 coefficients between consecutive
// trilinear samples, the coupled amplitude system of Eq. 2-4 solved for every
// truncation depth (Sec. 2.4), pixel = first difference of the echo d_0^(k),
// fan geometry, speckle and depth-dependent lateral blur (Sec. 2.4).
//
// The truncated systems are solved through the 2x2 transfer maps of the
// back-substitution: with Gamma = d/g,
//   Gamma_i = (A Gamma_{i+1} + R) / (B Gamma_{i+1} + 1),
//   M_i = [[A, R], [B, 1]],  A = a^2 (T T' - R R'),  B = -a^2 R',
// and P_k = M_0 ... M_{k-1}.  Only the bottom row v_k = [0 1] P_k and
// D_k = det P_k are needed:
//   e_{k+1} = R_k D_k / (v_k[1] v_{k+1}[1]),  v_{k+1}[1] = v_k[0] R_k + v_k[1],
// which is the exact first difference P01/P11 |_{k+1} - P01/P11 |_k without
// subtracting nearly equal numbers.  With R = rho and R' = s rho (s = +1 for
// the |R| of Eq. 1, -1 for the signed coefficient), T T' = 1 - rho^2, so one
// number per interface describes M.
//
// Layout of the work: one wavefront per ray.  A ray is cut into tiles of
// T = 64 C samples.  Phase 1 gathers 64 consecutive samples per instruction
// (good L1/L2 locality) and parks them in LDS in FP64.  Phase 2 gives each
// lane C consecutive interfaces: rho in registers, chunk product, 6-step
// wavefront scan of 2x2 products, carry between tiles, walk emitting pixels.
// The recurrence runs in FP64 (full rate on CDNA4 vector ALUs): the |R|
// convention makes the system nearly singular on some rays, where FP32 would
// lose the 1e-5 agreement with the reference.
//
// The adjoint kernel gathers the samples again, takes the states the forward
// recorded (or forms them itself), and runs the reverse recurrence as two
// sums over the deeper interfaces.  dL/dZ per sample goes to a scatter kernel
// that adds it into the volume gradient with FP32 atomics; pose gradients are
// reduced per ray in FP64.
#include <algorithm>
#include <math.h>
#include <mutex>
#include <stdint.h>

#include "../../include/diffus.h"
#include "dus_internal.h"

namespace dus {
namespace {

// --------------------------------------------------------------------------
// wavefront helpers
// --------------------------------------------------------------------------
__device__ __forceinline__ double lane_read(double x, int l)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b & 0xffffffffll), l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// a wave-uniform double made visibly uniform to the compiler (kept in SGPRs)
__device__ __forceinline__ double uniform(double x)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b & 0xffffffffll));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// the wavefront's own LDS traffic ordered (its lanes run in step and its LDS
// accesses complete in order: only the compiler has to be held)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adjoint with one wavefront per ray: four neighbouring rays share a block,
// and so a CU's L1, where their stencils mostly meet (64 x 256 x 1024: 132 us,
// against 138 us with one ray per block and 140 us with eight; the forward,
// which issues more per load, is as fast with one, 120 us, as with four).
constexpr int kBlockRays = 4;
constexpr int adjoint_waves(int w) { return w == 1 ? kBlockRays : w; }

// a barrier among the W wavefronts of a ray
template <int W>
__device__ __forceinline__ void ray_sync()
{
    if (W == 1) wave_sync();
    else __syncthreads();
}

__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
    return x;
}

__device__ __forceinline__ double wave_min(double x)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x = fmin(x, __shfl_xor(x, d));
    return x;
}

// FP64 reciprocal: hardware estimate refined by one Newton step (the step
// squares the estimate's relative error: below 2^-44 even for a
// single-precision estimate)
__device__ __forceinline__ double rcp64(double b)
{
    const double r = __builtin_amdgcn_rcp(b);
    return fma(fma(-b, r, 1.0), r, r);
}

// a / b correctly rounded but for the last place, from ib = rcp64(b): the
// quotient's residual corrects it (as it stands, rcp64 is good to 2^-48.7;
// next to a pole of the echo the recurrence magnifies that)
__device__ __forceinline__ double quot64(double a, double b, double ib)
{
    const double q = a * ib;
    return fma(fma(-b, q, a), ib, q);
}

// partial unroll of the sample-gather loops: enough independent gathers in
// flight without holding every tile sample in registers
#ifndef GATHER_UNROLL
#define GATHER_UNROLL 4
#endif

// blocks are handed to the 8 XCDs round-robin; keep runs of `grp`
// consecutive rays (neighbours in the fan, sharing voxels) on one XCD's L2
__device__ __forceinline__ int remap_block(int b, int G, int grp)
{
    if (grp <= 1) return b;
    const int super = 8 * grp;
    const int full = (G / super) * super;
    if (b >= full) return b;
    const int s = b / super, r = b - s * super;
    return s * super + (r & 7) * grp + (r >> 3);
}

__device__ __forceinline__ int find_fan(const FanTable &t, int g)
{
    int lo = 0, hi = t.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (t.f[mid].ray_begin <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ int find_blur_fan(const FanTable &t, int b)
{
    int lo = 0, hi = t.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (t.f[mid].blk_begin <= b) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// --------------------------------------------------------------------------
// geometry: probe pose -> per-ray affine sample positions in voxel units
// --------------------------------------------------------------------------
__device__ void rotation(const double w[3], double R[9])
{
    const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    const double th = sqrt(th2);
    double A, B;
    if (th < 1e-4) {
        A = 1.0 - th2 / 6.0;
        B = 0.5 - th2 / 24.0;
    } else {
        double sn, cs;
        sincos(th, &sn, &cs);
        A = sn / th;
        B = (1.0 - cs) / th2;
    }
    // R = I + A [w]x + B [w]x^2, [w]x^2 = w w^T - |w|^2 I
    R[0] = 1.0 + B * (w[0] * w[0] - th2);
    R[1] = -A * w[2] + B * w[0] * w[1];
    R[2] = A * w[1] + B * w[0] * w[2];
    R[3] = A * w[2] + B * w[1] * w[0];
    R[4] = 1.0 + B * (w[1] * w[1] - th2);
    R[5] = -A * w[0] + B * w[1] * w[2];
    R[6] = -A * w[1] + B * w[2] * w[0];
    R[7] = A * w[0] + B * w[2] * w[1];
    R[8] = 1.0 + B * (w[2] * w[2] - th2);
}

struct Ray {
    double u0[3], du[3];   // voxel coordinate of sample 0 and per-sample step
    double a2;             // round-trip amplitude over one step
    double dirx, dirz;     // probe-frame direction (y component is 0)
    double r0, ds;
    // orthonormal basis, world frame: the ray's direction D, its in-plane
    // normal T = R (cz, 0, -sx) and the fan plane's normal N = R (0, 1, 0),
    // each component over the voxel spacing of its axis
    double bd[3], bt[3], bn[3];
    // set_base: the voxel that VolArgs::Z points to after it, and whether all of
    // the ray's samples lie within 4 GiB of it
    unsigned first;
    bool narrow;
};

// wave_uniform: every lane of the wavefront traces the same ray (its
// parameters are then kept in scalar registers)
__device__ __forceinline__ void setup_ray(const VolArgs &v, const PhysArgs &p, const FanRec &fr,
                                          const float *__restrict__ poses, int j, Ray &ray,
                                          bool wave_uniform = true)
{
    const float *ps = poses + 6 * (size_t)fr.pose;
    const double t[3] = {ps[0], ps[1], ps[2]};
    const double w[3] = {ps[3], ps[4], ps[5]};
    double R[9];
    rotation(w, R);
    const double A = fr.aperture;
    const double th = fr.n_rays > 1 ? -0.5 * A + (double)j * A / (double)(fr.n_rays - 1) : 0.0;
    double sx, cz;
    sincos(th, &sx, &cz);
    const double d[3] = {R[0] * sx + R[2] * cz, R[3] * sx + R[5] * cz, R[6] * sx + R[8] * cz};
    const double r0 = fr.r0, ds = fr.ds;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double ih = 1.0 / (double)v.h[a];
        ray.u0[a] = (t[a] + r0 * d[a] - (double)v.o[a]) * ih;
        ray.du[a] = ds * d[a] * ih;
        ray.bd[a] = d[a] * ih;
        ray.bt[a] = (R[3 * a] * cz - R[3 * a + 2] * sx) * ih;
        ray.bn[a] = R[3 * a + 1] * ih;
    }
    const double amp = (p.atten == 0)
                           ? exp10(-(double)p.alpha * (double)p.freq * (ds / 10.0) / 20.0)
                           : 1.0;
    ray.a2 = amp * amp;
    ray.dirx = sx;
    ray.dirz = cz;
    ray.r0 = r0;
    ray.ds = ds;
    if (!wave_uniform) return;
    // every lane computed the same values: keep them in scalar registers
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ray.u0[a] = uniform(ray.u0[a]);
        ray.du[a] = uniform(ray.du[a]);
    }
    ray.a2 = uniform(ray.a2);
    ray.dirx = uniform(ray.dirx);
    ray.dirz = uniform(ray.dirz);
    ray.r0 = uniform(ray.r0);
    ray.ds = uniform(ray.ds);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ray.bd[a] = uniform(ray.bd[a]);
        ray.bt[a] = uniform(ray.bt[a]);
        ray.bn[a] = uniform(ray.bn[a]);
    }
}

// the ray's geometry, as the forward hands it to the adjoint (one lane)
__device__ __forceinline__ void store_geom(const Ray &ray, RayGeom *__restrict__ q)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q->u0[a] = ray.u0[a];
        q->du[a] = ray.du[a];
        q->bd[a] = ray.bd[a];
        q->bt[a] = ray.bt[a];
        q->bn[a] = ray.bn[a];
    }
    q->a2 = ray.a2;
    q->dirx = ray.dirx;
    q->dirz = ray.dirz;
}

// (q is the same on every lane: scalar loads; made opaque, so that each call
// loads again)
__device__ __forceinline__ void load_basis(const RayGeom *__restrict__ q, Ray &ray)
{
    asm volatile("" : "+s"(q));
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ray.bd[a] = q->bd[a];
        ray.bt[a] = q->bt[a];
        ray.bn[a] = q->bn[a];
    }
    ray.dirx = q->dirx;
    ray.dirz = q->dirz;
}

__device__ __forceinline__ void load_geom(const FanRec &fr, const RayGeom *__restrict__ q, Ray &ray)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        ray.u0[a] = q->u0[a];
        ray.du[a] = q->du[a];
    }
    ray.a2 = q->a2;
    ray.r0 = fr.r0;
    ray.ds = fr.ds;
}

// cell index (clamped) and fraction along one axis; NaN positions clamp to 0.
// INSIDE: the caller knows u lies in [0, n-1), where the clamps change
// nothing.  u >= 0 in both cases, so truncation is the floor.
template <bool INSIDE>
__device__ __forceinline__ void axis_cell(double u, int n, int &i0, double &f)
{
    const double uc = INSIDE ? u : fmin(fmax(u, 0.0), (double)(n - 1));
    const int i = INSIDE ? (int)uc : min((int)uc, n - 2);
    i0 = i;
    // inside, u - floor(u) is exact and one instruction
    f = INSIDE ? __builtin_amdgcn_fract(uc) : uc - (double)i;
}

struct Stencil {
    int idx;               // flat index of the (x0, y0, z0) corner
    int ix, iy, iz;        // that corner's voxel coordinates
    double fx, fy, fz;
};

// a slice of the volume holds fewer than 2^24 voxels (checked on the host),
// so the flat index takes two independent 24-bit multiplies
template <bool INSIDE = false>
__device__ __forceinline__ Stencil stencil_at(const VolArgs &v, const Ray &ray, int k)
{
    Stencil s;
    const double kk = (double)k;
    axis_cell<INSIDE>(fma(kk, ray.du[0], ray.u0[0]), v.nx, s.ix, s.fx);
    axis_cell<INSIDE>(fma(kk, ray.du[1], ray.u0[1]), v.ny, s.iy, s.fy);
    axis_cell<INSIDE>(fma(kk, ray.du[2], ray.u0[2]), v.nz, s.iz, s.fz);
    s.idx = (int)(__umul24((unsigned)s.iz, (unsigned)(v.nx * v.ny)) + __umul24((unsigned)s.iy, (unsigned)v.nx)) + s.ix;
    return s;
}

// every sample k in [ka, kb] lies in [0, n-1) on every axis: the position is
// affine in k and its FP64 rounding is monotone, so the two ends decide
__device__ __forceinline__ bool segment_inside(const VolArgs &v, const Ray &ray, int ka, int kb)
{
    const int n[3] = {v.nx, v.ny, v.nz};
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double ua = fma((double)ka, ray.du[a], ray.u0[a]);
        const double ub = fma((double)kb, ray.du[a], ray.u0[a]);
        const double hi = (double)(n[a] - 1);
        in = in && (ua >= 0.0) && (ua < hi) && (ub >= 0.0) && (ub < hi);
    }
    return in;
}

__device__ __forceinline__ double lerp(double a, double b, double t) { return fma(t, b - a, a); }

// two neighbouring voxels, at any multiple of 4 bytes
typedef float float2_u __attribute__((ext_vector_type(2), aligned(4)));

// Gathers address the volume from Z with 32-bit offsets (a 64-bit address per
// row takes an add each).  A volume of up to 4 GiB is within reach from its
// start; in a larger one Z moves to the lowest slice the ray's samples touch,
// which serves if they span no more than 4 GiB (`narrow`; else, and where
// tiles are clamped, the offsets have 64 bits).  1100 x 1024 x 1024 voxels, 16
// poses x 256 x 1024, every tile clamped with 64 bits / so: forward 102 / 89 us,
// pose adjoint 210 / 185; inside with 64 bits 102 / 213.
__host__ __device__ inline bool in_reach(const VolArgs &v) { return (long long)v.nx * v.ny * v.nz <= (1ll << 30); }

__device__ __forceinline__ void set_base(VolArgs &v, Ray &ray, int S)
{
    ray.first = 0;
    ray.narrow = true;
    if (in_reach(v)) return;
    const int sxy = v.nx * v.ny;
    int za, zb;
    double f;
    axis_cell<false>(ray.u0[2], v.nz, za, f);
    axis_cell<false>(fma((double)(S - 1), ray.du[2], ray.u0[2]), v.nz, zb, f);
    const int lo = __builtin_amdgcn_readfirstlane(min(za, zb)), hi = __builtin_amdgcn_readfirstlane(max(za, zb));
    ray.first = (unsigned)lo * (unsigned)sxy;
    ray.narrow = (long long)(hi + 2 - lo) * sxy <= (1ll << 30);
    v.Z += ray.first;
}

// voxels idx and idx + 1 of the row that Z points into, `first` voxels on
// (NARROW: 32-bit offsets)
template <bool NARROW>
__device__ __forceinline__ float2_u voxel_pair(const float *__restrict__ Z, int idx, unsigned first)
{
    if (NARROW)         // (the subtraction goes with the shift)
        return *reinterpret_cast<const float2_u *>(reinterpret_cast<const char *>(Z) +
                                                   (((unsigned)idx << 2) - (first << 2)));
    return *reinterpret_cast<const float2_u *>(Z + ((unsigned)idx - first));
}

// trilinear value (lerp along x, then y, then z), FP64 from FP32 corners
template <bool NARROW = false>
__device__ __forceinline__ double trilinear(const float *__restrict__ Z, int nx, int sxy,
                                            const Stencil &s, double *grad, unsigned first = 0)
{
    const float2_u p00 = voxel_pair<NARROW>(Z, s.idx, first), p10 = voxel_pair<NARROW>(Z + nx, s.idx, first);
    const float2_u p01 = voxel_pair<NARROW>(Z + sxy, s.idx, first);
    const float2_u p11 = voxel_pair<NARROW>(Z + sxy + nx, s.idx, first);
    const double c000 = p00.x, c100 = p00.y;
    const double c010 = p10.x, c110 = p10.y;
    const double c001 = p01.x, c101 = p01.y;
    const double c011 = p11.x, c111 = p11.y;
    const double a00 = lerp(c000, c100, s.fx), a10 = lerp(c010, c110, s.fx);
    const double a01 = lerp(c001, c101, s.fx), a11 = lerp(c011, c111, s.fx);
    const double b0 = lerp(a00, a10, s.fy), b1 = lerp(a01, a11, s.fy);
    if (grad) {
        const double gx0 = lerp(c100 - c000, c110 - c010, s.fy);
        const double gx1 = lerp(c101 - c001, c111 - c011, s.fy);
        grad[0] = lerp(gx0, gx1, s.fz);
        grad[1] = lerp(a10 - a00, a11 - a01, s.fz);
        grad[2] = b1 - b0;
    }
    return lerp(b0, b1, s.fz);
}

// Eq. 1 reflection coefficient between samples zl (shallower) and zr; dq
// (optional) receives d rho/d zr = dq zl and d rho/d zl = -dq zr, i.e.
// dq = 2 s / (zl + zr)^2 with s = sign(zr - zl) (ABS, sign(0) = 0) or 1
__device__ __forceinline__ double iface_rho(double zl, double zr, bool absm, double *dq = nullptr)
{
    const double sum = zl + zr, dif = zr - zl;
    const double is = rcp64(sum);
    const double q = dif * is;
    const double r = fma(fma(-sum, q, dif), is, q);
    if (dq) {
        const double sg = absm ? ((zr > zl) ? 1.0 : ((zr < zl) ? -1.0 : 0.0)) : 1.0;
        *dq = 2.0 * sg * is * is;
    }
    return absm ? fabs(r) : r;
}

// --------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11) and the unit-mean Rayleigh variate
// --------------------------------------------------------------------------
__device__ __forceinline__ void philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                       uint32_t k0, uint32_t k1, uint32_t out[4])
{
    // the round keys are formed here, ten scalar adds each beside the vector
    // work; hoisted out of the callers' loops they would hold (and spill)
    // twenty scalar registers
    asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // one 32 x 32 -> 64-bit product per multiplier (low and high words)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = hi1 ^ c1 ^ k0;
        const uint32_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// unit-mean Rayleigh: sqrt(-2 ln u) sqrt(2/pi) = sqrt(-(4 ln 2 / pi) log2 u);
// u in [2^-24, 1] is a normal number, so the hardware log2 and square root
// (about 1 ulp) apply directly
__device__ __forceinline__ float rayleigh(uint32_t x)
{
    const float u = fmaf((float)(x >> 8), 0x1p-24f, 0x1p-24f);      // (x >> 8) + 1 at most 2^24: exact
    return __builtin_amdgcn_sqrtf(-0.88254240061060638f * __builtin_amdgcn_logf(u));
}

// granular variates of samples 4 ctr .. 4 ctr + 3 of ray j
__device__ __forceinline__ void granular4(const PhysArgs &p, int ctr, int j, int sid, float x[4])
{
    uint32_t w[4];
    philox((uint32_t)ctr, (uint32_t)j, (uint32_t)sid, 0u, p.key0, p.key1, w);
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = rayleigh(w[q]);
}

// radial cell values covering the tile [t0, t0+T): s_xir[c - t0/cell]
template <int T>
__device__ __forceinline__ void speckle_radial(const PhysArgs &p, int t0, int j, int sid, int lane, float *s_xir)
{
    const int cell = p.cell;
    const int c_lo = t0 / cell, c_hi = (t0 + T - 1) / cell + 1;
    for (int b = (c_lo >> 2) + lane; b <= (c_hi >> 2); b += 64) {
        uint32_t w[4];
        philox((uint32_t)b, (uint32_t)j, (uint32_t)sid, 1u, p.key0, p.key1, w);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = 4 * b + q;
            if (c >= c_lo && c <= c_hi) s_xir[c - c_lo] = rayleigh(w[q]);
        }
    }
}

// Speckle inputs of one tile [t0, t0+T): granular variates per pixel and the
// radial cell values covering the tile.
template <int T>
__device__ __forceinline__ void speckle_fill(const PhysArgs &p, int t0, int j, int sid, int lane,
                                             float *s_xig, float *s_xir)
{
    for (int bb = lane; bb < T / 4; bb += 64) {
        float x[4];
        granular4(p, (t0 >> 2) + bb, j, sid, x);
        *reinterpret_cast<float4 *>(s_xig + 4 * bb) = make_float4(x[0], x[1], x[2], x[3]);
    }
    speckle_radial<T>(p, t0, j, sid, lane, s_xir);
}

// per-launch constants of pixel_gain: 1/(S-1) (1 for the one sample of S = 1,
// whose index is 0) and 1/cell
struct GainK {
    float inv_sm1, inv_cell;
};

__device__ __forceinline__ GainK gain_consts(const PhysArgs &p, int S)
{
    return GainK{S > 1 ? 1.0f / (float)(S - 1) : 1.0f, 1.0f / (float)p.cell};
}

// speckle multiplier of a pixel at depth fraction zeta, cell fraction fr
// between the radial cell values x0 and x1, granular variate xg.  zeta^gam
// with zeta in [1/(S-1), 1] (a normal number); a power below 2^-126 may
// flush to zero, which leaves the FP32 gain unchanged.
// POSITIVE: the caller knows zeta > 0.
template <bool POSITIVE = false>
__device__ __forceinline__ float speckle_mult(const PhysArgs &p, float zeta, float fr, float x0, float x1,
                                              float xg)
{
    const float xr = (1.0f - fr) * x0 + fr * x1;
    float pw;
    if (POSITIVE || zeta > 0.0f) pw = __builtin_amdgcn_exp2f(p.gam * __builtin_amdgcn_logf(zeta));
    else pw = (p.gam == 0.0f) ? 1.0f : 0.0f;
    return 1.0f + p.Ar * pw * (xr - 1.0f) + (p.Ag0 + p.Ag1 * zeta) * (xg - 1.0f);
}

// radial cell c = k div cell and remainder r of sample k (exact: the
// reciprocal's quotient is corrected by one step either way)
__device__ __forceinline__ void cell_of(const PhysArgs &p, const GainK &gk, int k, int &c, int &r)
{
    const int cell = p.cell;
    c = (int)((float)k * gk.inv_cell);
    r = k - c * cell;
    if (r < 0) { --c; r += cell; }
    if (r >= cell) { ++c; r -= cell; }
}

// Gain of pixel k: post-hoc attenuation (POST) times speckle (SPK), with xg
// the pixel's granular variate and s_xir the radial cell values of the tile
// starting at t0.  zeta = k/(S-1) and the cell fraction come from reciprocals
// (within an ulp of the quotients); the cell index is exact.
template <bool SPK, bool POST>
__device__ __forceinline__ float pixel_gain(const PhysArgs &p, const GainK &gk, int k, int t0, float postc,
                                            float xg, const float *s_xir)
{
    float g = 1.0f;
    if (POST) g = exp2f((float)((double)k * (double)postc));
    if (SPK) {
        int c, r;
        cell_of(p, gk, k, c, r);
        const int c_lo = t0 / p.cell;
        g *= speckle_mult(p, (float)k * gk.inv_sm1, (float)r * gk.inv_cell, s_xir[c - c_lo], s_xir[c + 1 - c_lo], xg);
    }
    return g;
}

// the same with the post-hoc switch read at run time
template <bool SPK>
__device__ __forceinline__ float pixel_gain_rt(const PhysArgs &p, const GainK &gk, int k, int t0, float postc,
                                               float xg, const float *s_xir)
{
    return (p.atten == 1) ? pixel_gain<SPK, true>(p, gk, k, t0, postc, xg, s_xir)
                          : pixel_gain<SPK, false>(p, gk, k, t0, postc, xg, s_xir);
}

__device__ __forceinline__ float posthoc_coef(const PhysArgs &p, float ds)
{
    // 10^(-2 alpha f (k ds / 10) / 20) = 2^(k * postc)
    return (float)(-(double)p.alpha * (double)p.freq * (double)ds / 100.0 * 3.321928094887362);
}

// --------------------------------------------------------------------------
// phase 1: gather the samples [t0, t0+T) of a ray into LDS, 64 consecutive
// samples per instruction: sample i of the tile at s_z[zi(i)], the sample
// before the tile at s_z[zi(-1)].  The lanes then read their chunks of
// consecutive samples back and form the interfaces' coefficients there: two
// neighbours sit in one lane, so nothing is exchanged between lanes, and the
// coefficients stay in registers.  Before a ray's first sample and past its
// last one the samples repeat, so the coefficient there is exactly zero
// without a select.  W (the caller's wavefronts per ray) only keeps the
// callers' instances apart: the compiler then derives each caller's index
// ranges from that caller alone.
// --------------------------------------------------------------------------
__device__ __forceinline__ int zi(int i) { return 2 + i + (i >> 4); }
template <int T> struct SampleTile { static constexpr int size = T + T / 16 + 2; };

template <int C, bool KEEPG, bool INSIDE, int W>
__device__ __forceinline__ double gather_tile_body(const VolArgs &v, const Ray &ray, int t0, int S, int lane,
                                                   double *s_z, float *s_g)
{
    constexpr int T = 64 * C;
    const int sxy = v.nx * v.ny;
    double z = 0.0;
#pragma unroll GATHER_UNROLL
    for (int jj = 0; jj < C; ++jj) {
        const int i = jj * 64 + lane;
        const int k = t0 + i;
        const Stencil st = stencil_at<INSIDE>(v, ray, min(k, S - 1));
        double gu[3];
        z = trilinear<INSIDE>(v.Z, v.nx, sxy, st, KEEPG ? gu : nullptr, ray.first);
        s_z[zi(i)] = z;
        if (k == 0) s_z[zi(-1)] = z;
        if (KEEPG) {
            // dZ/dp per mm (dZ/du / h, the spacing taken with the basis; zero
            // along an axis where the sample lies outside the volume:
            // clamped), kept in FP32 as its
            // components along the ray and across it (the ray's basis), so
            // that the rounding of the large component along the ray stays
            // along the ray, where it cannot reach the rotation gradient
            const double kk = (double)min(k, S - 1);
            const int n[3] = {v.nx, v.ny, v.nz};
            double gw[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double u = fma(kk, ray.du[a], ray.u0[a]);
                const bool inside = INSIDE || ((u >= 0.0) && (u <= (double)(n[a] - 1)));
                gw[a] = inside ? gu[a] : 0.0;
            }
            s_g[i] = (float)fma(gw[0], ray.bd[0], fma(gw[1], ray.bd[1], gw[2] * ray.bd[2]));
            s_g[T + i] = (float)fma(gw[0], ray.bt[0], fma(gw[1], ray.bt[1], gw[2] * ray.bt[2]));
            s_g[2 * T + i] = (float)fma(gw[0], ray.bn[0], fma(gw[1], ray.bn[1], gw[2] * ray.bn[2]));
        }
    }
    return z;      // lane 63: the tile's last sample
}

template <int C, bool KEEPG, int W>
__device__ __forceinline__ double gather_tile(const VolArgs &v, const Ray &ray, int t0, int S, int lane, double *s_z,
                                              float *s_g = nullptr)
{
    // a tile whose samples all lie inside the volume skips the clamps, and
    // takes 32-bit offsets where they reach (the ray is the same on every lane,
    // so the branch is uniform)
    if (ray.narrow && segment_inside(v, ray, t0, min(t0 + 64 * C - 1, S - 1)))
        return gather_tile_body<C, KEEPG, true, W>(v, ray, t0, S, lane, s_z, s_g);
    return gather_tile_body<C, KEEPG, false, W>(v, ray, t0, S, lane, s_z, s_g);
}

// Transfer map of interface rho (first column and determinant; the second
// column is (rho, 1)).  Interfaces outside [1, S) have rho = 0 and the map
// diag(a^2, 1), which leaves v1 alone and scales D by a^2: past the last
// sample that changes nothing stored, and the a^2 of the interface before
// sample 0 is taken out of the starting D (d_start).
struct Map {
    double m00, m10, det;
};

__device__ __forceinline__ Map make_map(double r, double a2, double sgn)
{
    Map m;
    const double r2 = r * r;
    m.m00 = a2 * (1.0 - r2 - sgn * r2);
    m.m10 = -a2 * sgn * r;
    m.det = a2 * (1.0 - r2);
    return m;
}

// D at the start of a ray: D = 1 after the first step
__device__ __forceinline__ double d_start(double a2) { return 1.0 / a2; }

struct Mat {
    double a, b, c, d;     // [[a, b], [c, d]]
};

__device__ __forceinline__ Mat matmul(const Mat &x, const Mat &y)
{
    Mat r;
    r.a = fma(x.a, y.a, x.b * y.c);
    r.b = fma(x.a, y.b, x.b * y.d);
    r.c = fma(x.c, y.a, x.d * y.c);
    r.d = fma(x.c, y.b, x.d * y.d);
    return r;
}

// the matrix d lanes up (DOWN: d lanes down)
template <bool DOWN>
__device__ __forceinline__ Mat shfl_mat(const Mat &m, int d)
{
    Mat r;
    r.a = DOWN ? __shfl_down(m.a, d) : __shfl_up(m.a, d);
    r.b = DOWN ? __shfl_down(m.b, d) : __shfl_up(m.b, d);
    r.c = DOWN ? __shfl_down(m.c, d) : __shfl_up(m.c, d);
    r.d = DOWN ? __shfl_down(m.d, d) : __shfl_up(m.d, d);
    return r;
}

// chunk product Q = M_first ... M_last of a lane's C interfaces, and det
template <int C>
__device__ __forceinline__ void chunk_product(const double (&rho)[C], double a2, double sgn, Mat &Q, double &qd)
{
    Q = Mat{1.0, 0.0, 0.0, 1.0};
    qd = 1.0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        const double r = rho[i];
        const Map m = make_map(r, a2, sgn);
        const double n00 = fma(Q.a, m.m00, Q.b * m.m10);
        const double n01 = fma(Q.a, r, Q.b);
        const double n10 = fma(Q.c, m.m00, Q.d * m.m10);
        const double n11 = fma(Q.c, r, Q.d);
        Q = Mat{n00, n01, n10, n11};
        qd *= m.det;
    }
}

// exclusive product scan over the 64 lanes in depth order; also returns the
// wave total.  The shallowest chunk is lane 0's, or lane 63's (DOWN).
template <bool DOWN>
__device__ __forceinline__ void scan_exclusive(int lane, Mat Q, double qd, Mat &X, double &xd,
                                               Mat &Tot, double &td)
{
    const int pos = DOWN ? 63 - lane : lane;
    constexpr int last = DOWN ? 0 : 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const Mat o = shfl_mat<DOWN>(Q, d);
        const double od = DOWN ? __shfl_down(qd, d) : __shfl_up(qd, d);
        if (pos >= d) {
            Q = matmul(o, Q);
            qd = od * qd;
        }
    }
    Tot = Mat{lane_read(Q.a, last), lane_read(Q.b, last), lane_read(Q.c, last), lane_read(Q.d, last)};
    td = lane_read(qd, last);
    X = shfl_mat<DOWN>(Q, 1);
    xd = DOWN ? __shfl_down(qd, 1) : __shfl_up(qd, 1);
    if (pos == 0) {
        X = Mat{1.0, 0.0, 0.0, 1.0};
        xd = 1.0;
    }
}

// scale the carried row vector by a power of two (exact; pixels are
// homogeneous of degree 0 in (v, sqrt(D)))
__device__ __forceinline__ int renorm_exp(double c0, double c1)
{
    const double m = fmax(fabs(c0), fabs(c1));
    if (!(m > 0.0) || !isfinite(m)) return 0;
    return ilogb(m);
}

// the carried state (c0, c1, cD) through a tile's total, renormalised
__device__ __forceinline__ void carry_through(const Mat &tot, double td, double &c0, double &c1, double &cD)
{
    const double n0 = fma(c0, tot.a, c1 * tot.c);
    const double n1 = fma(c0, tot.b, c1 * tot.d);
    const double nD = cD * td;
    const int ex = renorm_exp(n0, n1);
    c0 = ldexp(n0, -ex);
    c1 = ldexp(n1, -ex);
    cD = ldexp(nD, -2 * ex);
}

// Per-pixel gains (speckle, post-hoc attenuation) of the C consecutive
// samples that start at k0, a multiple of 4, so that the granular variates
// are C/4 whole Philox blocks; s_xir holds the radial cells of the tile
// starting at t0.
template <int C, bool SPK>
__device__ __forceinline__ void chunk_gains(const PhysArgs &p, const GainK &gk, int k0, int t0, int j, int sid,
                                            float postc, const float *s_xir, float (&gn)[C])
{
#pragma unroll
    for (int i = 0; i < C; ++i) gn[i] = 1.0f;
    if (SPK) {
#pragma unroll
        for (int q = 0; q < C / 4; ++q) {
            float x[4];
            granular4(p, (k0 >> 2) + q, j, sid, x);
#pragma unroll
            for (int u = 0; u < 4; ++u) gn[4 * q + u] = x[u];
        }
        // the lane's samples are consecutive: the radial cell index of the
        // first is exact (cell_of), the others step it, and the sample and
        // remainder step as floats (whole numbers: exact)
        int c, r0;
        cell_of(p, gk, k0, c, r0);
        const float *x = s_xir + (c - t0 / p.cell);
        const float kf = (float)k0, cellf = (float)p.cell;
        float r = (float)r0;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float zeta = (kf + (float)i) * gk.inv_sm1;
            gn[i] = (i == 0) ? speckle_mult(p, zeta, r * gk.inv_cell, x[0], x[1], gn[i])
                             : speckle_mult<true>(p, zeta, r * gk.inv_cell, x[0], x[1], gn[i]);
            r += 1.0f;
            const bool wrap = (r == cellf);
            x += wrap ? 1 : 0;
            r = wrap ? 0.0f : r;
        }
        if (p.atten == 1) {
#pragma unroll
            for (int i = 0; i < C; ++i) gn[i] *= exp2f((float)((double)(k0 + i) * (double)postc));
        }
    } else if (p.atten == 1) {
#pragma unroll
        for (int i = 0; i < C; ++i) gn[i] = pixel_gain<false, true>(p, gk, k0 + i, t0, postc, 1.0f, s_xir);
    }
}

// four floats, or two doubles, at any multiple of 4 bytes (global memory
// takes 16-byte accesses at dword alignment)
typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef double double2_u __attribute__((ext_vector_type(2), aligned(4)));

// --------------------------------------------------------------------------
// forward kernel
//
// W = 1: one wavefront per ray walks its tiles in order.  W > 1 (rays of
// many tiles): W wavefronts share a ray and take W consecutive tiles at a
// time.  A tile's gather, chunk products and lane scan need nothing from the
// tiles before it; only the state carried into its walk does, and that is
// the state at the round's start pushed through the scan totals of the
// tiles before it (one 1x2 by 2x2 product and a power-of-two renormalisation
// per tile, in the order and with the operations of W = 1, so the results
// are the same bit for bit).  The sample before the tile comes from its own
// trilinear lookup instead of the previous tile's gather.
//
// For the adjoint it records the state at every 4th sample as the two
// numbers that no renormalisation changes, w = v0 / v1 and t = D / v1^2
// (states: four floats' room each), and the sample before every 256th
// (zcar).  With zcar NULL the states of a ray sit in its own row of an image
// layout, that of sample 4 c at element 4 (c - 1), and the first one, a
// constant, is left out.  out may be NULL (states, and gains if wanted).
// --------------------------------------------------------------------------
template <int C, bool SPK, int W, bool PIV>
__global__ __launch_bounds__(64 * W) void k_forward(VolArgs v, PhysArgs p, FanTable tab,
                                                    const float *__restrict__ poses,
                                                    float *__restrict__ out, float *__restrict__ minpiv,
                                                    int pivot_base, double *__restrict__ zcar,
                                                    float *__restrict__ states,
                                                    float *__restrict__ gain_out, int xgrp, ZeroArgs zero)
{
    constexpr int T = 64 * C;
    static_assert(T % kCarryBlock == 0, "tiles hold whole carry blocks");
    static_assert(C % kStateStride == 0, "chunks hold whole state strides");
    constexpr int LB = kCarryBlock / C;     // lanes per carry block
    __shared__ double s_z_w[W][SampleTile<T>::size];
    __shared__ float s_xir_w[W][SPK ? T / 4 + 8 : 1];
    __shared__ double s_tot[W > 1 ? W : 1][5];     // scan totals of a round's tiles
    __shared__ double s_piv[W > 1 ? W : 1];

    const int lane = (W == 1) ? (int)threadIdx.x : (int)(threadIdx.x & 63);
    const int wv = (W == 1) ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double *s_z = s_z_w[wv];
    float *s_xir = s_xir_w[wv];
    if (zero.na > 0 || zero.nb > 0) {
        // the step's clears, spread over the forward's wavefronts: the stores
        // drain while the wavefront renders its ray
        const long long stride = (long long)gridDim.x * 64 * W;
        const long long i0 = (long long)blockIdx.x * 64 * W + threadIdx.x;
        if ((reinterpret_cast<uintptr_t>(zero.a) & 15) == 0) {
            float4 *a4 = reinterpret_cast<float4 *>(zero.a);
            const long long n4 = zero.na / 4;
            for (long long i = i0; i < n4; i += stride) a4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            for (long long i = 4 * n4 + i0; i < zero.na; i += stride) zero.a[i] = 0.0f;
        } else {
            for (long long i = i0; i < zero.na; i += stride) zero.a[i] = 0.0f;
        }
        for (long long i = i0; i < zero.nb; i += stride) zero.b[i] = 0.0;
    }
    const int g = remap_block(blockIdx.x, gridDim.x, xgrp);
    if (W == 1 && g < tab.ray0) return;          // walked by several wavefronts in another launch
    const int fi = find_fan(tab, g);
    const FanRec fr = tab.f[fi];
    const int j = g - fr.ray_begin;
    const int S = fr.n_samples;
    Ray ray;
    setup_ray(v, p, fr, poses, j, ray);
    if (tab.geom && threadIdx.x == 0) store_geom(ray, tab.geom + g);
    set_base(v, ray, S);
    const bool absm = (p.refl == 0);
    const double sgn = absm ? 1.0 : -1.0;
    const double a2 = ray.a2;
    const float postc = posthoc_coef(p, fr.ds);
    const GainK gk = gain_consts(p, fr.n_samples);
    const long long obase = fr.out_offset + (long long)j * S;

    // state carried into the round (W > 1) or the tile (W = 1)
    double c0 = 0.0, c1 = 1.0, cD = d_start(a2), zprev = 0.0;
    double piv = 1e300;
    const long long crec = (long long)fr.carry_begin + (long long)j * ((S + kCarryBlock - 1) / kCarryBlock);
    float *srow = nullptr;
    if (states) srow = states + (zcar ? crec * kStateFloats : obase - 4);

    for (int r0 = 0; r0 < S; r0 += W * T) {
        const int t0 = r0 + wv * T;
        const bool act = (W == 1) || (t0 < S);      // uniform over the wavefront
        if (W > 1 && act && t0 > 0) {
            const Stencil st = stencil_at<false>(v, ray, t0 - 1);
            zprev = trilinear(v.Z, v.nx, v.nx * v.ny, st, nullptr, ray.first);
        }
        if (act) {
            if (lane == 0 && t0 > 0) s_z[zi(-1)] = zprev;
            const double zl = gather_tile<C, false, W>(v, ray, t0, S, lane, s_z);
            if (W == 1) zprev = lane_read(zl, 63);
            if (SPK) speckle_radial<T>(p, t0, j, fr.speckle_id, lane, s_xir);
        }
        ray_sync<W>();

        const int base = lane * C;
        Mat Q, X, Tot;
        double qd, xd, td;
        double tc0 = c0, tc1 = c1, tcD = cD;        // the state carried into this tile
        double rho[C];
        if (act) {
            double zl = s_z[zi(base - 1)];
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const double zr = s_z[zi(base) + i];
                rho[i] = iface_rho(zl, zr, absm);
                zl = zr;
            }
            chunk_product<C>(rho, a2, sgn, Q, qd);
            scan_exclusive<false>(lane, Q, qd, X, xd, Tot, td);
        }
        if (W > 1) {
            if (act && lane == 0) {
                s_tot[wv][0] = Tot.a;
                s_tot[wv][1] = Tot.b;
                s_tot[wv][2] = Tot.c;
                s_tot[wv][3] = Tot.d;
                s_tot[wv][4] = td;
            }
            ray_sync<W>();
            // the round's carry through the tiles before this one; then on
            // through the rest of the round for the next round's carry
            for (int u = 0; u < W; ++u) {
                if (u == wv) {
                    tc0 = c0;
                    tc1 = c1;
                    tcD = cD;
                }
                if (r0 + u * T >= S) break;
                carry_through(Mat{s_tot[u][0], s_tot[u][1], s_tot[u][2], s_tot[u][3]}, s_tot[u][4], c0, c1, cD);
            }
        }
        if (act) {
            double v0 = fma(tc0, X.a, tc1 * X.c);
            double v1 = fma(tc0, X.b, tc1 * X.d);
            double D = tcD * xd;
            if (zcar) {
                // the sample before every carry block of the tile
                const int kb = t0 + base;
                if ((lane % LB) == 0 && kb < S) zcar[crec + kb / kCarryBlock] = s_z[zi(base - 1)];
            }
            float pix[C];
#pragma unroll
            for (int i = 0; i < C; ++i) {
                // branch-free: outside [1, S) rho = 0, so the pixel is 0 and v1
                // unchanged (make_map)
                const int k = t0 + base + i;
                // the states and the gains below are read once, by the adjoint
                // after the blur: non-temporal stores keep them from displacing
                // the volume and the images in the caches
                if ((i % kStateStride) == 0 && srow && k < S && (k > 0 || zcar)) {
                    const double iv = rcp64(v1);
                    const double2_u st = {quot64(v0, v1, iv), quot64(quot64(D, v1, iv), v1, iv)};
                    __builtin_nontemporal_store(st, reinterpret_cast<double2_u *>(srow + k));
                }
                const double r = rho[i];
                const Map m = make_map(r, a2, sgn);
                const double v1n = fma(v0, r, v1);
                // the pixel leaves in FP32: the hardware FP64 reciprocal, without
                // the Newton step, is accurate well beyond that
                pix[i] = (float)(r * D * __builtin_amdgcn_rcp(v1 * v1n));
                if (PIV) piv = (k >= 1 && k < S) ? fmin(piv, fabs(v1n * rcp64(v1))) : piv;
                const double v0n = fma(v0, m.m00, v1 * m.m10);
                v0 = v0n;
                v1 = v1n;
                D *= m.det;
            }
            // carry to the next tile, renormalised by a power of two
            if (W == 1) carry_through(Tot, td, c0, c1, cD);
            // per-pixel gains and the stores, in the lane's chunk order
            if (out || gain_out) {
                float gn[C];
                chunk_gains<C, SPK>(p, gk, t0 + base, t0, j, fr.speckle_id, postc, s_xir, gn);
                const bool has_gain = SPK || p.atten == 1;
                const long long o = obase + t0 + base;
                if (t0 + base + C <= S) {
#pragma unroll
                    for (int i = 0; i < C; i += 4) {
                        const float4_u px = {pix[i] * gn[i], pix[i + 1] * gn[i + 1], pix[i + 2] * gn[i + 2],
                                             pix[i + 3] * gn[i + 3]};
                        if (out) *reinterpret_cast<float4_u *>(out + o + i) = px;
                        if (has_gain && gain_out) {
                            const float4_u g4 = {gn[i], gn[i + 1], gn[i + 2], gn[i + 3]};
                            __builtin_nontemporal_store(g4, reinterpret_cast<float4_u *>(gain_out + o + i));
                        }
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < C; ++i) {
                        if (t0 + base + i < S) {
                            if (out) out[o + i] = pix[i] * gn[i];
                            if (has_gain && gain_out) gain_out[o + i] = gn[i];
                        }
                    }
                }
            }
        }
        ray_sync<W>();
    }
    if (PIV) {
        piv = wave_min(piv);
        if (W == 1) {
            if (lane == 0) minpiv[pivot_base + fr.pivot_begin + j] = (float)piv;
        } else {
            if (lane == 0) s_piv[wv] = piv;
            ray_sync<W>();
            if (threadIdx.x == 0) {
                for (int u = 1; u < W; ++u) piv = fmin(piv, s_piv[u]);
                minpiv[pivot_base + fr.pivot_begin + j] = (float)piv;
            }
        }
    }
}

// --------------------------------------------------------------------------
// adjoint kernel
// --------------------------------------------------------------------------
// The pixels depend on the state only through w = v0 / v1 and t = D / v1^2.
// With p = 1 + w R and q = 1 / p, interface by interface,
//   e = R t q,   w' = (A w + B) q,   t' = t E q^2,
// and dw'/dw = dt'/dt = E q^2 = t'/t.  Scaled by t the adjoint recurrence
// therefore has no factor left: with L = t dl/dt and O = t dl/dw (l the loss),
//   L_k = L_{k+1} + e_k dl/de_k,   O_k = O_{k+1} - e_k (L_k + L_{k+1}),
// two sums over the deeper interfaces, and
//   dl/dR_k = -O_{k+1} N / (t (1 - R^2)) - 2 L_{k+1} (R / (1 - R^2) + w q)
//             + dl/de_k t q^2,   N = w^2 - 1 + (1 + s) p^2.
// (A wavefront's 64 lanes so add two FP64 numbers each, with register moves
// between lanes, where the recurrence of (v0, v1, D) itself composes 2x2
// affine maps of eight numbers.)
//
// Lane l takes the chunk 63 - l of the tile's interfaces, so that the sums
// run over the lanes below.
//
// Bound by memory latency and VALU issue (0.66 busy at 3.1 wavefronts per SIMD,
// 128 VGPRs).  64 poses x 256 rays x 1024 samples with the forward's records,
// one launch: 239 us with the (v0, v1, D) adjoint, 151 us with the sums, 132
// us with the rays' geometry handed over, 32-bit gather offsets, loads ahead
// of the gather and no barrier that drains them, 134 us with the quotients
// taken to the last place.
//
// Where the state (w, t) at a chunk's start comes from (FROM):
//   kRecords: the records of the fused step's forward (states, zcar, geom).
//   kRows: states alone, in the rays' rows; the ray is set up again.
//     W = 1: one wavefront per ray walks its tiles from the deepest up.
//     W > 1 (rays of many tiles): W wavefronts share a ray and take W
//     consecutive tiles at a time.
//   kWholeRay (rays of at most W tiles): chunk products and a lane scan of
//     the wavefront's own tile, and the carries pushed through the tiles
//     before it, as k_forward does it with several wavefronts: the ray is
//     gathered once, and no forward pass comes before.
// Tile totals are added tile by tile in the same order for every W, so dL/dZ
// does not depend on W (bit for bit); the pose sums and the loss are added
// over the W wavefronts in a fixed order.
//
// zbar and states may name the same memory (with zcar NULL): a tile's states
// lie in its own part of the ray's row (the first in the part before it),
// and are read before the tile's dL/dZ overwrites it.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_zero(double x)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffll), CTRL, ROWS, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)((unsigned long long)b >> 32), CTRL, ROWS,
                                                              0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// x of the lane below (UP: above); the end lane takes `edge`
template <bool UP>
__device__ __forceinline__ double lane_next(double x, double edge)
{
    constexpr int ctrl = UP ? 0x130 : 0x138;     // wave_shl:1, wave_shr:1
    const long long b = __double_as_longlong(x), e = __double_as_longlong(edge);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(e & 0xffffffffll),
                                                              (int)(unsigned)(b & 0xffffffffll), ctrl, 0xf, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)((unsigned long long)e >> 32),
                                                              (int)(unsigned)((unsigned long long)b >> 32), ctrl, 0xf,
                                                              0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// sum over this lane and those below it (row_shr 1, 2, 4, 8 within the rows
// of 16 lanes, then the rows' last lanes handed on by row_bcast)
__device__ __forceinline__ double lanes_below(double x)
{
    x += dpp_zero<0x111>(x);
    x += dpp_zero<0x112>(x);
    x += dpp_zero<0x114>(x);
    x += dpp_zero<0x118>(x);
    x += dpp_zero<0x142, 0xa>(x);
    x += dpp_zero<0x143, 0xc>(x);
    return x;
}

__device__ __forceinline__ double lanes_sum(double x) { return lane_read(lanes_below(x), 63); }

// a lane's C consecutive values from sample k0 on; `fill` past sample S
template <int C>
__device__ __forceinline__ void load_chunk(const float *__restrict__ row, int k0, int S, float fill, float (&x)[C])
{
    if (k0 + C <= S) {
#pragma unroll
        for (int i = 0; i < C; i += 4) {
            const float4_u q = *reinterpret_cast<const float4_u *>(row + k0 + i);
            x[i] = q.x;
            x[i + 1] = q.y;
            x[i + 2] = q.z;
            x[i + 3] = q.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < C; ++i) x[i] = (k0 + i < S) ? row[k0 + i] : fill;
    }
}

enum { kRecords = 0, kRows = 1, kWholeRay = 2 };

// NEAR: the volume lies within 4 GiB (in_reach), known at the launch: the
// recorded one-wavefront instances are short of scalar registers for a base of
// their own (pose-only step of 32 x 384 x 1536: 309 us, 317 with it).
template <int C, bool SPK, bool FUSED, int W, int FROM, bool NEAR = false>
__global__ __launch_bounds__(64 * adjoint_waves(W), (C == 4 && W == 1 && FROM == kRecords && !FUSED && NEAR) ? 4 : 1)
void k_backward(VolArgs v, PhysArgs p, FanTable tab,
                                                 const float *__restrict__ poses,
                                                 RayRec *__restrict__ rays_out,
                                                 const float *__restrict__ gsrc,
                                                 const float *__restrict__ target,
                                                 float *zbar,
                                                 double *__restrict__ pose_part,
                                                 double *__restrict__ loss_acc,
                                                 const double *__restrict__ zcar,
                                                 const float *states,
                                                 const RayGeom *__restrict__ geom,
                                                 const float *__restrict__ gain_in, int xgrp)
{
    constexpr int T = 64 * C;
    constexpr int NW = adjoint_waves(W);
    constexpr bool WHOLE = FROM == kWholeRay;
    static_assert(C % kStateStride == 0, "a chunk starts on a recorded state");
    __shared__ __align__(16) float s_g_w[NW][3 * T];     // dZ/dp of every sample of the tile, in the ray's basis
    __shared__ double s_z_w[NW][SampleTile<T>::size];
    __shared__ float s_xir_w[NW][SPK ? T / 4 + 8 : 1];
    __shared__ double s_tot[WHOLE ? W : 1][5];    // the tiles' scan totals
    __shared__ double s_l[W], s_o[W], s_q[W];     // a round's tiles: sums of L and O, first interface's dL/dZ factor
    __shared__ double s_red[W][7];                // per-wavefront pose sums and loss

    const int lane = (int)(threadIdx.x & 63);
    const int slot = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));     // wavefront of the block
    const int wv = (W == 1) ? 0 : slot;                                             // wavefront of the ray
    float *s_g = s_g_w[slot];
    double *s_z = s_z_w[slot];
    float *s_xir = s_xir_w[slot];
    int g = remap_block(blockIdx.x, gridDim.x, xgrp);
    if (W == 1) {
        g = g * kBlockRays + slot;
        if (WHOLE) g += tab.ray0;
        // (below ray0: walked by several wavefronts in another launch)
        if (g < tab.ray0 || g >= (WHOLE ? tab.ray1 : tab.total_rays)) return;
    } else if (WHOLE) {
        g += tab.ray0;
    }
    const int fi = find_fan(tab, g);
    const FanRec fr = tab.f[fi];
    const int j = g - fr.ray_begin;
    const int S = fr.n_samples;
    if (S <= 0) return;
    Ray ray;
    if (FROM == kRecords) load_geom(fr, geom + g, ray);
    else setup_ray(v, p, fr, poses, j, ray);
    if (NEAR) {
        ray.first = 0;
        ray.narrow = in_reach(v);       // (a constant here costs six spilled registers: 138 -> 151 us)
    } else {
        set_base(v, ray, S);
    }
    if (rays_out && lane == 0 && wv == 0) {
        // the ray's geometry for the scatter
        RayRec r;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            r.u0[a] = ray.u0[a];
            r.du[a] = ray.du[a];
        }
        rays_out[g] = r;
    }
    const bool absm = (p.refl == 0);
    const double sgn = absm ? 1.0 : -1.0, onep = 1.0 + sgn;
    const double a2 = ray.a2;
    const float postc = posthoc_coef(p, fr.ds);
    const GainK gk = gain_consts(p, fr.n_samples);
    const long long obase = fr.out_offset + (long long)j * S;
    const int ntiles = (S + T - 1) / T;
    const double inv_npix = 1.0 / ((double)fr.n_rays * (double)S);
    const long long crec = (long long)fr.carry_begin + (long long)j * ((S + kCarryBlock - 1) / kCarryBlock);
    const float *srow = WHOLE ? nullptr : states + (FROM == kRecords ? crec * kStateFloats : obase - 4);
    const float *src = (FUSED ? target : gsrc) + obase;

    // the sums L and O over everything deeper than the (round's deepest)
    // tile, and the interface factor and sample just past it
    double l_in = 0.0, o_in = 0.0, qz_in = 0.0, z_in = 0.0;
    double loss = 0.0;
    double gsum[3] = {0.0, 0.0, 0.0}, gssum[3] = {0.0, 0.0, 0.0};
    // wavefront w takes tile rt - w of a round
    for (int rt = ntiles - 1; rt >= 0; rt -= W) {
        // uniform over the wavefront; an idle wavefront of the last round
        // repeats tile 0 and stores nothing
        const bool act = (W == 1) || (rt - wv >= 0);
        const int t = act ? rt - wv : 0;
        const int t0 = t * T;
        const int base = (63 - lane) * C;
        const int k0 = t0 + base;
        // wave priority 1 while this wavefront issues its loads and its gather
        // (they go out ahead of co-resident wavefronts' FP64 arithmetic) and
        // during the lane sums, 0 elsewhere
        __builtin_amdgcn_s_setprio(1);
        double w = 0.0, tt = d_start(a2);        // state before the ray's first interface
        double zm = 0.0;                          // the sample before the tile
        if (!WHOLE) {
            const int ks = min(k0, S - 1) & ~(kStateStride - 1);
            if (ks > 0) {
                const double2_u st = *reinterpret_cast<const double2_u *>(srow + ks);
                w = st.x;
                tt = st.y;
            }
            if (t0 > 0) {
                if (FROM == kRecords) {
                    zm = zcar[crec + t0 / kCarryBlock];
                } else {
                    const Stencil st = stencil_at<false>(v, ray, t0 - 1);
                    zm = trilinear(v.Z, v.nx, v.nx * v.ny, st, nullptr, ray.first);
                }
            }
        }
        // dL/de (or the target for the fused loss) and the recorded gains: on
        // their way before the gather
        float ebf[C], gn[C];
        load_chunk<C>(src, k0, S, 0.0f, ebf);
        if (FROM == kRecords) {
            if (gain_in) {
                load_chunk<C>(gain_in + obase, k0, S, 1.0f, gn);
            } else {                              // the forward records them whenever there are any
#pragma unroll
                for (int i = 0; i < C; ++i) gn[i] = 1.0f;
            }
        }
        // (the basis is needed here alone: loaded again per tile, it holds no
        // scalar registers through the walks)
        if (FROM == kRecords && pose_part) load_basis(geom + g, ray);
        if (pose_part) gather_tile<C, true, W>(v, ray, t0, S, lane, s_z, s_g);
        else gather_tile<C, false, W>(v, ray, t0, S, lane, s_z);
        if (SPK) speckle_radial<T>(p, t0, j, fr.speckle_id, lane, s_xir);
        __builtin_amdgcn_s_setprio(0);
        ray_sync<W>();

        if (FROM != kRecords) {
            chunk_gains<C, SPK>(p, gk, k0, t0, j, fr.speckle_id, postc, s_xir, gn);
            // past the ray's end the depth fraction exceeds 1 and its power may
            // overflow: no gain there (0 times infinity would reach the sums)
            if (k0 + C > S) {
#pragma unroll
                for (int i = 0; i < C; ++i) gn[i] = (k0 + i < S) ? gn[i] : 1.0f;
            }
        }

        // the chunk's samples, those on either side of it, and its interfaces
        double z[C], rho[C], dq[C];
#pragma unroll
        for (int i = 0; i < C; ++i) z[i] = s_z[zi(base) + i];
        if (W > 1 && WHOLE && t > 0) zm = s_z_w[wv + 1][zi(T - 1)];
        const double zp = (W > 1 && wv > 0) ? s_z_w[wv - 1][zi(0)] : z_in;
        const double zl = lane_next<true>(z[C - 1], (t > 0) ? zm : z[0]);
        const double zr = lane_next<false>(z[0], zp);
#pragma unroll
        for (int i = 0; i < C; ++i) rho[i] = iface_rho(i > 0 ? z[i - 1] : zl, z[i], absm, &dq[i]);
        if (k0 == 0) dq[0] = 0.0;                 // no interface before sample 0

        if (WHOLE) {
            Mat Q, X, Tot;
            double qd, xd, td;
            chunk_product<C>(rho, a2, sgn, Q, qd);
            scan_exclusive<true>(lane, Q, qd, X, xd, Tot, td);
            double c0 = 0.0, c1 = 1.0, cD = d_start(a2);
            if (W > 1) {
                if (act && lane == 0) {
                    s_tot[wv][0] = Tot.a;
                    s_tot[wv][1] = Tot.b;
                    s_tot[wv][2] = Tot.c;
                    s_tot[wv][3] = Tot.d;
                    s_tot[wv][4] = td;
                }
                ray_sync<W>();
                for (int u = rt; u > wv && u < W; --u)      // tiles 0 .. t - 1, at wavefronts rt .. wv + 1
                    carry_through(Mat{s_tot[u][0], s_tot[u][1], s_tot[u][2], s_tot[u][3]}, s_tot[u][4], c0, c1, cD);
            }
            const double v0 = fma(c0, X.a, c1 * X.c), v1 = fma(c0, X.b, c1 * X.d);
            const double iv = rcp64(v1);
            w = quot64(v0, v1, iv);
            tt = quot64(quot64(cD * xd, v1, iv), v1, iv);
        }

        // walk down the chunk: every interface's pixel e and be = e dl/de, and
        // its dL/dZ factor qz (dl/dR times d rho / dZ's common factor) as
        // cz - cl L - co O of the sums below it, so that the states themselves
        // end here
        double e[C], be[C], co[C], cl[C], qz[C];
        double lsum = 0.0;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const double r = rho[i];
            const double pp = fma(w, r, 1.0);
            double q = rcp64(pp);
            q = fma(fma(-pp, q, 1.0), q, q);      // (carried on in w: to the last place)
            const double r2 = r * r, om = 1.0 - r2;
            const double x = tt * q;
            e[i] = r * x;
            double eb;
            if (FUSED) {
                const double diff = fma(e[i], (double)gn[i], -(double)ebf[i]);
                loss += act ? diff * diff * inv_npix : 0.0;
                eb = 2.0 * diff * inv_npix * (double)gn[i];
            } else {
                eb = (double)(ebf[i] * gn[i]);
            }
            be[i] = eb * e[i];
            lsum += be[i];
            const double tom = tt * om;
            // for |t| below 1e-150 O (about t^2 dl/de) over t is far under FP32's
            // smallest number, and near t's own underflow it is 0 / 0.  (t is
            // negative past an interface with |R| > 1, which impedances of
            // both signs give.)
            const double inv = (fabs(tt) < 1e-150) ? 0.0 : rcp64(tom);
            const double N = fma(onep * pp, pp, fma(w, w, -1.0));
            co[i] = dq[i] * inv * N;
            cl[i] = 2.0 * dq[i] * fma(r * tt, inv, w * q);
            qz[i] = dq[i] * (eb * x * q);
            w = fma(w, a2 * (om - sgn * r2), -a2 * sgn * r) * q;
            tt = a2 * tom * q * q;
        }
        __builtin_amdgcn_s_setprio(1);
        // L at the chunk's end: the tiles and the chunks below
        double l_end, lb = lanes_below(lsum);
        {
            const double tot = lane_read(lb, 63);
            double l_tile = l_in;
            if (W == 1) {
                l_in += tot;
            } else {
                if (lane == 0) s_l[wv] = tot;
                ray_sync<W>();
                for (int u = 0; u < W; ++u) {
                    if (u == wv) l_tile = l_in;
                    if (rt - u < 0) break;
                    l_in += s_l[u];
                }
            }
            l_end = l_tile + lane_next<false>(lb, 0.0);
        }
        // then O, from the true L
        double o_end, osum = 0.0;
        {
            double l = l_end;
#pragma unroll
            for (int i = C - 1; i >= 0; --i) {
                const double up = l + be[i];
                osum = fma(e[i], l + up, osum);
                l = up;
            }
            const double ob = lanes_below(osum);
            const double tot = lane_read(ob, 63);
            double o_tile = o_in;
            if (W == 1) {
                o_in -= tot;
            } else {
                if (lane == 0) s_o[wv] = tot;
                ray_sync<W>();
                for (int u = 0; u < W; ++u) {
                    if (u == wv) o_tile = o_in;
                    if (rt - u < 0) break;
                    o_in -= s_o[u];
                }
            }
            o_end = o_tile - lane_next<false>(ob, 0.0);
        }
        __builtin_amdgcn_s_setprio(0);

        // walk up: the interfaces' dL/dZ factors
#pragma unroll
        for (int i = C - 1; i >= 0; --i) {
            qz[i] = fma(-co[i], o_end, fma(-cl[i], l_end, qz[i]));
            const double up = l_end + be[i];
            o_end = fma(-e[i], l_end + up, o_end);
            l_end = up;
        }
        // dL/dZ_k per sample (rho depends on the samples on both sides: dL/dzr
        // = rb dq zl, dL/dzl = -rb dq zr): sample k is the right end of
        // interface k and the left end of interface k + 1, whose factor is the
        // lane below's, or the deeper tile's
        double qn = qz_in;
        if (W > 1) {
            if (lane == 63) s_q[wv] = qz[0];
            ray_sync<W>();
            if (wv > 0) qn = s_q[wv - 1];
        }
        qn = lane_next<false>(qz[0], qn);
        // (the samples are read again, rather than held through the sums)
        int zat = zi(base);
        asm volatile("" : "+v"(zat));
#pragma unroll
        for (int i = 0; i < C; ++i) z[i] = s_z[zat + i];
        double zb[C];
#pragma unroll
        for (int i = 0; i < C; ++i)
            zb[i] = fma(-(i + 1 < C ? qz[i + 1] : qn), i + 1 < C ? z[i + 1] : zr, qz[i] * (i > 0 ? z[i - 1] : zl));
        // zbar is NULL when no volume gradient is wanted (nothing reads it)
        if (zbar && act) {
            float *zrow = zbar + obase + k0;
            if (k0 + C <= S) {
#pragma unroll
                for (int i = 0; i < C; i += 4) {
                    const float4_u q = {(float)zb[i], (float)zb[i + 1], (float)zb[i + 2], (float)zb[i + 3]};
                    *reinterpret_cast<float4_u *>(zrow + i) = q;
                }
            } else {
#pragma unroll
                for (int i = 0; i < C; ++i)
                    if (k0 + i < S) zrow[i] = (float)zb[i];
            }
        }
        if (pose_part && act) {
            // dL/dp = zb dZ/dp; dL/dR accumulates (s_k dir) outer dL/dp
            const double s0 = fma((double)k0, ray.ds, ray.r0);
            double sz[C];
#pragma unroll
            for (int i = 0; i < C; ++i) sz[i] = fma((double)i, ray.ds, s0) * zb[i];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
                for (int i = 0; i < C; i += 4) {
                    const float4 q = *reinterpret_cast<const float4 *>(s_g + a * T + base + i);
                    gsum[a] = fma(zb[i], (double)q.x, gsum[a]);
                    gsum[a] = fma(zb[i + 1], (double)q.y, gsum[a]);
                    gsum[a] = fma(zb[i + 2], (double)q.z, gsum[a]);
                    gsum[a] = fma(zb[i + 3], (double)q.w, gsum[a]);
                    gssum[a] = fma(sz[i], (double)q.x, gssum[a]);
                    gssum[a] = fma(sz[i + 1], (double)q.y, gssum[a]);
                    gssum[a] = fma(sz[i + 2], (double)q.z, gssum[a]);
                    gssum[a] = fma(sz[i + 3], (double)q.w, gssum[a]);
                }
            }
        }
        // for the next tile up, or the next round's deepest: this (round's
        // shallowest) tile's first interface and sample
        if (W == 1) {
            qz_in = lane_read(qz[0], 63);
            z_in = lane_read(z[0], 63);
        } else {
            qz_in = s_q[W - 1];
            z_in = s_z_w[W - 1][zi(0)];
        }
        ray_sync<W>();
    }
    double r[6];
    if (pose_part) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            r[a] = lanes_sum(gsum[a]);
            r[3 + a] = lanes_sum(gssum[a]);
        }
    }
    double ls = 0.0;
    if (FUSED && loss_acc) ls = lanes_sum(loss);
    if (W > 1) {
        // the wavefronts' shares added in a fixed order
        if (lane == 0) {
#pragma unroll
            for (int a = 0; a < 6; ++a) s_red[wv][a] = pose_part ? r[a] : 0.0;
            s_red[wv][6] = ls;
        }
        ray_sync<W>();
        if (wv == 0) {
            for (int u = 1; u < W; ++u) {
#pragma unroll
                for (int a = 0; a < 6; ++a) r[a] += s_red[u][a];
                ls += s_red[u][6];
            }
        }
    }
    if (pose_part) {
        if (FROM == kRecords) load_basis(geom + g, ray);
        if (lane == 0 && wv == 0) {
            // this ray's share of dL/dt = sum g and dL/dR = sum g (s dir)^T,
            // dir = (sx, 0, cz), with g back from the ray's basis to the world
            // frame; k_pose_reduce sums the rays of each pose (in a fixed
            // order: no contended atomics on the pose's entries)
            double *pr = pose_part + (size_t)kRayPart * g;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double h = v.h[a];      // out of the basis again
                const double gt = h * fma(r[0], ray.bd[a], fma(r[1], ray.bt[a], r[2] * ray.bn[a]));
                const double gs = h * fma(r[3], ray.bd[a], fma(r[4], ray.bt[a], r[5] * ray.bn[a]));
                pr[a] = gt;
                pr[3 + 2 * a] = gs * ray.dirx;
                pr[4 + 2 * a] = gs * ray.dirz;
            }
        }
    }
    if (FUSED && loss_acc) {
        // one partial per ray, summed by k_sum_f64 (no contended atomics)
        if (lane == 0 && wv == 0) loss_acc[g] = ls;
    }
}

// --------------------------------------------------------------------------
// scatter of dL/dZ_k: trilinear weights into the volume gradient.  One
// wavefront takes RB neighbouring rays of one fan (64/RB lanes per ray) and
// one segment of `seg` depths, and walks them together in groups of
// (64/RB) spl depths; every lane owns spl (4, 2 or 1) consecutive depths of
// its ray.
// A straight ray meets each cell once, so a
// lane's consecutive samples in one cell form a run that it sums in
// registers before touching memory.  The stencils of a group fill a small
// box of the volume (neighbouring rays of a fan overlap); the runs go into an
// LDS copy of that box with LDS atomics, and the box is then flushed with one
// global atomic per touched voxel, consecutive lanes on consecutive x.  A
// group whose box does not fit takes its rays in halves (quarters, ...), or
// at coarse steps its depths, and what still does not fit goes to per-sample
// global atomics.
//
// The box holds FP64: FP64 LDS atomics (ds_add_f64) run at the rate of
// plain LDS stores on gfx950, FP32 LDS atomics several times slower.  The
// FP64 sum of a voxel's FP32 contributions is rounded to FP32 once, when the
// box is flushed.
// --------------------------------------------------------------------------
//
// Bound by LDS instructions: every 64-bit LDS store or atomic of a wavefront
// takes about 8 clocks of its CU however many lanes are active (measured), and
// a group of 256 samples issues about 32 to accumulate and 16 to flush; and by
// the global atomics where many rays meet (40 of 131 us with eight rays to a
// box).  64 poses x 256 rays x 1024 samples 139 -> 134 us with half the vector
// instructions (no clamps inside the volume, box by register reductions, a
// flush that steps along one axis), 63 fans of 256 x 256 and one of 64 x 16384
// 218 -> 101 us with boxes for parts of the rays; 134 -> 129 and 101 -> 94 us
// with sixteen rays to a box.
constexpr int kScatterSpl = 4;     // consecutive depths per lane, at most

// floor(a / b) for a >= 0, b >= 1, a + b < 2^21, from rb = rcp(b) (within
// 1 ulp): (a + 0.5) / b lies at least 0.5 / b from an integer, more than the
// product's error (a / b + 1) 2^-22.  A few instructions, where an integer
// division takes about thirty.
__device__ __forceinline__ int small_quot(int a, float rb)
{
    return (int)(((float)a + 0.5f) * rb);
}

template <int RB>
struct ScatterBox {
    static constexpr int cap = RB == 2 ? 4096 : (RB == 4 ? 2048 : 1024);   // FP64 entries
};

// smallest value over the wavefront (every lane active), in a scalar register
__device__ __forceinline__ int wave_min_int(int x)
{
    x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x111, 0xf, 0xf, false));
    x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x112, 0xf, 0xf, false));
    x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x114, 0xf, 0xf, false));
    x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x118, 0xf, 0xf, false));
    x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x142, 0xa, 0xf, false));
    x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(x, 63);
}

template <int RB>
__global__ __launch_bounds__(64) void k_scatter(VolArgs v, FanTable tab, const RayRec *__restrict__ rays,
                                                const float *__restrict__ zbar, float *__restrict__ gZ,
                                                int seg_shift, int few, int xgrp,
                                                unsigned long long *__restrict__ fix,
                                                const double *__restrict__ fscale)
{
    constexpr int LPR = 64 / RB;                 // lanes per ray
    constexpr int CAP = ScatterBox<RB>::cap - 1;
    // s_box is all zeros between groups: cleared once here, and every flush
    // clears the entries it reads; the last entry, outside the box, stays zero
    __shared__ double s_box[CAP + 1];
    const int lane = threadIdx.x;
    const int slot = lane / LPR, ll = lane % LPR;
    // depth chunk of this lane, rotated by the ray slot: in one instruction
    // the rays of the wavefront sit at different depths (>= 1 mm apart), so
    // lanes of one LDS atomic rarely meet in one cell
    const int ch = (ll + slot * LPR / RB) % LPR;
    // block -> (fan, depth segment, first ray).  Each fan owns ceil(n_rays /
    // RB) ray blocks.  One-dimensional grid: the fans one after the other,
    // each with its ceil(n_samples / seg) segments of ray blocks (ray blocks
    // fastest: neighbouring wavefronts share voxels).  Two-dimensional grid:
    // the ray blocks of all fans along x, the segment along y (a fan's
    // blocks past its depth exit at once).  The launcher records each fan's
    // first block in unit_begin.
    const int b = remap_block(blockIdx.x, gridDim.x, xgrp);
    const bool two_d = gridDim.y > 1;
    const int seg = 1 << seg_shift;              // a power of two: no division per fan
    int fi = 0;
    {
        // the fan whose wavefronts hold b: binary search over the fans' first units
        int hi = tab.n - 1;
        while (fi < hi) {
            const int mid = (fi + hi + 1) >> 1;
            if (tab.f[mid].unit_begin <= b) fi = mid; else hi = mid - 1;
        }
    }
    const FanRec fr = tab.f[fi];
    const int acc = fr.unit_begin, nrb = (fr.n_rays + RB - 1) / RB;
    const int sgi = two_d ? (int)blockIdx.y : (b - acc) / nrb;
    const int j = (b - acc - (two_d ? 0 : sgi * nrb)) * RB + slot;
    const bool ray_ok = j < fr.n_rays;
    const int jr = min(j, fr.n_rays - 1);        // lanes past the fan repeat its last ray, with zeros
    const int S = fr.n_samples;
    const int k_begin = sgi * seg;
    if (k_begin >= S) return;                   // whole wavefront: past this fan's depth
    const int k_end = min(S, k_begin + seg);
    // RB rays per wavefront, their geometry as the adjoint set it up
    Ray ray;
    {
        const RayRec &r = rays[fr.ray_begin + jr];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            ray.u0[a] = r.u0[a];
            ray.du[a] = r.du[a];
        }
    }
    const float *zrow = zbar + fr.out_offset + (long long)jr * S;
    const int sxy = v.nx * v.ny;
    // depths per lane (4, 2 or 1) from the step length in voxels, so that a
    // group spans about 11 voxels along the rays and its box fits LDS also
    // for coarse steps (one sample per voxel and more); the wavefront's
    // first ray decides (the rays of a fan share their step length)
    int spl;
    bool coarse;
    {
        const double s2 = ray.du[0] * ray.du[0] + ray.du[1] * ray.du[1] + ray.du[2] * ray.du[2];
        spl = (s2 <= 0.35 * 0.35) ? 4 : ((s2 <= 0.7 * 0.7) ? 2 : 1);
        spl = __builtin_amdgcn_readfirstlane(spl);
        coarse = __builtin_amdgcn_readfirstlane((int)(s2 > 1.2 * 1.2)) != 0;
    }
    const int G = LPR * spl;                     // depths per group (divides LPR kScatterSpl)
    // deterministic mode: 64-bit fixed-point sums (integer adds, in any
    // order the same) with the step's scale instead of FP32 atomics
    const double fsc = fix ? fscale[0] : 0.0;
    for (int t = lane; t <= CAP; t += 64) s_box[t] = 0.0;
    // dL/dZ of the lane's depths from k on, zero past the segment and for
    // lanes past the fan (the depths past spl stay zero)
    auto load = [&](int k, float (&x)[kScatterSpl]) {
        if (spl == kScatterSpl && k + kScatterSpl <= S) {
            const float4_u q = *reinterpret_cast<const float4_u *>(zrow + k);
            x[0] = q.x;
            x[1] = q.y;
            x[2] = q.z;
            x[3] = q.w;
        } else {
#pragma unroll
            for (int q = 0; q < kScatterSpl; ++q) x[q] = (q < spl) ? zrow[min(k + q, S - 1)] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < kScatterSpl; ++q) x[q] = (ray_ok && q < spl && k + q < k_end) ? x[q] : 0.0f;
    };
    // loaded one group ahead
    float zn[kScatterSpl];
    load(k_begin + ch * spl, zn);
    for (int k0 = k_begin; k0 < k_end; k0 += G) {
        const int kl = k0 + ch * spl;            // the lane's first depth
        float zb[kScatterSpl];
#pragma unroll
        for (int q = 0; q < kScatterSpl; ++q) zb[q] = zn[q];
        // the segment's last group loads nothing ahead (the next segment
        // belongs to another wavefront)
        if (k0 + G < k_end) load(kl + G, zn);
        const bool some = zb[0] != 0.0f || zb[1] != 0.0f || zb[2] != 0.0f || zb[3] != 0.0f;
        if (__ballot(some) == 0ull) continue;    // nothing to scatter in this group (uniform)
        // Cells and weights of the lane's depths, from their FP64 positions;
        // without the clamps where every lane's first and last depth, and so
        // (the position is affine) all between, lie inside the volume.  Lanes
        // past the segment repeat its last depth.
        int ci[kScatterSpl][3];
        float wf[kScatterSpl][3];
        const int kf = min(kl, k_end - 1), kb = min(kl + spl - 1, k_end - 1);
        const bool inside = __ballot(!segment_inside(v, ray, kf, kb)) == 0ull;
#pragma unroll
        for (int q = 0; q < kScatterSpl; ++q) {
            const int k = min(kf + q, kb);
            const Stencil st = inside ? stencil_at<true>(v, ray, k) : stencil_at<false>(v, ray, k);
            ci[q][0] = st.ix;
            ci[q][1] = st.iy;
            ci[q][2] = st.iz;
            wf[q][0] = (float)st.fx;
            wf[q][1] = (float)st.fy;
            wf[q][2] = (float)st.fz;
        }
        // A box for all the lanes at once, or for halves, quarters, ... of the
        // rays where that box would not fit (rays of a coarse fan lie far
        // apart).  At steps over 1.2 voxels for halves and quarters of the
        // depths: the group is long, and near the probe its rays share cells
        // that are worth a box; past that its samples share too few for one.
        // (Not where samples lie outside the volume: those are many to a voxel
        // at its faces, and are summed in FP64 ray by ray.)
        // In small launches (few) rays at steps of 0.35 and 0.7 voxels and more
        // down to two and four at a time: boxes for single rays' 16 or 8 depths,
        // one after the other, take longer than their atomics (9 voxels apart: 1
        // pose x 8 x 103 55 / 26 us); where many wavefronts' atomics meet near the
        // probes they don't (64 poses x 85 x 267 120 / 179).
        // (full step's scatter by rays / by depths, us: 12 poses x 40 x 147 at
        // 1.2 voxels 41 / 28, 18 x 257 x 95 at 1.8 34 / 25, 12 x 287 x 73 at 2.3
        // 74 / 25; 25 x 82 x 178 at 1.16 37 / 41).
        const bool deep = coarse && inside;
        const int key = deep ? ch : slot, all = deep ? LPR : RB;
        const int least = deep ? min(4, LPR) : (few && inside ? 4 / spl : 1);
        int part = all;
        for (int s0 = 0; s0 < all;) {
            // (lanes with zeros alone take no part: those past a fan of few rays
            // lie on its last ray, and their atomics would queue behind its own)
            const bool mine = some && (unsigned)(key - s0) < (unsigned)part;
            if (__ballot(mine) == 0ull) {
                s0 += part;
                continue;
            }
            // (opaque, or the weights' products would be held across the loop)
#pragma unroll
            for (int q = 0; q < kScatterSpl; ++q)
                asm volatile("" : "+v"(zb[q]), "+v"(wf[q][0]), "+v"(wf[q][1]), "+v"(wf[q][2]));
            // bounding box of the rays' cells: monotone along a straight ray, so
            // the lane's first and last depth hold its extremes
            int lo[3], hi[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int c0 = ci[0][a], c1 = ci[kScatterSpl - 1][a];
                lo[a] = wave_min_int(mine ? min(c0, c1) : 0x7fffffff);
                hi[a] = -wave_min_int(mine ? -max(c0, c1) : 0x7fffffff);
            }
            const int ox = lo[0], oy = lo[1], oz = lo[2];
            const int bx = hi[0] - ox + 2, by = hi[1] - oy + 2, bz = hi[2] - oz + 2;
            // odd row and plane strides: neighbouring cells along any axis land
            // in different LDS banks
            const int rs = bx | 1;
            const int ps = (rs * by) | 1;
            const bool fits = bx <= 64 && by <= CAP && (long long)ps * bz <= CAP;
            if (!fits && part > least) {
                part >>= 1;
                continue;
            }
            s0 += part;
            if (!fits) {
#pragma unroll
                for (int q = 0; q < kScatterSpl; ++q) {
                    if (!mine || zb[q] == 0.0f) continue;
                    const long long at = (long long)ci[q][2] * sxy + (long long)ci[q][1] * v.nx + ci[q][0];
#pragma unroll 1
                    for (int c = 0; c < 8; ++c) {       // (rare: kept small in registers)
                        const float x = (c & 1) ? wf[q][0] : 1.0f - wf[q][0];
                        const float y = (c & 2) ? wf[q][1] : 1.0f - wf[q][1];
                        const float w = zb[q] * x * y * ((c & 4) ? wf[q][2] : 1.0f - wf[q][2]);
                        const long long to = at + (c & 1) + ((c & 2) ? v.nx : 0) + ((c & 4) ? sxy : 0);
                        if (w == 0.0f) continue;
                        if (fix) atomicAdd(fix + to, (unsigned long long)__double2ll_rn((double)w * fsc));
                        else atomicAdd(gZ + to, w);
                    }
                }
                continue;
            }
            // runs of a lane summed in registers, one LDS atomic per corner and run
            if (mine) {
                const int off[8] = {0, 1, rs, rs + 1, ps, ps + 1, ps + rs, ps + rs + 1};
                // box index of a cell from its volume coordinates (24-bit
                // products; the constant wraps)
                const unsigned org = (unsigned)oz * (unsigned)ps + (unsigned)oy * (unsigned)rs + (unsigned)ox;
                float ra[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                int cur = 0;
#pragma unroll
                for (int q = 0; q < kScatterSpl; ++q) {
                    const int l = (int)(__umul24((unsigned)ci[q][2], (unsigned)ps) +
                                        __umul24((unsigned)ci[q][1], (unsigned)rs) + (unsigned)ci[q][0] - org);
                    if (q > 0 && l != cur) {
#pragma unroll
                        for (int c = 0; c < 8; ++c) {
                            atomicAdd(&s_box[cur + off[c]], (double)ra[c]);
                            ra[c] = 0.0f;
                        }
                    }
                    cur = l;
                    const float wx = wf[q][0], wy = wf[q][1], wz = wf[q][2];
                    const float gy = 1.0f - wy, gz = 1.0f - wz;
                    const float x1 = zb[q] * wx, x0 = zb[q] * (1.0f - wx);
                    const float x0y0 = x0 * gy, x1y0 = x1 * gy, x0y1 = x0 * wy, x1y1 = x1 * wy;
                    ra[0] = fmaf(x0y0, gz, ra[0]);
                    ra[1] = fmaf(x1y0, gz, ra[1]);
                    ra[2] = fmaf(x0y1, gz, ra[2]);
                    ra[3] = fmaf(x1y1, gz, ra[3]);
                    ra[4] = fmaf(x0y0, wz, ra[4]);
                    ra[5] = fmaf(x1y0, wz, ra[5]);
                    ra[6] = fmaf(x0y1, wz, ra[6]);
                    ra[7] = fmaf(x1y1, wz, ra[7]);
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) atomicAdd(&s_box[cur + off[c]], (double)ra[c]);
            }
            wave_sync();
            // wave priority 1 for the flush (LDS reads and the global atomics wait
            // on latency): in the two-chain step it then runs ahead of the other
            // chain's arithmetic on the same CUs (step 0.5% faster)
            __builtin_amdgcn_s_setprio(1);
            // Flush: the lanes cover the (x, y) plane of the box, x fastest
            // (consecutive lanes on consecutive voxels of a row), and step along
            // z with one add per entry; or (x, z) planes along y, whichever fills
            // the lanes better.  Four entries' LDS reads go out before their
            // atomics; lanes past the plane read the entry that stays zero.
            {
                const bool xy = ((bx * by + 63) >> 6) * bz <= ((bx * bz + 63) >> 6) * by;
                const int b2 = xy ? by : bz, b3 = xy ? bz : by;
                const int s2 = xy ? rs : ps, s3 = xy ? ps : rs;
                // (voxel indices fit 31 bits)
                const unsigned g2 = xy ? v.nx : sxy, g3 = xy ? sxy : v.nx;
                const unsigned org = (unsigned)oz * sxy + (unsigned)oy * v.nx + ox;
                const float rbx = __builtin_amdgcn_rcpf((float)bx);
                for (int e0 = 0; e0 < bx * b2; e0 += 64) {
                    const int e = e0 + lane;
                    const int y = small_quot(e, rbx), x = e - y * bx;
                    const bool ok = y < b2;
                    int at = ok ? x + y * s2 : CAP;
                    const int sa = ok ? s3 : 0;
                    unsigned gi = org + x + (ok ? y * g2 : 0);
                    for (int z = 0; z < b3; z += 4) {
                        double val[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) val[u] = (z + u < b3) ? s_box[at + u * sa] : 0.0;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (val[u] != 0.0) {
                                s_box[at + u * sa] = 0.0;
                                if (fix) {
                                    atomicAdd(fix + gi + u * g3, (unsigned long long)__double2ll_rn(val[u] * fsc));
                                } else {
                                    const float xv = (float)val[u];
                                    if (xv != 0.0f) atomicAdd(gZ + gi + u * g3, xv);
                                }
                            }
                        }
                        at += 4 * sa;
                        gi += 4 * g3;
                    }
                }
            }
            __builtin_amdgcn_s_setprio(0);
            wave_sync();
        }
    }
}

// --------------------------------------------------------------------------
// lateral blur (Sec. 2.4): per depth row k, a normalised Gaussian along the
// ray index, sigma_k = s0 + (s1 - s0) k / (S - 1) rays, radius ceil(3 sigma)
// decided in float32, edge replicate.  A block of 4 wavefronts takes 64 rays
// x 64 depths; lanes run along depth (coalesced 256-byte rows) and each
// wavefront owns 16 consecutive rays.  A wavefront loads its rows plus the
// halo of RM rays on either side straight into registers (all loads issued
// before the first use) and keeps its depth's weights in registers, so no
// LDS staging and no block barrier sits between the loads and the sums.
//   MODE 0: out = B in            MODE 1: out = B^T in
//   MODE 2: image = B in, out = 2 (image - target) / P, loss += |.|^2 / P
// RM (4, 8, 16, 32) is a register bound on the radius: taps beyond a row's
// own radius carry weight zero and leave the sums unchanged.
// --------------------------------------------------------------------------
constexpr int kBlurRays = 64;      // rays per block
constexpr int kBlurRows = 16;      // rays per wavefront

// normalised weights w_t (t = 0..RM, zero beyond the row radius r) of depth
// row k; returns r (-1: identity row, w_0 = 1)
template <int RM>
__device__ __forceinline__ int blur_weights(const PhysArgs &p, int S, int k, float (&w)[RM + 1])
{
    const float frac = S > 1 ? __fdiv_rn((float)k, (float)(S - 1)) : 0.0f;
    const float d = __fsub_rn(p.s1, p.s0);
    const float sig = __fadd_rn(p.s0, __fmul_rn(d, frac));
    if (!(sig >= 1e-3f)) {
#pragma unroll
        for (int t = 0; t <= RM; ++t) w[t] = (t == 0) ? 1.0f : 0.0f;
        return -1;
    }
    int r = (int)ceilf(__fmul_rn(3.0f, sig));
    r = min(r, min(p.blur_rmax, RM));
    const float c = -0.5f / (sig * sig);
    float e[RM + 1];
    float tot = 1.0f;
#pragma unroll
    for (int t = 1; t <= RM; ++t) {
        e[t] = (t <= r) ? expf(c * (float)(t * t)) : 0.0f;
        if (t <= r) tot += 2.0f * e[t];
    }
    const float inv = 1.0f / tot;
    w[0] = inv;
#pragma unroll
    for (int t = 1; t <= RM; ++t) w[t] = e[t] * inv;
    return r;
}

template <int MODE, int RM>
__global__ __launch_bounds__(256) void k_blur(PhysArgs p, FanTable tab, const float *__restrict__ in,
                                              const float *__restrict__ target, float *__restrict__ out,
                                              float *__restrict__ image, double *__restrict__ loss_acc)
{
    constexpr int W = kBlurRows + 2 * RM;      // window rows j0 - RM .. j0 + 16 + RM - 1
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int b = blockIdx.x;
    const int fi = find_blur_fan(tab, b);
    const FanRec fr = tab.f[fi];
    const int S = fr.n_samples, n = fr.n_rays;
    const int nkb = (S + 63) / 64;
    const int lb = b - fr.blk_begin;
    const int kb = lb % nkb, jb = lb / nkb;
    const int k = kb * 64 + lane;
    const int j0 = jb * kBlurRays + wv * kBlurRows;
    const bool active = (k < S) && (j0 < n);
    const long long col = fr.out_offset + k;
    const double inv_npix = 1.0 / ((double)n * (double)S);
    const float two_inv_npix = (float)(2.0 * inv_npix);
    double lsum = 0.0;
    if (active) {
        // every load clamped into the fan (no per-load branches): MODE 1
        // then zeroes the rows outside it, the others replicate the edge
        float x[W];
#pragma unroll
        for (int m = 0; m < W; ++m) {
            const int g = j0 - RM + m;
            x[m] = in[col + (long long)min(max(g, 0), n - 1) * S];
        }
        float tg[MODE == 2 ? kBlurRows : 1];
        if (MODE == 2) {
#pragma unroll
            for (int o = 0; o < kBlurRows; ++o) tg[o] = target[col + (long long)min(j0 + o, n - 1) * S];
        }
        if (MODE == 1) {
#pragma unroll
            for (int m = 0; m < W; ++m) {
                const int g = j0 - RM + m;
                x[m] = (g >= 0 && g < n) ? x[m] : 0.0f;
            }
        }
        float w[RM + 1];
        const int r = blur_weights<RM>(p, S, k, w);
        // transpose at the edge rows 0 and n-1: the replicated taps fold back
        // onto the edge, weight tail_m = sum_{t >= m} w_t for the tap |t| + 1
        float tl[RM + 2];
        if (MODE == 1) {
            float acc = 0.0f;
            tl[RM + 1] = 0.0f;
#pragma unroll
            for (int t = RM; t >= 0; --t) {
                if (t <= r) acc += w[t];
                tl[t] = (t <= r) ? acc : 0.0f;
            }
        }
#pragma unroll
        for (int o = 0; o < kBlurRows; ++o) {
            const int j = j0 + o;
            if (j >= n) break;
            float acc = 0.0f;
#pragma unroll
            for (int t = -RM; t <= RM; ++t) acc = fmaf(w[t < 0 ? -t : t], x[o + RM + t], acc);
            if (MODE == 1 && (j == 0 || j == n - 1)) {
                const float mult = (j == 0 && j == n - 1) ? 2.0f : 1.0f;
                float e = 0.0f;
#pragma unroll
                for (int t = -RM; t <= RM; ++t) e = fmaf(tl[(t < 0 ? -t : t) + 1], x[o + RM + t], e);
                acc = fmaf(mult, e, acc);
            }
            const long long oidx = col + (long long)j * S;
            if (MODE == 2) {
                // residual in FP32 (one rounding of the difference of two
                // floats); its square summed in FP64, scaled once at the end
                const float d = acc - tg[o];
                if (image) image[oidx] = acc;
                out[oidx] = d * two_inv_npix;
                lsum += (double)(d * d);
            } else {
                out[oidx] = acc;
            }
        }
    }
    if (MODE == 2 && loss_acc) {
        // one partial per block, summed by k_sum_f64 (no contended atomics)
        __shared__ double s_part[4];
        lsum = wave_sum(lsum) * inv_npix;
        if (lane == 0) s_part[wv] = lsum;
        __syncthreads();
        if (tid == 0) loss_acc[b] = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
    }
}

// Residual and transpose blur in one pass (the fused step with blur, radius
// bound RM <= 8): ebar = B^T (2 (B pre - target) / P), image = B pre
// (optional), one loss partial per block.  A block of 4 wavefronts takes 64
// rays x 64 depths as k_blur does.  It first forms the residual of its rays
// and of RM rays on either side (each wavefront RW of those 64 + 2 RM rows,
// from a register window of pre, as MODE 2), parks it in LDS (zero outside
// the fan, as MODE 1 reads it), and then applies B^T to its own rows from
// LDS, as MODE 1.  The arithmetic of each value is that of the two-kernel
// path; only the loss partials group the rows differently.  The residual
// never goes to memory.
template <int RM>
__global__ __launch_bounds__(256) void k_blur_fused(PhysArgs p, FanTable tab, const float *__restrict__ pre,
                                                    const float *__restrict__ target, float *__restrict__ ebar,
                                                    float *__restrict__ image, double *__restrict__ loss_acc)
{
    constexpr int NR = kBlurRays + 2 * RM;     // residual rows J0 - RM .. J0 + 64 + RM - 1
    constexpr int RW = NR / 4;                 // residual rows per wavefront
    constexpr int W = RW + 2 * RM;             // pre window of a wavefront
    static_assert(NR % 4 == 0, "residual rows split over four wavefronts");
    __shared__ float s_r[NR][65];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int b = blockIdx.x;
    const int fi = find_blur_fan(tab, b);
    const FanRec fr = tab.f[fi];
    const int S = fr.n_samples, n = fr.n_rays;
    const int nkb = (S + 63) / 64;
    const int lb = b - fr.blk_begin;
    const int kb = lb % nkb, jb = lb / nkb;
    const int k = kb * 64 + lane;
    const int J0 = jb * kBlurRays;
    const bool kin = k < S;
    const long long col = fr.out_offset + min(k, S - 1);
    const double inv_npix = 1.0 / ((double)n * (double)S);
    const float two_inv_npix = (float)(2.0 * inv_npix);
    float w[RM + 1];
    const int r = blur_weights<RM>(p, S, min(k, S - 1), w);
    double lsum = 0.0;
    {
        // residual rows g0 .. g0 + RW - 1 of this wavefront
        const int g0 = J0 - RM + wv * RW;
        float x[W];
#pragma unroll
        for (int m = 0; m < W; ++m) {
            const int g = g0 - RM + m;
            x[m] = pre[col + (long long)min(max(g, 0), n - 1) * S];
        }
        float tg[RW];
#pragma unroll
        for (int o = 0; o < RW; ++o) tg[o] = target[col + (long long)min(max(g0 + o, 0), n - 1) * S];
#pragma unroll
        for (int o = 0; o < RW; ++o) {
            const int g = g0 + o;
            float acc = 0.0f;
#pragma unroll
            for (int t = -RM; t <= RM; ++t) acc = fmaf(w[t < 0 ? -t : t], x[o + RM + t], acc);
            const float d = acc - tg[o];
            const bool in_fan = kin && g >= 0 && g < n;
            s_r[wv * RW + o][lane] = in_fan ? d * two_inv_npix : 0.0f;
            // the block's own rows: image and loss
            if (in_fan && g >= J0 && g < J0 + kBlurRays) {
                if (image) image[col + (long long)g * S] = acc;
                lsum += (double)(d * d);
            }
        }
    }
    __syncthreads();
    // transpose blur of this wavefront's 16 rays from the LDS residual
    const int j0 = J0 + wv * kBlurRows;
    if (kin && j0 < n) {
        float tl[RM + 2];
        {
            float acc = 0.0f;
            tl[RM + 1] = 0.0f;
#pragma unroll
            for (int t = RM; t >= 0; --t) {
                if (t <= r) acc += w[t];
                tl[t] = (t <= r) ? acc : 0.0f;
            }
        }
        float x[kBlurRows + 2 * RM];
#pragma unroll
        for (int m = 0; m < kBlurRows + 2 * RM; ++m) x[m] = s_r[wv * kBlurRows + m][lane];
#pragma unroll
        for (int o = 0; o < kBlurRows; ++o) {
            const int j = j0 + o;
            if (j >= n) break;
            float acc = 0.0f;
#pragma unroll
            for (int t = -RM; t <= RM; ++t) acc = fmaf(w[t < 0 ? -t : t], x[o + RM + t], acc);
            if (j == 0 || j == n - 1) {
                const float mult = (j == 0 && j == n - 1) ? 2.0f : 1.0f;
                float e = 0.0f;
#pragma unroll
                for (int t = -RM; t <= RM; ++t) e = fmaf(tl[(t < 0 ? -t : t) + 1], x[o + RM + t], e);
                acc = fmaf(mult, e, acc);
            }
            ebar[col + (long long)j * S] = acc;
        }
    }
    if (loss_acc) {
        // one partial per block, summed by k_sum_f64 (no contended atomics)
        __shared__ double s_part[4];
        lsum = wave_sum(lsum) * inv_npix;
        if (lane == 0) s_part[wv] = lsum;
        __syncthreads();
        if (tid == 0) loss_acc[b] = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
    }
}

// --------------------------------------------------------------------------
// pose gradient: dL/dt and dL/dw from the accumulated dL/dR (Gallego-Yezzi)
// --------------------------------------------------------------------------
__device__ void skew(const double w[3], double W[9])
{
    W[0] = 0.0;   W[1] = -w[2]; W[2] = w[1];
    W[3] = w[2];  W[4] = 0.0;   W[5] = -w[0];
    W[6] = -w[1]; W[7] = w[0];  W[8] = 0.0;
}

__device__ void mm3(const double *A, const double *B, double *Cm)
{
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
            Cm[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}

// dL/dw_c of pose pi from its accumulator a (dL/dt, dL/dR)
__device__ double pose_rotation_grad(const double *a, const float *__restrict__ poses, int pi, int c)
{
    const double w[3] = {poses[6 * pi + 3], poses[6 * pi + 4], poses[6 * pi + 5]};
    const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
    double W[9];
    skew(w, W);
    double dR[9];
    double e[3];
    for (int q = 0; q < 3; ++q) e[q] = (q == c) ? 1.0 : 0.0;
    double E[9];
    skew(e, E);
    if (th2 < 1e-10) {
        double EW[9], WE[9];
        mm3(E, W, EW);
        mm3(W, E, WE);
        for (int q = 0; q < 9; ++q) dR[q] = E[q] + 0.5 * (EW[q] + WE[q]);
    } else {
        double R[9];
        rotation(w, R);
        double vv[3];
        for (int q = 0; q < 3; ++q) vv[q] = e[q] - (c == 0 ? R[3 * q] : (c == 1 ? R[3 * q + 1] : R[3 * q + 2]));
        const double x[3] = {w[1] * vv[2] - w[2] * vv[1], w[2] * vv[0] - w[0] * vv[2],
                             w[0] * vv[1] - w[1] * vv[0]};
        const double wc = (c == 0) ? w[0] : (c == 1 ? w[1] : w[2]);
        double X[9], Sm[9];
        skew(x, X);
        for (int q = 0; q < 9; ++q) Sm[q] = (wc * W[q] + X[q]) / th2;
        mm3(Sm, R, dR);
    }
    double s = 0.0;
    for (int q = 0; q < 9; ++q) s += a[3 + q] * dR[q];
    return s;
}

// (dL/dt, dL/dw) of every pose, one thread per component
__device__ __forceinline__ void pose_finalize(const double *__restrict__ acc, const float *__restrict__ poses, int n,
                                              float *__restrict__ grad, int i)
{
    const int pi = i / 6, c = i - 6 * pi;
    if (pi >= n) return;
    const double *a = acc + (size_t)kPoseAcc * pi;
    grad[i] = (float)(c < 3 ? a[c] : pose_rotation_grad(a, poses, pi, c - 3));
}

__global__ __launch_bounds__(192) void k_pose_finalize(const double *__restrict__ acc, const float *__restrict__ poses,
                                                       int n, float *__restrict__ grad)
{
    pose_finalize(acc, poses, n, grad, blockIdx.x * 192 + threadIdx.x);
}

// One block per fan of a table: the per-ray partials of the adjoint summed
// (in a fixed order) and, with tab.grad_pose, turned into the pose's gradient
// at once; without, added into the pose's accumulator.  With tab.loss, one
// block more sums a small step's loss partials, which saves it a launch
// (pose-only step of 4 poses x 296 rays x 127 samples 18.7 -> 15.8 us, full
// step of 6 x 171 x 729 54 -> 52).
__global__ __launch_bounds__(256) void k_pose_reduce(FanTable tab, const double *__restrict__ part,
                                                     double *__restrict__ acc)
{
    __shared__ double s_w[4][kRayPart];
    __shared__ double s_a[kPoseAcc];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if ((int)blockIdx.x == tab.n) {
        double x[4] = {0.0, 0.0, 0.0, 0.0};
        for (int i = threadIdx.x; i < tab.n_part; i += 1024) {
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] += (i + 256 * u < tab.n_part) ? tab.loss_part[i + 256 * u] : 0.0;
        }
        const double t = lanes_sum((x[0] + x[1]) + (x[2] + x[3]));
        if (lane == 0) s_w[wv][0] = t;
        __syncthreads();
        if (threadIdx.x == 0) *tab.loss = (s_w[0][0] + s_w[1][0]) + (s_w[2][0] + s_w[3][0]);
        return;
    }
    const FanRec fr = tab.f[blockIdx.x];
    double s[kRayPart];
#pragma unroll
    for (int c = 0; c < kRayPart; ++c) s[c] = 0.0;
    for (int j = threadIdx.x; j < fr.n_rays; j += 256) {
        const double *pr = part + (size_t)kRayPart * (fr.ray_begin + j);
#pragma unroll
        for (int c = 0; c < kRayPart; ++c) s[c] += pr[c];
    }
#pragma unroll
    for (int c = 0; c < kRayPart; ++c) {
        s[c] = lanes_sum(s[c]);
        if (lane == 0) s_w[wv][c] = s[c];
    }
    __syncthreads();
    // entry c of the partials is entry at[c] of (dL/dt, dL/dR by rows)
    if (threadIdx.x < kRayPart) {
        const int c = threadIdx.x;
        const int at = (c < 3) ? c : 3 + 3 * ((c - 3) >> 1) + 2 * ((c - 3) & 1);
        s_a[at] = (s_w[0][c] + s_w[1][c]) + (s_w[2][c] + s_w[3][c]);
        if (c < 3) s_a[4 + 3 * c] = 0.0;        // the ray direction's y component
    }
    __syncthreads();
    if (tab.grad_pose) {
        if (threadIdx.x < 6) {
            const int c = threadIdx.x;
            tab.grad_pose[6 * (size_t)fr.pose + c] =
                (float)(c < 3 ? s_a[c] : pose_rotation_grad(s_a, tab.poses, fr.pose, c - 3));
        }
    } else if (threadIdx.x < kPoseAcc) {
        acc[(size_t)kPoseAcc * fr.pose + threadIdx.x] += s_a[threadIdx.x];
    }
}

// --------------------------------------------------------------------------
// footprint: mark every stencil corner of every sample
// --------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_footprint(VolArgs v, FanTable tab, const float *__restrict__ poses,
                                                  uint8_t *__restrict__ mask)
{
    const int lane = threadIdx.x;
    const int g = blockIdx.x;
    const int fi = find_fan(tab, g);
    const FanRec fr = tab.f[fi];
    const int j = g - fr.ray_begin;
    PhysArgs p{};
    p.atten = 2;
    Ray ray;
    setup_ray(v, p, fr, poses, j, ray);
    const int sxy = v.nx * v.ny;
    for (int k = lane; k < fr.n_samples; k += 64) {
        const Stencil st = stencil_at(v, ray, k);
        uint8_t *q = mask + st.idx;
        q[0] = 1;
        q[1] = 1;
        q[v.nx] = 1;
        q[v.nx + 1] = 1;
        q[sxy] = 1;
        q[sxy + 1] = 1;
        q[sxy + v.nx] = 1;
        q[sxy + v.nx + 1] = 1;
    }
}

// --------------------------------------------------------------------------
// sampling-only render: the impedance at every ray sample (one wavefront per
// ray, coalesced stores)
// --------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_sample_rays(VolArgs v, FanTable tab, const float *__restrict__ poses,
                                                   float *__restrict__ out, int xgrp)
{
    const int lane = threadIdx.x;
    const int g = remap_block(blockIdx.x, gridDim.x, xgrp);
    const int fi = find_fan(tab, g);
    const FanRec fr = tab.f[fi];
    const int j = g - fr.ray_begin;
    const int S = fr.n_samples;
    PhysArgs p{};
    p.atten = 2;
    Ray ray;
    setup_ray(v, p, fr, poses, j, ray);
    const long long obase = fr.out_offset + (long long)j * S;
    const int sxy = v.nx * v.ny;
#pragma unroll 4
    for (int k = lane; k < S; k += 64) {
        const Stencil st = stencil_at(v, ray, k);
        out[obase + k] = (float)trilinear(v.Z, v.nx, sxy, st, nullptr);
    }
}

// --------------------------------------------------------------------------
// scan conversion of one fan's polar image onto a Cartesian grid of the
// probe's x-z plane (one thread per output pixel, FP64 geometry)
// --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_scan_convert(const float *__restrict__ img, int n_r, int S, double A,
                                                      double r0, double ds, int nx, int nz, double x0, double z0,
                                                      double dx, double dz, float fill, float *__restrict__ out)
{
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)nx * nz) return;
    const int iz = (int)(idx / nx), ix = (int)(idx - (long long)iz * nx);
    const double x = x0 + (double)ix * dx, z = z0 + (double)iz * dz;
    const double r = sqrt(x * x + z * z);
    const double th = atan2(x, z);
    const double jr = (th + 0.5 * A) * (double)(n_r - 1) / A;
    const double kr = (r - r0) / ds;
    if (!(jr >= 0.0 && jr <= (double)(n_r - 1) && kr >= 0.0 && kr <= (double)(S - 1))) {
        out[idx] = fill;
        return;
    }
    const int j0 = min((int)floor(jr), n_r - 2), k0 = min((int)floor(kr), S - 2);
    const double fj = jr - (double)j0, fk = kr - (double)k0;
    const float *p0 = img + (long long)j0 * S + k0;
    const float *p1 = p0 + S;
    const double a = lerp((double)p0[0], (double)p0[1], fk);
    const double b = lerp((double)p1[0], (double)p1[1], fk);
    out[idx] = (float)lerp(a, b, fj);
}

// --------------------------------------------------------------------------
// small utilities
// --------------------------------------------------------------------------
__global__ void k_zero_f64(double *p, long long n)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

__global__ void k_zero_f32(float *p, long long n)
{
    const long long n4 = n / 4;
    float4 *p4 = reinterpret_cast<float4 *>(p);
    const bool aligned = ((reinterpret_cast<uintptr_t>(p) & 15) == 0);
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long i0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (aligned) {
        for (long long i = i0; i < n4; i += stride) p4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (long long i = 4 * n4 + i0; i < n; i += stride) p[i] = 0.0f;
    } else {
        for (long long i = i0; i < n; i += stride) p[i] = 0.0f;
    }
}

// out = sum of n partials, or out += it (single block, fixed order:
// deterministic); four partials of a thread in flight
constexpr int kSumThreads = 1024;

__device__ __forceinline__ void sum_block(const double *__restrict__ part, long long n, double *__restrict__ out,
                                          int accumulate)
{
    __shared__ double s_w[kSumThreads / 64];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (long long i = threadIdx.x; i < n; i += 4 * kSumThreads) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long at = i + u * kSumThreads;
            const double x = part[at < n ? at : i];
            acc[u] += at < n ? x : 0.0;
        }
    }
    const double t = lanes_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x < 64) {
        const double all = lanes_sum(threadIdx.x < kSumThreads / 64 ? s_w[threadIdx.x] : 0.0);
        if (threadIdx.x == 0) *out = accumulate ? *out + all : all;
    }
}

__global__ __launch_bounds__(kSumThreads) void k_sum_f64(const double *__restrict__ part, long long n,
                                                         double *__restrict__ out, int accumulate)
{
    sum_block(part, n, out, accumulate);
}

// the loss and the pose gradients in one launch: block 0 sums the loss
// partials (when loss is given), the other blocks finalise the poses
__global__ __launch_bounds__(kSumThreads) void k_finish(const double *__restrict__ part, long long n_part,
                                                double *__restrict__ loss, const double *__restrict__ acc,
                                                const float *__restrict__ poses, int n_poses,
                                                float *__restrict__ grad)
{
    if (loss && blockIdx.x == 0) {
        sum_block(part, n_part, loss, 0);
        return;
    }
    if (grad) pose_finalize(acc, poses, n_poses, grad, (blockIdx.x - (loss ? 1 : 0)) * kSumThreads + threadIdx.x);
}

// deterministic dL/dZ: the sum of |dL/dZ| over every sample of the step
// bounds every voxel's sum (the trilinear weights of a sample are at most 1
// and add up to 1), and sets the fixed-point scale 2^e with that bound times
// 2^e below 2^61, so no 64-bit sum can overflow however the atomics are
// ordered.  Each wavefront sums one ray's row (the rows of the fans only:
// gaps between pose images are never read), in a fixed order
__global__ __launch_bounds__(256) void k_abs_rows(FanTable tab, const float *__restrict__ zbar,
                                                  double *__restrict__ part)
{
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (g >= tab.total_rays) return;            // whole wavefront
    const FanRec fr = tab.f[find_fan(tab, g)];
    const int S = fr.n_samples;
    const float *row = zbar + fr.out_offset + (long long)(g - fr.ray_begin) * S;
    double acc = 0.0;
    for (int k = lane; k < S; k += 64) acc += fabs((double)row[k]);
    acc = wave_sum(acc);
    if (lane == 0) part[g] = acc;
}

// fscale[2] = the sum of the n per-ray sums (one block, fixed order), and
// fscale[0..1] = 2^e, 2^-e
__global__ __launch_bounds__(kSumThreads) void k_fix_scale(const double *__restrict__ part, long long n,
                                                   double *__restrict__ fscale)
{
    sum_block(part, n, fscale + 2, 0);
    __syncthreads();
    if (threadIdx.x == 0) {
        const double a = fscale[2];
        const int e = (a > 0.0 && isfinite(a)) ? 60 - ilogb(a) : 0;
        fscale[0] = ldexp(1.0, e);
        fscale[1] = ldexp(1.0, -e);
    }
}

// grad_Z (+)= the fixed-point sums times 2^-e, rounded once to FP32
__global__ __launch_bounds__(256) void k_fix_to_f32(const unsigned long long *__restrict__ fix, long long n,
                                                    const double *__restrict__ fscale, float *__restrict__ gZ,
                                                    int overwrite)
{
    const double inv = fscale[1];
    const long long stride = (long long)gridDim.x * 256;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
        const double x = (double)(long long)fix[i] * inv;
        gZ[i] = overwrite ? (float)x : (float)((double)gZ[i] + x);
    }
}

// two buffers cleared in one launch (grid-stride over both)
__global__ void k_zero_pair(float *__restrict__ a, long long na, double *__restrict__ b, long long nb)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    const long long i0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    const long long n4 = na / 4;
    float4 *a4 = reinterpret_cast<float4 *>(a);
    if ((reinterpret_cast<uintptr_t>(a) & 15) == 0) {
        for (long long i = i0; i < n4; i += stride) a4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (long long i = 4 * n4 + i0; i < na; i += stride) a[i] = 0.0f;
    } else {
        for (long long i = i0; i < na; i += stride) a[i] = 0.0f;
    }
    for (long long i = i0; i < nb; i += stride) b[i] = 0.0;
}

// --------------------------------------------------------------------------
// volume reconstruction helpers: the smoothness prior
//   R = w sum_axes sum_{pairs along the axis} ((Z_b - Z_a) / h_axis)^2
// (four voxels per thread: grad_Z += dR/dZ of its own voxels, and the energy
// of the pairs to their +x, +y, +z neighbours into a per-block partial), and
// the element-wise Adam update with the result clamped to [lo, hi].  Both are
// bound by memory.  The prior with 16-byte accesses and 32-bit index
// arithmetic, one pair of divisions per thread instead of 64-bit ones per
// voxel: 256^3 voxels 126 -> 38 us (201 MB, 5.3 TB/s), 128^3 with its sum 20.6
// -> 12.6 us; rows that are no multiple of four take the voxels one by one,
// as fast as before (97^3: 12.5 us).
// --------------------------------------------------------------------------
constexpr int kSmoothVoxels = 1024;     // per block

// a voxel's gradient from its neighbours (axis weights w / h^2; d(Z_b - Z_a)^2
// / dZ = -2 (Z_b - Z_a) for a, +2 for b), and its energy added to e.  At the
// faces the missing neighbour is the voxel itself: its difference is zero.
__device__ __forceinline__ float smooth_voxel(float z, float xm, float xp, float ym, float yp, float zm, float zp,
                                              float wx, float wy, float wz, double &e)
{
    float g = 0.0f;
    g += 2.0f * wx * (z - xm);
    { const float d = xp - z; g -= 2.0f * wx * d; e += (double)wx * (double)d * (double)d; }
    g += 2.0f * wy * (z - ym);
    { const float d = yp - z; g -= 2.0f * wy * d; e += (double)wy * (double)d * (double)d; }
    g += 2.0f * wz * (z - zm);
    { const float d = zp - z; g -= 2.0f * wz * d; e += (double)wz * (double)d * (double)d; }
    return g;
}

__global__ __launch_bounds__(256) void k_smooth(const float *__restrict__ Z, int nx, int ny, int nz, float wx,
                                                float wy, float wz, float *__restrict__ gZ,
                                                double *__restrict__ part)
{
    const unsigned n = (unsigned)nx * ny * nz;      // below 2^31
    const unsigned v0 = (blockIdx.x * 256 + threadIdx.x) * 4;
    const int sxy = nx * ny;
    double e = 0.0;
    if (v0 < n) {
        const unsigned row = v0 / (unsigned)nx;
        int ix = (int)(v0 - row * nx), iy = (int)(row % (unsigned)ny), iz = (int)(row / (unsigned)ny);
        if ((nx & 3) == 0) {
            // the four voxels lie in one row
            const float4_u z = *reinterpret_cast<const float4_u *>(Z + v0);
            const float4_u ym = *reinterpret_cast<const float4_u *>(Z + v0 - (iy > 0 ? nx : 0));
            const float4_u yp = *reinterpret_cast<const float4_u *>(Z + v0 + (iy + 1 < ny ? nx : 0));
            const float4_u zm = *reinterpret_cast<const float4_u *>(Z + v0 - (iz > 0 ? sxy : 0));
            const float4_u zp = *reinterpret_cast<const float4_u *>(Z + v0 + (iz + 1 < nz ? sxy : 0));
            const float xm = Z[v0 - (ix > 0 ? 1 : 0)], xp = Z[v0 + (ix + 4 < nx ? 4 : 3)];
            float4_u g = *reinterpret_cast<const float4_u *>(gZ + v0);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                g[u] += smooth_voxel(z[u], u > 0 ? z[u > 0 ? u - 1 : 0] : xm, u < 3 ? z[u < 3 ? u + 1 : 3] : xp, ym[u],
                                     yp[u], zm[u], zp[u], wx, wy, wz, e);
            *reinterpret_cast<float4_u *>(gZ + v0) = g;
        } else {
            for (int u = 0; u < 4 && v0 + u < n; ++u) {
                const float *p = Z + v0 + u;
                gZ[v0 + u] += smooth_voxel(p[0], p[-(ix > 0 ? 1 : 0)], p[ix + 1 < nx ? 1 : 0], p[-(iy > 0 ? nx : 0)],
                                           p[iy + 1 < ny ? nx : 0], p[-(iz > 0 ? sxy : 0)], p[iz + 1 < nz ? sxy : 0],
                                           wx, wy, wz, e);
                if (++ix == nx) {
                    ix = 0;
                    if (++iy == ny) {
                        iy = 0;
                        ++iz;
                    }
                }
            }
        }
    }
    __shared__ double s_w[4];
    e = lanes_sum(e);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
}

__global__ __launch_bounds__(256) void k_adam(float *__restrict__ x, const float *__restrict__ g,
                                              float *__restrict__ m, float *__restrict__ v, long long n, float lr,
                                              float b1, float b2, float eps, float c1, float c2, float lo, float hi)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        // bias corrections c1 = 1 - b1^t, c2 = 1 - b2^t
        const float step = lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        x[i] = fminf(fmaxf(x[i] - step, lo), hi);
    }
}

// --------------------------------------------------------------------------
// impedance mapping (Sec. 2.2): the paper turns MRI or CT intensities into
// impedance voxel by voxel.  Here the map is a piecewise-linear table
// (x_j, z_j), constant beyond its ends; a voxel of intensity v in
// [x_j, x_{j+1}) maps to z_j + t (z_{j+1} - z_j), t = (v - x_j) / (x_{j+1} - x_j).
//
// Both directions are bound by memory.  A thread takes four neighbouring
// voxels (16-byte accesses), and the next four's loads go out before this
// four's arithmetic.  A table of up to kScanKnots knots is searched by
// counting the knots below v, in scalar registers (two vector instructions a
// knot, no LDS round trip); a longer one by halving in LDS.  256^3 voxels, 12
// knots: the map 40 -> 26 us (134 MB at 5.1 TB/s, the rate of a large copy),
// its adjoint 86 -> 47 us (201 MB; 42 us without the table gradient); 40
// knots: 46 -> 41 and 119 -> 64 us.
// --------------------------------------------------------------------------
constexpr int kScanKnots = 16;

// a segment's values, read with one LDS access
struct alignas(16) LutSeg {
    float x, dx, z, dz;
};

// segment j of v (x_j <= v < x_{j+1}, 0 <= j <= n - 2) for x_0 < v < x_{n-1};
// else some segment (0 for NaN).  top: the largest power of two <= n - 2, or
// 0 when n = 2.
template <bool SCAN>
__device__ __forceinline__ int lut_segment(const LutArgs &lut, const float *sx, int top, float v)
{
    int j = 0;
    if (SCAN) {
        // (lut.x beyond the table's inner knots holds +inf, which no v below
        // x_{n-1} reaches)
#pragma unroll
        for (int k = 1; k < kScanKnots - 1; ++k) j += (v >= lut.x[k]) ? 1 : 0;
        return min(j, lut.n - 2);
    }
    // branch-free search in LDS, one halving step per bit of n - 2
    for (int s = top; s > 0; s >>= 1) {
        const int c = j + s;
        j = (c <= lut.n - 2 && v >= sx[c]) ? c : j;      // (c <= 2 top - 1 < kMaxKnots)
    }
    return j;
}

__device__ __forceinline__ int lut_top(int n) { return n > 2 ? 1 << (31 - __builtin_clz(n - 2)) : 0; }

__device__ __forceinline__ float lut_fraction(float v, const LutSeg &s) { return __fdiv_rn(v - s.x, s.dx); }

// the table in LDS: segments, and for the halving search the knots packed
// (their banks differ)
__device__ __forceinline__ void lut_fill(const LutArgs &lut, LutSeg *seg, float *sx)
{
    const int i = threadIdx.x;
    if (i < lut.n - 1) seg[i] = LutSeg{lut.x[i], lut.x[i + 1] - lut.x[i], lut.z[i], lut.z[i + 1] - lut.z[i]};
    if (i < kMaxKnots) sx[i] = lut.x[i];
    __syncthreads();
}

// four floats from element i of an array of n, those past its end zero (and
// not stored)
__device__ __forceinline__ float4_u load4(const float *__restrict__ p, long long i, long long n)
{
    if (i + 4 <= n) return *reinterpret_cast<const float4_u *>(p + i);
    float4_u x = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int u = 0; u < 4; ++u)
        if (i + u < n) x[u] = p[i + u];
    return x;
}

__device__ __forceinline__ void store4(float *__restrict__ p, long long i, long long n, const float4_u &x)
{
    if (i + 4 <= n) {
        // (not read again here: past the caches, the map 30 -> 26 us)
        __builtin_nontemporal_store(x, reinterpret_cast<float4_u *>(p + i));
        return;
    }
    for (int u = 0; u < 4; ++u)
        if (i + u < n) p[i + u] = x[u];
}

template <bool SCAN>
__global__ __launch_bounds__(256) void k_map(const float *__restrict__ in, long long n, LutArgs lut,
                                             float *__restrict__ Z)
{
    __shared__ LutSeg s_seg[kMaxKnots];
    __shared__ float s_x[kMaxKnots];
    lut_fill(lut, s_seg, s_x);
    const float x0 = lut.x0, xn = lut.xn, z0 = lut.z[0], zn = lut.z[lut.n - 1];
    const int top = lut_top(lut.n);
    const long long stride = (long long)gridDim.x * 1024;
    long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= n) return;
    float4_u v = load4(in, i, n);
    for (; i < n; i += stride) {
        const float4_u next = load4(in, i + stride, n);
        float4_u z;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const LutSeg s = s_seg[lut_segment<SCAN>(lut, s_x, top, v[u])];
            const float inner = fmaf(lut_fraction(v[u], s), s.dz, s.z);
            // NaN fails both tests and stays NaN
            z[u] = (v[u] <= x0) ? z0 : ((v[u] >= xn) ? zn : inner);
        }
        store4(Z, i, n, z);
        v = next;
    }
}

// dL/dv = dL/dZ (z_{j+1} - z_j) / (x_{j+1} - x_j) inside the table (the right
// segment at a knot), 0 beyond its ends; dL/dz_j += (1 - t) dL/dZ and
// dL/dz_{j+1} += t dL/dZ, or all of dL/dZ to the end knot beyond an end.
// The table gradient is a histogram over the knots: FP64 LDS atomics, one
// column per lane, so that lanes of a wavefront never meet on an address or
// a bank whatever their knots (smooth volumes aim whole wavefronts at one
// knot; with eight columns the atomics cost 28 of 77 us).  The columns are
// added per block, then one global FP64 atomic per knot and block, all knots
// in one instruction: every block's goes to the same few cache lines, about 8
// ns apiece, so the blocks are few and large.
constexpr int kMapThreads = 1024;

template <bool SCAN>
__global__ __launch_bounds__(kMapThreads) void k_map_backward(const float *__restrict__ in, long long n, LutArgs lut,
                                                      const float *__restrict__ gZ, float *__restrict__ grad_in,
                                                      double *__restrict__ grad_z)
{
    __shared__ LutSeg s_seg[kMaxKnots];
    __shared__ double s_g[SCAN ? kScanKnots : kMaxKnots][64];
    __shared__ float s_x[kMaxKnots];
    __shared__ double s_sum[kMaxKnots];
    const int m = lut.n;
    for (int i = threadIdx.x; i < m * 64; i += kMapThreads) s_g[i >> 6][i & 63] = 0.0;
    lut_fill(lut, s_seg, s_x);
    const int lane = threadIdx.x & 63;
    const float x0 = lut.x0, xn = lut.xn;
    const int top = lut_top(m);
    const long long stride = (long long)gridDim.x * 4 * kMapThreads;
    long long i = ((long long)blockIdx.x * kMapThreads + threadIdx.x) * 4;
    float4_u v = load4(in, i, n), g = load4(gZ, i, n);
    for (; i < n; i += stride) {
        const float4_u vn = load4(in, i + stride, n), gn = load4(gZ, i + stride, n);
        float4_u gi;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool below = v[u] <= x0, above = v[u] >= xn;
            const int j = above ? m - 2 : lut_segment<SCAN>(lut, s_x, top, v[u]);
            const LutSeg s = s_seg[j];
            gi[u] = (below || above) ? 0.0f : g[u] * __fdiv_rn(s.dz, s.dx);
            if (grad_z && i + u < n) {
                const double t = (double)lut_fraction(v[u], s), gd = (double)g[u];
                if (!above) atomicAdd(&s_g[j][lane], below ? gd : (1.0 - t) * gd);
                if (!below) atomicAdd(&s_g[j + 1][lane], above ? gd : t * gd);
            }
        }
        if (grad_in) store4(grad_in, i, n, gi);
        v = vn;
        g = gn;
    }
    if (grad_z) {
        __syncthreads();
        // a wavefront per knot
        for (int k = threadIdx.x >> 6; k < m; k += kMapThreads / 64) {
            const double t = lanes_sum(s_g[k][lane]);
            if (lane == 0) s_sum[k] = t;
        }
        __syncthreads();
        if (threadIdx.x < m && s_sum[threadIdx.x] != 0.0) atomicAdd(grad_z + threadIdx.x, s_sum[threadIdx.x]);
    }
}

__global__ void k_philox(const uint32_t *__restrict__ ctr, long long n, uint32_t k0, uint32_t k1,
                         uint32_t *__restrict__ out)
{
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t w[4];
    philox(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1, w);
    for (int q = 0; q < 4; ++q) out[4 * i + q] = w[q];
}

template <bool SPK>
__global__ __launch_bounds__(64) void k_gain(PhysArgs p, FanRec fr, float *__restrict__ out)
{
    constexpr int T = 256;
    __shared__ float s_xig[SPK ? T : 1];
    __shared__ float s_xir[SPK ? T / 4 + 8 : 1];
    const int lane = threadIdx.x;
    const int j = blockIdx.y;
    const int t0 = blockIdx.x * T;
    const int S = fr.n_samples;
    if (SPK) speckle_fill<T>(p, t0, j, fr.speckle_id, lane, s_xig, s_xir);
    __syncthreads();
    const float postc = posthoc_coef(p, fr.ds);
    const GainK gk = gain_consts(p, fr.n_samples);
    for (int m = 0; m < T / 64; ++m) {
        const int i = m * 64 + lane;
        const int k = t0 + i;
        if (k < S) out[(long long)j * S + k] = pixel_gain_rt<SPK>(p, gk, k, t0, postc, SPK ? s_xig[i] : 1.0f, s_xir);
    }
}

inline int grid_for(long long n, int block)
{
    long long g = (n + block - 1) / block;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (int)g;
}

// adjoint blocks for n rays of w wavefronts each, and how many consecutive
// blocks keep `rays` consecutive rays on one XCD
inline int ray_blocks(int w, int n) { return w == 1 ? (n + kBlockRays - 1) / kBlockRays : n; }
inline int block_group(int w, int rays) { return w == 1 ? std::max(rays / kBlockRays, 1) : rays; }

// the side stream starts after what st has queued; st waits for it at the
// join (graph capture turns both into graph edges)
inline hipError_t fork_side(hipStream_t st, const SideStream &s)
{
    hipError_t e = hipEventRecord(s.fork, st);
    if (e == hipSuccess) e = hipStreamWaitEvent(s.st, s.fork, 0);
    return e;
}

inline hipError_t join_side(hipStream_t st, const SideStream &s)
{
    hipError_t e = hipEventRecord(s.join, s.st);
    if (e == hipSuccess) e = hipStreamWaitEvent(st, s.join, 0);
    return e;
}

}  // namespace

// --------------------------------------------------------------------------
// launch wrappers
// --------------------------------------------------------------------------
// the instance that also reports the smallest pivots is one of its own (the
// others carry no test for it)
#define DUS_FWD_LAUNCH_(CH, SPK, WV, PIV, NG, TAB, ZERO, STR)                                   \
    hipLaunchKernelGGL((k_forward<CH, SPK, WV, PIV>), dim3(NG), dim3(64 * WV), 0, STR, v, p, TAB, poses, out, \
                       min_pivot, pivot_base, zcar, reinterpret_cast<float *>(states), gain, xcd_group, ZERO)
#define DUS_FWD_LAUNCH(CH, SPK, WV, NG, TAB, ZERO, STR)                                         \
    do {                                                                                        \
        if (min_pivot) DUS_FWD_LAUNCH_(CH, SPK, WV, true, NG, TAB, ZERO, STR);                   \
        else DUS_FWD_LAUNCH_(CH, SPK, WV, false, NG, TAB, ZERO, STR);                            \
    } while (0)

#define DUS_FWD_LONG(CH, WV, NG, ZERO)                                                          \
    do {                                                                                        \
        if (p.speckle) DUS_FWD_LAUNCH(CH, true, WV, NG, t, ZERO, sst);                          \
        else DUS_FWD_LAUNCH(CH, false, WV, NG, t, ZERO, sst);                                   \
    } while (0)

// few rays (chunk 4 and 8: split_rays gives none past kFewFwdChunk)
#define DUS_FWD_FEW(CH)                                                                        \
    if (r.few == 2) DUS_FWD_LONG(CH, 2, t.total_rays, zero);                                   \
    else if (r.few == 4) DUS_FWD_LONG(CH, 4, t.total_rays, zero);                              \
    else if (r.few == 8) DUS_FWD_LONG(CH, 8, t.total_rays, zero);                              \
    if (r.few) break;

#define DUS_FWD_SPLIT(CH)                                                                      \
    if (r.n_span > 0) DUS_FWD_LONG(CH, kSpanWaves, r.n_span, r.n_one > 0 ? ZeroArgs{} : zero); \
    if (r.n_one > 0) {                                                                         \
        if (p.speckle) DUS_FWD_LAUNCH(CH, true, 1, t.total_rays, t1, zero, st);                \
        else DUS_FWD_LAUNCH(CH, false, 1, t.total_rays, t1, zero, st);                         \
    }                                                                                          \
    break;

// automatic forward tile (chunk 0): 8 x 64 samples, unless the table's rays
// fill 512-sample tiles clearly worse than 256-sample ones.  On full tiles
// the 4 x 64 tile costs 20% more per sample (64 poses x 256 x 1024: 141
// against 118 us), so the uneven batch of 64 fans of up to 512 x 2048, whose
// rays pad to 1.1 times as many samples in the longer tiles, is still faster
// in those (163 against 189 us); rays of 600 samples pad to 1.33 times.
// Few rays that share out their tiles take the shorter ones as long as one
// round of eight holds the ray at least twice over (256 x 1024: 13.6 -> 12.6
// us; 384 x 1500 in eight 4 x 64 tiles against four of 8 x 64: 20.0 / 16.9).
// A plan's forward (step) keeps to the line of 7% and to its own tile for few
// rays: the last place of a pixel next to a pole depends on the tile, one
// such pixel can hold most of an FP64 loss (seen to move it by 2e-7), and the
// step gains 1% at most.
static int auto_fwd_chunk(const FanTable &t, int span_samples, bool step)
{
    if (!step && longest_ray(t) <= 1024 && few_ray_waves(t, 256, span_samples)) return 4;
    long long pad4 = 0, pad8 = 0;
    for (int f = 0; f < t.n; ++f) {
        const long long r = t.f[f].n_rays, s = t.f[f].n_samples;
        pad4 += r * ((s + 255) / 256) * 256;
        pad8 += r * ((s + 511) / 512) * 512;
    }
    return (pad8 * 100 > pad4 * (step ? 107 : 120)) ? 4 : 8;
}

hipError_t launch_forward(int chunk, int xcd_group, const VolArgs &v, const PhysArgs &p,
                          const FanTable &t, const float *poses, float *out, float *min_pivot,
                          int pivot_base, double *zcar, int32_t *, double *states, float *gain,
                          hipStream_t st, const ZeroArgs &zero, int span_samples, const SideStream *side)
{
    if (t.total_rays <= 0) return hipSuccess;
    if (chunk == 0) chunk = auto_fwd_chunk(t, span_samples, zcar != nullptr);
    if (chunk != 4 && chunk != 8 && chunk != 16) return hipErrorInvalidValue;
    const RaySplit r = split_rays(t, chunk, kFewFwdChunk, span_samples);
    // the clears go with the one-wavefront launch where there is one
    FanTable t1 = t;
    t1.ray0 = r.n_span;
    hipStream_t sst = st;
    if (r.both() && side) {
        hipError_t e = fork_side(st, *side);
        if (e != hipSuccess) return e;
        sst = side->st;
    }
    switch (chunk) {
    case 4:
        DUS_FWD_FEW(4)
        DUS_FWD_SPLIT(4)
    case 8:
        DUS_FWD_FEW(8)
        DUS_FWD_SPLIT(8)
    case 16:
        DUS_FWD_SPLIT(16)
    default:
        return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (sst != st) {
        // joined also after a failed launch: a capture must not end with a
        // fork left open, and the caller's stream must wait for the side's work
        const hipError_t ej = join_side(st, *side);
        if (e == hipSuccess) e = ej;
    }
    return e;
}

#define DUS_BWD_LAUNCH(CH, SPK, FUSED, WV, FROM, NG, TAB, STR) DUS_BWD_LAUNCH_(CH, SPK, FUSED, WV, FROM, false, NG, TAB, STR)
#define DUS_BWD_LAUNCH_(CH, SPK, FUSED, WV, FROM, NEAR, NG, TAB, STR)                             \
    hipLaunchKernelGGL((k_backward<CH, SPK, FUSED, WV, FROM, NEAR>), dim3(ray_blocks(WV, NG)), dim3(64 * adjoint_waves(WV)), \
                       0, STR, v, p, TAB, poses, zbar ? rays : nullptr, gsrc, target, zbar, pose_acc ? pose_part : nullptr, \
                       loss, zcar, reinterpret_cast<const float *>(states), t.geom, gain, block_group(WV, xcd_group))

// from the forward's records: the long rays (the table's first n_span) take
// kSpanWaves * 4 / C wavefronts each (the registers of C = 8 allow half as many)
#define DUS_BWD_CASE(CH)                                                                       \
    case CH:                                                                                   \
        if (r.n_span > 0) {                                                                      \
            if (fused) DUS_BWD_LAUNCH(CH, false, true, kSpanWaves * 4 / CH, kRecords, r.n_span, t, sst);  \
            else if (spk) DUS_BWD_LAUNCH(CH, true, false, kSpanWaves * 4 / CH, kRows, r.n_span, t, sst); \
            else if (!zcar) DUS_BWD_LAUNCH(CH, false, false, kSpanWaves * 4 / CH, kRows, r.n_span, t, sst); \
            else DUS_BWD_LAUNCH(CH, false, false, kSpanWaves * 4 / CH, kRecords, r.n_span, t, sst);       \
        }                                                                                      \
        if (r.n_one > 0) {                                                                       \
            if (fused && in_reach(v)) DUS_BWD_LAUNCH_(CH, false, true, 1, kRecords, true, t.total_rays, t1, st); \
            else if (fused) DUS_BWD_LAUNCH(CH, false, true, 1, kRecords, t.total_rays, t1, st);         \
            else if (spk) DUS_BWD_LAUNCH(CH, true, false, 1, kRows, t.total_rays, t1, st);            \
            else if (!zcar) DUS_BWD_LAUNCH(CH, false, false, 1, kRows, t.total_rays, t1, st); \
            else if (in_reach(v)) DUS_BWD_LAUNCH_(CH, false, false, 1, kRecords, true, t.total_rays, t1, st); \
            else DUS_BWD_LAUNCH(CH, false, false, 1, kRecords, t.total_rays, t1, st);                    \
        }                                                                                      \
        break;

// from the records, few rays
#define DUS_FEW_CASE(WV)                                                                       \
    case WV:                                                                                   \
        if (fused) DUS_BWD_LAUNCH(4, false, true, WV, kRecords, t.total_rays, t, st);           \
        else DUS_BWD_LAUNCH(4, false, false, WV, kRecords, t.total_rays, t, st);               \
        break;

// without records (rays of at most kWholeSamples): W wavefronts per ray, one
// per 256 samples
#define DUS_WHOLE_CASE(WV)                                                                     \
    case WV:                                                                                   \
        if (fused) {                                                                           \
            if (spk) DUS_BWD_LAUNCH(4, true, true, WV, kWholeRay, n, t1, st);                              \
            else DUS_BWD_LAUNCH(4, false, true, WV, kWholeRay, n, t1, st);                                 \
        } else {                                                                               \
            if (spk) DUS_BWD_LAUNCH(4, true, false, WV, kWholeRay, n, t1, st);                             \
            else DUS_BWD_LAUNCH(4, false, false, WV, kWholeRay, n, t1, st);                                \
        }                                                                                      \
        break;

hipError_t launch_adjoint(int chunk, int xcd_group, const VolArgs &v, const PhysArgs &p,
                          const FanTable &t, const float *poses, RayRec *rays, const float *gsrc,
                          const float *target, float *zbar, double *pose_acc, double *pose_part, double *loss,
                          const double *zcar, const int32_t *, const double *states,
                          const float *gain, hipStream_t st, int span_samples, const SideStream *side)
{
    if (t.total_rays <= 0) return hipSuccess;
    if (pose_acc && !pose_part) return hipErrorInvalidValue;
    if (zbar && !rays) return hipErrorInvalidValue;
    if (chunk != 4 && chunk != 8) return hipErrorInvalidValue;
    const bool fused = (target != nullptr);
    const bool spk = p.speckle && !gain;      // recorded gains replace the speckle variates
    FanTable t1 = t;
    if (!states) {
        if (longest_ray(t) > kWholeSamples) return hipErrorInvalidValue;
        // fans of one wavefront count after the other (a table lists its fans
        // longest first)
        for (int f = 0; f < t.n;) {
            int w = 1, n = 0;
            while (w * kCarryBlock < t.f[f].n_samples) w *= 2;
            t1.ray0 = t.f[f].ray_begin;
            for (; f < t.n && (w == 1 || 2 * t.f[f].n_samples > w * kCarryBlock); ++f) n += t.f[f].n_rays;
            if (n <= 0) continue;
            t1.ray1 = t1.ray0 + n;
            switch (w) {
                DUS_WHOLE_CASE(1)
                DUS_WHOLE_CASE(2)
                DUS_WHOLE_CASE(4)
                DUS_WHOLE_CASE(8)
            }
        }
        return hipGetLastError();
    }
    // the fused step records its gains and the rays' geometry
    if ((fused && (spk || !zcar)) || (spk && zcar) || (zcar && !t.geom)) return hipErrorInvalidValue;
    // several wavefronts per long ray, or for every ray where they are few
    const RaySplit r = split_rays(t, zcar ? chunk : kFewBwdChunk + 1, kFewBwdChunk, span_samples);
    if (r.few) {
        switch (r.few) {
            DUS_FEW_CASE(2)
            DUS_FEW_CASE(4)
            DUS_FEW_CASE(8)
        }
        return hipGetLastError();
    }
    t1.ray0 = r.n_span;
    hipStream_t sst = st;
    if (r.both() && side) {
        hipError_t e = fork_side(st, *side);
        if (e != hipSuccess) return e;
        sst = side->st;
    }
    switch (chunk) {
        DUS_BWD_CASE(4)
        DUS_BWD_CASE(8)
    default:
        return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (sst != st) {
        // joined also after a failed launch: a capture must not end with a
        // fork left open, and the caller's stream must wait for the side's work
        const hipError_t ej = join_side(st, *side);
        if (e == hipSuccess) e = ej;
    }
    return e;
}

hipError_t launch_pose_reduce(const FanTable &t, const double *pose_part, double *pose_acc, hipStream_t st)
{
    if (t.n <= 0 || t.total_rays <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pose_reduce, dim3(t.n + (t.loss ? 1 : 0)), dim3(256), 0, st, t, pose_part, pose_acc);
    return hipGetLastError();
}

// Whether most of a table's samples lie in fans whose scatter does better with
// boxes of sixteen rays and half the depths: fewer voxels are flushed twice.
// At least 128 rays, at most 0.65 voxels apart at mid-depth, and steps of at
// least 0.22 voxels, since shorter ones leave a group of sixteen depths a few
// cells (eight rays / sixteen, us: 64 poses x 256 x 1024 at 0.25 voxels 140 /
// 126, 56 x 432 x 72 at 1.7 70 / 45, 43 x 181 x 108 at 0.5 28 / 23; 64 x 256 x 512
// at 0.2 69 / 84, 64 x 512 x 2048 uneven at 0.12 155 / 185; rays a voxel
// apart, 61 x 72 x 213, 34 / 41).
static bool dense_fans(const VolArgs &v, const FanTable &t)
{
    const float h = std::min(v.h[0], std::min(v.h[1], v.h[2]));
    long long all = 0, dense = 0;
    for (int f = 0; f < t.n; ++f) {
        const FanRec &r = t.f[f];
        const long long n = (long long)r.n_rays * r.n_samples;
        const float mid = r.r0 + 0.5f * r.ds * (float)r.n_samples;
        all += n;
        if (r.n_rays >= 128 && r.ds >= 0.22f * h && r.aperture * mid <= 0.65f * h * (float)r.n_rays) dense += n;
    }
    return 2 * dense > all;
}

// Whether most of a table's samples lie in fans of few rays, or of rays more
// than two voxels apart at mid-depth
static bool sparse_fans(const VolArgs &v, const FanTable &t)
{
    const float h = std::min(v.h[0], std::min(v.h[1], v.h[2]));
    long long all = 0, sparse = 0;
    for (int f = 0; f < t.n; ++f) {
        const FanRec &r = t.f[f];
        const long long n = (long long)r.n_rays * r.n_samples;
        const float mid = r.r0 + 0.5f * r.ds * (float)r.n_samples;
        all += n;
        if (r.n_rays < 8 || r.aperture * mid > 2.0f * h * (float)r.n_rays) sparse += n;
    }
    return 2 * sparse > all;
}

// the most depths that a lane takes in any fan (k_scatter's rule, by the step
// along the widest spacing)
static int depths_per_lane(const VolArgs &v, const FanTable &t)
{
    const float h = std::max(v.h[0], std::max(v.h[1], v.h[2]));
    float ds = t.f[0].ds;
    for (int f = 1; f < t.n; ++f) ds = std::min(ds, t.f[f].ds);
    return ds <= 0.35f * h ? 4 : (ds <= 0.7f * h ? 2 : 1);
}

// whether some ray is longer than the volume's diagonal
static bool runs_outside(const VolArgs &v, const FanTable &t)
{
    const float x = v.h[0] * (float)v.nx, y = v.h[1] * (float)v.ny, z = v.h[2] * (float)v.nz;
    const float diag = sqrtf(x * x + y * y + z * z);
    for (int f = 0; f < t.n; ++f)
        if (t.f[f].r0 + t.f[f].ds * (float)t.f[f].n_samples > diag) return true;
    return false;
}

hipError_t launch_scatter(int scatter_rays, int xcd_group, const VolArgs &v, const FanTable &t,
                          const RayRec *rays, const float *zbar, float *gZ, hipStream_t st,
                          unsigned long long *fix, const double *fscale, int wave_target)
{
    if (t.total_rays <= 0 || (!gZ && !fix)) return hipSuccess;
    if (!zbar || !rays || (fix && !fscale)) return hipErrorInvalidValue;
    // depth segments, the same power-of-two length for every fan, a whole
    // number of the largest groups (256 / RB depths, or in a small launch
    // those of its shortest steps, so that no wavefront walks several groups
    // while others are missing: 140 sparse fans 1.36 times as fast): the shortest that
    // keeps the launch within wave_target wavefronts, about 32 per SIMD over
    // the launches that run at the same time (a wavefront's set-up is a few
    // loads, so short segments cost little and even out the finishing times;
    // a fan of long rays gets as many wavefronts per ray as its length asks
    // for)
    auto units = [&](int rb, int sg) {
        long long u = 0;
        for (int f = 0; f < t.n; ++f)
            u += (long long)((t.f[f].n_rays + rb - 1) / rb) * ((t.f[f].n_samples + sg - 1) / sg);
        return u;
    };
    // 0: sixteen rays per wavefront where most samples lie in dense fans (above);
    // two where few rays run on outside the volume: their samples there meet in
    // few voxels, and groups of four times the depths add to them a quarter as
    // often (35 x 607, 22 x 1297 and 7 x 1434 rays of up to 1600 mm past a volume
    // of 39 mm: largest error 1e-6 of the largest voxel, 3e-6 with eight); else
    // eight, also where that leaves few wavefronts: a
    // box of two rays and four times the depths is longer than LDS holds, and
    // the cells where the rays meet take four times the global atomics (two
    // rays / eight, us: 2 poses x 46 x 224 24 / 16, 9 x 93 x 142 50 / 23, 23 x 77
    // x 142 72 / 12, 6 x 488 x 90 150 / 27); or four where those wavefronts' rays
    // are few or far apart and would be taken in quarters and singly (direct
    // adjoint, two rays / eight / four, us: 1 pose x 8 x 150 9 voxels apart 33 / 44
    // / 24, 4 x 13 x 105 at 7 36 / 46 / 29, 2 x 14 x 161 at 7 35 / 45 / 34; over
    // 140 fans of 2 to 64 rays four are 11% faster than eight in the mean).
    // Over 310 small launches dL/dZ is 0.90 (few rays 0.98, rays running on
    // outside 0.95) times as far from 64 bits, rel. l2, as with two throughout.
    const bool few = units(8, 32) < 2048;
    if (scatter_rays == 0)
        scatter_rays = (few && runs_outside(v, t)) ? 2 : (dense_fans(v, t) ? 16 : (few && sparse_fans(v, t) ? 4 : 8));
    else if (scatter_rays == 16) return hipErrorInvalidValue;
    int seg = 64 * (few ? depths_per_lane(v, t) : kScatterSpl) / scatter_rays, seg_shift = 0;
    while (seg < DUS_MAX_SAMPLES && units(scatter_rays, seg) > std::max(wave_target, 1024)) seg *= 2;
    while ((1 << seg_shift) < seg) ++seg_shift;
    const long long nunits = units(scatter_rays, seg);
    if (nunits <= 0) return hipSuccess;
    if (nunits > INT32_MAX) return hipErrorInvalidValue;
    // fans of different lengths run faster segment by segment (a 2-D grid,
    // uneven 64-pose batch: 188 -> 178 us) unless most of that grid would be
    // empty blocks (a few very long fans: 1-D); equal fans run faster fan by
    // fan (bench step 144 -> 137 us)
    long long nrb_all = 0;
    int smax = 0;
    for (int f = 0; f < t.n; ++f) {
        nrb_all += (t.f[f].n_rays + scatter_rays - 1) / scatter_rays;
        smax = std::max(smax, t.f[f].n_samples);
    }
    const long long nseg_max = (smax + seg - 1) / seg;
    const long long grid2 = nrb_all * nseg_max;
    const bool two_d = grid2 > nunits && grid2 <= 2 * nunits;
    const dim3 grid = two_d ? dim3((unsigned)nrb_all, (unsigned)nseg_max) : dim3((unsigned)nunits);
    // each fan's first wavefront (along x for the 2-D grid)
    FanTable ts = t;
    long long u = 0;
    for (int f = 0; f < t.n; ++f) {
        ts.f[f].unit_begin = (int32_t)u;
        const long long nrb = (t.f[f].n_rays + scatter_rays - 1) / scatter_rays;
        u += two_d ? nrb : nrb * ((t.f[f].n_samples + seg - 1) / seg);
    }
    switch (scatter_rays) {
    case 2:
        hipLaunchKernelGGL((k_scatter<2>), grid, dim3(64), 0, st, v, ts, rays, zbar, gZ, seg_shift, few, xcd_group,
                           fix, fscale);
        break;
    case 4:
        hipLaunchKernelGGL((k_scatter<4>), grid, dim3(64), 0, st, v, ts, rays, zbar, gZ, seg_shift, few, xcd_group,
                           fix, fscale);
        break;
    case 8:
        hipLaunchKernelGGL((k_scatter<8>), grid, dim3(64), 0, st, v, ts, rays, zbar, gZ, seg_shift, few, xcd_group,
                           fix, fscale);
        break;
    case 16:
        hipLaunchKernelGGL((k_scatter<16>), grid, dim3(64), 0, st, v, ts, rays, zbar, gZ, seg_shift, few, xcd_group,
                           fix, fscale);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

#define DUS_BLUR_LAUNCH(MODE, TGT, IMG, LOSS)                                                       \
    do {                                                                                           \
        if (R <= 4)                                                                                \
            hipLaunchKernelGGL((k_blur<MODE, 4>), dim3(grid), dim3(256), 0, st, p, t, in, TGT, out, IMG, LOSS);  \
        else if (R <= 8)                                                                           \
            hipLaunchKernelGGL((k_blur<MODE, 8>), dim3(grid), dim3(256), 0, st, p, t, in, TGT, out, IMG, LOSS);  \
        else if (R <= 16)                                                                          \
            hipLaunchKernelGGL((k_blur<MODE, 16>), dim3(grid), dim3(256), 0, st, p, t, in, TGT, out, IMG, LOSS); \
        else                                                                                       \
            hipLaunchKernelGGL((k_blur<MODE, 32>), dim3(grid), dim3(256), 0, st, p, t, in, TGT, out, IMG, LOSS); \
    } while (0)

hipError_t launch_blur(bool transpose, const PhysArgs &p, const FanTable &t, const float *in,
                       float *out, hipStream_t st)
{
    const int grid = t.total_blur_blocks;
    if (grid <= 0) return hipSuccess;
    const int R = p.blur_rmax;
    if (R > DUS_MAX_BLUR_RADIUS) return hipErrorInvalidValue;
    if (transpose)
        DUS_BLUR_LAUNCH(1, nullptr, nullptr, nullptr);
    else
        DUS_BLUR_LAUNCH(0, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_blur_residual(const PhysArgs &p, const FanTable &t, const float *pre,
                                const float *target, float *image, float *resid, float *ebar,
                                double *loss, hipStream_t st)
{
    const int grid = t.total_blur_blocks;
    if (grid <= 0) return hipSuccess;
    const int R = p.blur_rmax;
    if (R > DUS_MAX_BLUR_RADIUS) return hipErrorInvalidValue;
    // radius up to 8: one pass, the residual kept in LDS
    if (R <= 4) {
        hipLaunchKernelGGL((k_blur_fused<4>), dim3(grid), dim3(256), 0, st, p, t, pre, target, ebar, image, loss);
        return hipGetLastError();
    }
    if (R <= 8) {
        hipLaunchKernelGGL((k_blur_fused<8>), dim3(grid), dim3(256), 0, st, p, t, pre, target, ebar, image, loss);
        return hipGetLastError();
    }
    if (!resid) return hipErrorInvalidValue;
    {
        const float *in = pre;
        float *out = resid;
        DUS_BLUR_LAUNCH(2, target, image, loss);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_blur(true, p, t, resid, ebar, st);
}

// --------------------------------------------------------------------------
// Static device scratch of the allocation-free entry points.  The array is
// part of the code object: every GPU that loads the library holds its own
// copy, at its own address, until the process ends.  In host code its name
// stands for the host-side shadow, not for device memory, so the device
// address is looked up once per device (with that device current) and only
// that address is handed to kernels.
// --------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(void **ptr)
{
    *ptr = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_pose_finalize(const double *acc, const float *poses, int n_poses,
                                float *grad_pose, hipStream_t st)
{
    if (n_poses <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pose_finalize, dim3((6 * n_poses + 191) / 192), dim3(192), 0, st, acc, poses,
                       n_poses, grad_pose);
    return hipGetLastError();
}

hipError_t launch_sample(int xcd_group, const VolArgs &v, const FanTable &t, const float *poses, float *out,
                         hipStream_t st)
{
    if (t.total_rays <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sample_rays, dim3(t.total_rays), dim3(64), 0, st, v, t, poses, out, xcd_group);
    return hipGetLastError();
}

hipError_t launch_scan_convert(const float *img, int n_rays, int n_samples, double aperture, double r0,
                               double ds, int nx, int nz, double x0, double z0, double dx, double dz,
                               float fill, float *out, hipStream_t st)
{
    const long long n = (long long)nx * nz;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scan_convert, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, img, n_rays,
                       n_samples, aperture, r0, ds, nx, nz, x0, z0, dx, dz, fill, out);
    return hipGetLastError();
}

hipError_t launch_footprint(const VolArgs &v, const FanTable &t, const float *poses, uint8_t *mask,
                            hipStream_t st)
{
    if (t.total_rays <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_footprint, dim3(t.total_rays), dim3(64), 0, st, v, t, poses, mask);
    return hipGetLastError();
}

hipError_t launch_zero_f64(double *ptr, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_f64, dim3(grid_for(n, 256)), dim3(256), 0, st, ptr, (long long)n);
    return hipGetLastError();
}

hipError_t launch_zero_f32(float *ptr, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_f32, dim3(grid_for((n + 3) / 4, 256)), dim3(256), 0, st, ptr,
                       (long long)n);
    return hipGetLastError();
}

hipError_t launch_finish(const double *part, int64_t n_part, double *loss, const double *acc, const float *poses,
                         int n_poses, float *grad, hipStream_t st)
{
    const int pose_blocks = grad ? (6 * n_poses + kSumThreads - 1) / kSumThreads : 0;
    const int grid = (loss ? 1 : 0) + pose_blocks;
    if (grid == 0) return hipSuccess;
    hipLaunchKernelGGL(k_finish, dim3(grid), dim3(kSumThreads), 0, st, part, (long long)n_part, loss, acc, poses, n_poses,
                       grad);
    return hipGetLastError();
}

hipError_t launch_abs_rows(const FanTable &t, const float *zbar, double *part, hipStream_t st)
{
    if (t.total_rays <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_abs_rows, dim3((t.total_rays + 3) / 4), dim3(256), 0, st, t, zbar, part);
    return hipGetLastError();
}

hipError_t launch_fix_scale(const double *part, int64_t n, double *fscale, hipStream_t st)
{
    hipLaunchKernelGGL(k_fix_scale, dim3(1), dim3(kSumThreads), 0, st, part, (long long)n, fscale);
    return hipGetLastError();
}

hipError_t launch_fix_to_f32(const unsigned long long *fix, int64_t n, const double *fscale, float *gZ,
                             bool overwrite, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fix_to_f32, dim3(grid_for((n + 3) / 4, 256)), dim3(256), 0, st, fix, (long long)n, fscale,
                       gZ, overwrite ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_zero_pair(float *a, int64_t na, double *b, int64_t nb, hipStream_t st)
{
    if (na <= 0 && nb <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_pair, dim3(grid_for(std::max<int64_t>((na + 3) / 4, nb), 256)), dim3(256), 0, st, a,
                       (long long)na, b, (long long)nb);
    return hipGetLastError();
}

hipError_t launch_sum_f64(const double *part, int64_t n, double *out, hipStream_t st, bool accumulate)
{
    hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(kSumThreads), 0, st, part, (long long)n, out, accumulate ? 1 : 0);
    return hipGetLastError();
}

int64_t smooth_blocks(int nx, int ny, int nz) { return ((int64_t)nx * ny * nz + kSmoothVoxels - 1) / kSmoothVoxels; }

hipError_t launch_smooth(const float *Z, int nx, int ny, int nz, float wx, float wy, float wz, float *gZ,
                         double *part, hipStream_t st)
{
    const int64_t blocks = smooth_blocks(nx, ny, nz);
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_smooth, dim3((unsigned)blocks), dim3(256), 0, st, Z, nx, ny, nz, wx, wy, wz, gZ, part);
    return hipGetLastError();
}

hipError_t launch_adam(float *x, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, float lo, float hi, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n, 256)), dim3(256), 0, st, x, g, m, v, (long long)n, lr, b1, b2,
                       eps, c1, c2, lo, hi);
    return hipGetLastError();
}

// the table with its inner knots padded for the scan
static bool scan_table(const LutArgs &lut, LutArgs &t)
{
    t = lut;
    t.x0 = lut.x[0];
    t.xn = lut.x[lut.n - 1];
    if (lut.n > kScanKnots) return false;
    for (int k = lut.n; k < kScanKnots; ++k) t.x[k] = INFINITY;
    return true;
}

// blocks of 1024 voxels a pass, at most 16 per CU
static int map_grid(int64_t n) { return (int)std::min<int64_t>((n + 1023) / 1024, 4096); }

hipError_t launch_map(const float *in, int64_t n, const LutArgs &lut, float *Z, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    LutArgs t;
    if (scan_table(lut, t)) hipLaunchKernelGGL(k_map<true>, dim3(map_grid(n)), dim3(256), 0, st, in, (long long)n, t, Z);
    else hipLaunchKernelGGL(k_map<false>, dim3(map_grid(n)), dim3(256), 0, st, in, (long long)n, t, Z);
    return hipGetLastError();
}

hipError_t launch_map_backward(const float *in, int64_t n, const LutArgs &lut, const float *gZ, float *grad_in,
                               double *grad_z, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((n + 4 * kMapThreads - 1) / (4 * kMapThreads), 512);
    LutArgs t;
    if (scan_table(lut, t))
        hipLaunchKernelGGL(k_map_backward<true>, dim3(grid), dim3(kMapThreads), 0, st, in, (long long)n, t, gZ, grad_in,
                           grad_z);
    else
        hipLaunchKernelGGL(k_map_backward<false>, dim3(grid), dim3(kMapThreads), 0, st, in, (long long)n, t, gZ, grad_in,
                           grad_z);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr, int64_t n, uint32_t k0, uint32_t k1, uint32_t *out,
                         hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const long long g = (n + 255) / 256;
    if (g > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_philox, dim3((unsigned)g), dim3(256), 0, st, ctr, (long long)n, k0, k1,
                       out);
    return hipGetLastError();
}

hipError_t launch_pixel_gain(const PhysArgs &p, const FanRec &f, float *out, hipStream_t st)
{
    if (f.n_rays <= 0 || f.n_samples <= 0) return hipSuccess;
    dim3 grid((f.n_samples + 255) / 256, f.n_rays);
    if (p.speckle)
        hipLaunchKernelGGL((k_gain<true>), grid, dim3(64), 0, st, p, f, out);
    else
        hipLaunchKernelGGL((k_gain<false>), grid, dim3(64), 0, st, p, f, out);
    return hipGetLastError();
}

}  // namespace dus
