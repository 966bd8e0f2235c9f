// Internal launch records shared by the HIP kernels and the host ABI layer.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace dus {

// Fans per launch: the fan table travels in the kernel arguments.
constexpr int kMaxFans = 64;
// rays of at least span_samples samples (kSpanSamples by default; <= 0:
// none) are walked by kSpanWaves wavefronts each, which take consecutive
// tiles of the ray together (forward and plan adjoint); shorter rays by one
// wavefront.  At the default also shorter rays take several where a launch
// has few (few_ray_waves), and long ones one where there are many (span_rays)
constexpr int kSpanSamples = 4096;
constexpr int kSpanWaves = 8;

struct FanRec {
    int32_t n_rays, n_samples;
    float aperture, ds, r0;
    int32_t speckle_id;
    int64_t out_offset;     // element offset of the [n_rays][n_samples] image
    int32_t ray_begin;      // first launch-wide ray index of this fan
    int32_t blk_begin;      // first blur block of this fan
    int32_t pose;           // row of the poses array
    int32_t pivot_begin;    // pose-major index of this fan's first ray
    int32_t carry_begin;    // first tile-carry record of this fan's first ray
    int32_t unit_begin;     // first wavefront of this fan in a scatter launch (set by launch_scatter)
};
static_assert(sizeof(FanRec) == 56, "FanRec layout");

// What the forward kernel records for the adjoint, per carry block of 256
// samples of a ray: the sample before the block, and the state
// (w, t) = (v0 / v1, D / v1^2) at every 4th sample, two doubles side by side.
constexpr int kCarryBlock = 256;
inline int64_t carry_records(int32_t n_rays, int32_t n_samples)
{
    return (int64_t)n_rays * ((n_samples + kCarryBlock - 1) / kCarryBlock);
}
constexpr int kStateStride = 4;
constexpr int kStateFloats = kCarryBlock / kStateStride * 4;     // in units of 4 bytes
// rays of at most this many samples need no records: the adjoint gathers
// them once, one wavefront per 256 samples
constexpr int kWholeSamples = 8 * kCarryBlock;

// A ray's geometry, written by the adjoint kernel (which sets it up from the
// pose and the fan) for the dL/dZ scatter: sample k sits at voxel coordinate
// u0 + k du.
struct RayRec {
    double u0[3], du[3];
};
static_assert(sizeof(RayRec) == 48, "RayRec layout");

// A ray's geometry as the fused step's forward sets it up, read by its
// adjoint: sample k sits at voxel coordinate u0 + k du; round-trip amplitude
// a2 over one step; the probe-frame direction (dirx, 0, dirz); the ray's
// orthonormal basis in the world, over the voxel spacing.
struct RayGeom {
    double u0[3], du[3], bd[3], bt[3], bn[3], a2, dirx, dirz;
};
static_assert(sizeof(RayGeom) == 144, "RayGeom layout");

struct FanTable {
    int32_t n;              // fans in this launch
    int32_t total_rays;
    int32_t total_blur_blocks;
    int32_t ray0;           // forward and adjoint, one wavefront per ray: rays below ray0 are
                            // another launch's (their wavefronts return at once)
    int32_t ray1;           // adjoint without records: the launch's rays are [ray0, ray1)
    RayGeom *geom;          // forward: if not NULL, where to record the rays' geometry; adjoint with
                            // the forward's records: where to find it (else set up again)
    const float *poses;     // pose sums: with grad_pose, the poses, and where the gradients of the
    float *grad_pose;       // table's poses go (NULL: into the accumulators)
    const double *loss_part;    // pose sums: with loss, one more block writes there the sum of the n_part
    double *loss;               // partials at loss_part
    int32_t n_part;
    FanRec f[kMaxFans];
};

inline int longest_ray(const FanTable &t)
{
    int s = 0;
    for (int f = 0; f < t.n; ++f)
        if (t.f[f].n_samples > s) s = t.f[f].n_samples;
    return s;
}

// Rays of the fans at the front of a table whose rays are walked by
// kSpanWaves wavefronts each (a table lists its fans longest first).  At the
// default length only up to 512 of them: more fill the chip with one
// wavefront each (direct adjoint and forward, kSpanWaves / one, us: 512 x 5000
// 67 + 30 / 80 + 34, 1024 x 5000 132 + 58 / 92 + 36, 3072 x 5000 391 + 187 / 158
// + 64).
constexpr int kSpanRays = 512;
inline int span_rays(const FanTable &t, int span_samples)
{
    int n = 0;
    if (span_samples <= 0) return 0;
    for (int f = 0; f < t.n && t.f[f].n_samples >= span_samples; ++f) n += t.f[f].n_rays;
    return (span_samples == kSpanSamples && n > kSpanRays) ? 0 : n;
}

// Wavefronts per ray (2, 4 or 8: one per tile of the longest ray, as far as
// they go) where a launch's rays are too few to fill the chip by themselves;
// 0: the usual split.  A launch of few rays takes as long as its longest ray's
// chain of tiles, which the wavefronts share: forward (with blur) and
// pose-only step with one wavefront a ray against several, us:
//   64 x 300    11.7 ->  11.0    34.3 -> 31.1
//   256 x 1024  16.2 ->  12.6    42.4 -> 32.9
//   512 x 1024  17.6 ->  14.8    44.4 -> 36.8
//   64 x 2048   24.2 ->  13.5    59.8 -> 34.8
//   512 x 2048  27.5 ->  18.1    65.7 -> 49.4
//   512 x 3000  39.3 ->  31.6    89.4 -> 72.9
// The line is where the wavefronts, idle ones included, begin to cost more
// than the shorter chain saves: 2048 of them, 4096 for rays over 1024
// samples.  Past it: 1024 x 520 in four wavefronts (4096) 45.8 -> 48.1 and
// 2048 x 300 in two 49.5 -> 54.5 (pose-only step); 1024 x 1500 in eight
// (8192) 63.7 -> 75.1, against 64.6 where only its forward takes four.
// Results are the same but for the order of the pose gradient's and the
// fused loss's sums, as with the long rays' wavefronts; a schedule that sets
// another span length than the default keeps to what it says.
inline int few_ray_waves(const FanTable &t, int tile, int span_samples)
{
    if (span_samples != kSpanSamples) return 0;
    const int s = longest_ray(t);
    int w = 1;
    while (w < 8 && w * tile < s) w *= 2;
    return (w > 1 && (long long)t.total_rays * w <= (s > 1024 ? 4096 : 2048)) ? w : 0;
}

// How a launch with tiles of 64 * chunk samples walks a table's rays: all of
// them by `few` wavefronts each (up to chunk `most`, whose registers allow
// it), or else the first n_span (a table lists its fans longest first) by
// kSpanWaves each and the n_one others by one.  With both, the n_span may take
// the side stream; a plan asks the same question to lay out its streams.
struct RaySplit {
    int few, n_span, n_one;
    bool both() const { return n_span > 0 && n_one > 0; }
};

inline RaySplit split_rays(const FanTable &t, int chunk, int most, int span_samples)
{
    RaySplit r;
    r.few = chunk <= most ? few_ray_waves(t, 64 * chunk, span_samples) : 0;
    r.n_span = r.few ? 0 : span_rays(t, span_samples);
    r.n_one = t.total_rays - r.n_span;
    return r;
}
constexpr int kFewFwdChunk = 8, kFewBwdChunk = 4;

struct VolArgs {
    const float *Z;
    int32_t nx, ny, nz, pad_;
    float h[3];
    float o[3];
};

struct PhysArgs {
    float alpha, freq;
    int32_t refl, atten;
    int32_t speckle, cell;
    float Ar, gam, Ag0, Ag1;
    int32_t blur;
    float s0, s1;
    uint32_t key0, key1;
    int32_t blur_rmax;      // ceil(3 * max sigma), <= DUS_MAX_BLUR_RADIUS
};

// Per-pose accumulator of the adjoint: dL/dt (3) and dL/dR (9), FP64.
constexpr int kPoseAcc = 12;
// Per-ray partial of the adjoint: dL/dt (3) and the two non-zero columns of
// dL/dR (the ray direction has no y component in the probe frame), FP64.
constexpr int kRayPart = 9;

// Launch wrappers (kernels.hip).  All enqueue on `st` and return the HIP
// error of the launch.
// states: optional records for the adjoint, kStateFloats floats' room per
// carry block, with zcar (one double per block, the sample before it); with
// zcar NULL they lie in the rays' own rows of an image layout, without the
// first of each ray, and may share the memory of the adjoint's zbar;
// gain: optional per-pixel gain (speckle x post-hoc attenuation) output.
// (The int32 pointer is not used.)
// Buffers a kernel clears on the side (a[0..na) and b[0..nb) set to zero)
// A second stream for the launch of the long rays (several wavefronts per
// ray), forked from and joined back into the launch stream with two events,
// so that it runs beside the one-wavefront launch of the other rays.
struct SideStream {
    hipStream_t st;
    hipEvent_t fork, join;
};

struct ZeroArgs {
    float *a;
    long long na;
    double *b;
    long long nb;
};

// zero: cleared by the forward's wavefronts besides their rays (the fused
// step's dL/dZ and pose accumulators), or {} for none
hipError_t launch_forward(int chunk, int xcd_group, const VolArgs &v, const PhysArgs &p,
                          const FanTable &t, const float *poses, float *out,
                          float *min_pivot, int pivot_base, double *zcar, int32_t *,
                          double *states, float *gain, hipStream_t st, const ZeroArgs &zero = ZeroArgs{},
                          int span_samples = kSpanSamples, const SideStream *side = nullptr);
// adjoint: dL/dZ per sample into zbar (image layout), pose sums; in the fused
// form (target given) loss receives one partial per ray.  With pose_acc (a
// flag here), pose_part receives kRayPart doubles per ray of the table;
// launch_pose_reduce then adds them into the pose accumulators.  rays: one
// RayRec per ray of the table, written by the adjoint when zbar is (the
// scatter reads them).  states, zcar: the forward's records; NULL for tables
// whose rays have at most kWholeSamples samples.
hipError_t launch_adjoint(int chunk, int xcd_group, const VolArgs &v, const PhysArgs &p,
                          const FanTable &t, const float *poses, RayRec *rays, const float *gsrc,
                          const float *target, float *zbar, double *pose_acc, double *pose_part, double *loss,
                          const double *zcar, const int32_t *, const double *states,
                          const float *gain, hipStream_t st, int span_samples = kSpanSamples,
                          const SideStream *side = nullptr);
// the sum of the table's per-ray partials per fan (fixed order), into
// t.grad_pose as the pose's finished gradient, or without it added to
// pose_acc[pose]
hipError_t launch_pose_reduce(const FanTable &t, const double *pose_part, double *pose_acc, hipStream_t st);
// fix (nullable): deterministic mode, 64-bit fixed-point sums at the scale
// fscale[0] (launch_fix_scale) instead of FP32 atomics into gZ; wave_target:
// about how many wavefronts the depth segments should make (that of the
// launches running at the same time)
hipError_t launch_scatter(int scatter_rays, int xcd_group, const VolArgs &v, const FanTable &t,
                          const RayRec *rays, const float *zbar, float *gZ, hipStream_t st,
                          unsigned long long *fix = nullptr, const double *fscale = nullptr,
                          int wave_target = 32768);
// deterministic dL/dZ: part[r] = the sum of |zbar| along the table's ray r
// (one double per ray); fscale[2] = the sum of part[0..n), fscale[0..1] =
// 2^e and 2^-e from it; the conversion of the fixed-point sums into gZ
// (overwritten or added)
hipError_t launch_abs_rows(const FanTable &t, const float *zbar, double *part, hipStream_t st);
hipError_t launch_fix_scale(const double *part, int64_t n, double *fscale, hipStream_t st);
hipError_t launch_fix_to_f32(const unsigned long long *fix, int64_t n, const double *fscale, float *gZ,
                             bool overwrite, hipStream_t st);
hipError_t launch_blur(bool transpose, const PhysArgs &p, const FanTable &t, const float *in,
                       float *out, hipStream_t st);
// image = B pre (optional), ebar = B^T (2 (image - target) / P); loss
// receives one MSE partial per blur block (total_blur_blocks entries)
hipError_t launch_blur_residual(const PhysArgs &p, const FanTable &t, const float *pre,
                                const float *target, float *image, float *resid, float *ebar,
                                double *loss, hipStream_t st);
hipError_t launch_pose_finalize(const double *acc, const float *poses, int n_poses,
                                float *grad_pose, hipStream_t st);
hipError_t launch_footprint(const VolArgs &v, const FanTable &t, const float *poses, uint8_t *mask,
                            hipStream_t st);
// impedance at every ray sample (image layout)
hipError_t launch_sample(int xcd_group, const VolArgs &v, const FanTable &t, const float *poses, float *out,
                         hipStream_t st);
// one fan's polar image onto an nz x nx grid of the probe's x-z plane
hipError_t launch_scan_convert(const float *img, int n_rays, int n_samples, double aperture, double r0,
                               double ds, int nx, int nz, double x0, double z0, double dx, double dz,
                               float fill, float *out, hipStream_t st);
hipError_t launch_zero_f64(double *p, int64_t n, hipStream_t st);
hipError_t launch_zero_f32(float *p, int64_t n, hipStream_t st);
// *out = sum of the n partials (the loss of the fused step)
hipError_t launch_sum_f64(const double *part, int64_t n, double *out, hipStream_t st, bool accumulate = false);
// loss = sum of the partials (if loss) and grad = the finalised pose
// gradients (if grad), in one launch
hipError_t launch_finish(const double *part, int64_t n_part, double *loss, const double *acc, const float *poses,
                         int n_poses, float *grad, hipStream_t st);
// a[0..na) = 0 and b[0..nb) = 0 in one launch
hipError_t launch_zero_pair(float *a, int64_t na, double *b, int64_t nb, hipStream_t st);
// smoothness prior of the reconstruction: per-axis weights w / h^2; one
// energy partial per block of voxels (smooth_blocks of them)
int64_t smooth_blocks(int nx, int ny, int nz);
hipError_t launch_smooth(const float *Z, int nx, int ny, int nz, float wx, float wy, float wz, float *gZ,
                         double *part, hipStream_t st);
// Adam with bias corrections c1 = 1 - b1^t, c2 = 1 - b2^t, result clamped to [lo, hi]
hipError_t launch_adam(float *x, const float *g, float *m, float *v, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, float lo, float hi, hipStream_t st);
hipError_t launch_philox(const uint32_t *ctr, int64_t n, uint32_t k0, uint32_t k1, uint32_t *out,
                         hipStream_t st);
// impedance mapping: piecewise-linear table from intensity to impedance
constexpr int kMaxKnots = 64;
struct LutArgs {
    int n;                      // knots, 2..kMaxKnots, x strictly increasing
    float x[kMaxKnots];
    float z[kMaxKnots];
    float x0, xn;               // its ends (set by the launchers)
};
hipError_t launch_map(const float *in, int64_t n, const LutArgs &lut, float *Z, hipStream_t st);
// grad_in (nullable): overwritten; grad_z (nullable): += per knot (FP64)
hipError_t launch_map_backward(const float *in, int64_t n, const LutArgs &lut, const float *gZ, float *grad_in,
                               double *grad_z, hipStream_t st);
hipError_t launch_pixel_gain(const PhysArgs &p, const FanRec &f, float *out, hipStream_t st);

// Static device scratch of the allocation-free entry points (a file-scope
// __device__ array of kernels.hip): *ptr receives its device address on the
// current device, looked up on the first call per device.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
hipError_t static_scratch(void **ptr);

}  // namespace dus
