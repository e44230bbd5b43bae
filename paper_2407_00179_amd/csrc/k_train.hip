// Differentiable emission-absorption render of one whole FP32 volume (ERT off, no
// skipping) and its hand-written adjoint.
//
// Forward: the same quadrature as the brick renderer (32.32 fixed-point sample
// points, trilinear, TF lerp, tau = D A l, T = exp(-sum tau)), storing per ray the
// total optical depth and a checkpoint of the optical depth before every 64th
// segment.
// Backward: per ray, segments are visited in reverse.  Transmittance is never
// stored per sample: the optical depth before a segment is the one after it minus
// its own tau (recomputed from the volume), and it is reset to the stored value at
// every checkpoint.  With g_C = dL/dC, g_a = dL/dalpha and C_{>s} the colour of the
// segments behind s (accumulated on the way back):
//   dL/dc_s   = T_s (1 - e^{-tau_s}) g_C
//   dL/dtau_s = g_C . (T_{s+1} c_s - C_{>s}) + g_a T_S,   dL/dA_s = dL/dtau_s D l_s
// The TF gradient goes to the two lerp entries (weights 1-w, w) through FP64 LDS copies
// flushed once per workgroup; the volume gradient goes to the 8 trilinear corners, through
// an FP64 LDS patch that follows a wave's rays (the kernels on blocked copies) or with global
// atomics, pre-summed in registers while consecutive samples share a cell (the kernels on
// the linear layout).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "march.h"
#include "runtime.hpp"

namespace dpr {

constexpr int kCkpt = 64;  // segments per checkpoint

struct TrainG {
  int dims[3];
  double h, inv_h, dt;
  float dt_f, density, tf_lo, tf_scale;
  int ntf;
  int W, H, n_cams;
  int ws_stride;  // doubles per ray: total optical depth + checkpoints
};

struct TrainRay {
  int64_t p[3], dp[3];
  double t_in, t_out;
  int s0, s1;
  float dl_first, dl_last;
};

__device__ __forceinline__ bool train_begin(const TrainG& g, const double o[3], const double d[3], TrainRay& r) {
  const double lo[3] = {0.0, 0.0, 0.0};
  const double hi[3] = {g.dims[0] * g.h, g.dims[1] * g.h, g.dims[2] * g.h};
  if (!clip_box(o, d, lo, hi, r.t_in, r.t_out)) return false;
  const double dt = g.dt;
  int s0 = (int)floor(r.t_in / dt);
  int s1 = (int)ceil(r.t_out / dt) - 1;
  double lf = fmin((s0 + 1) * dt, r.t_out) - fmax(s0 * dt, r.t_in);
  if (!(lf > 0.0)) {
    ++s0;
    lf = fmin((s0 + 1) * dt, r.t_out) - fmax(s0 * dt, r.t_in);
  }
  double ll = fmin((s1 + 1) * dt, r.t_out) - fmax(s1 * dt, r.t_in);
  if (!(ll > 0.0)) {
    --s1;
    ll = fmin((s1 + 1) * dt, r.t_out) - fmax(s1 * dt, r.t_in);
  }
  r.s0 = s0;
  r.s1 = s1;
  r.dl_first = g.density * (float)lf;
  r.dl_last = g.density * (float)ll;
  const double tm = (s0 + 0.5) * dt;
  for (int a = 0; a < 3; ++a) {
    const double dv = d[a] * g.inv_h;
    r.p[a] = __double2ll_rn(fma(tm, dv, o[a] * g.inv_h - 0.5) * kFix);
    r.dp[a] = __double2ll_rn(dt * dv * kFix);
  }
  return true;
}

// Trilinear stencil of a fixed-point point in the global volume (clamp-to-edge).
struct Stencil {
  int i, j, k;  // base corner
  float fx, fy, fz;
};

__device__ __forceinline__ void stencil_axis(int64_t p, int n, int& i0, float& f) {
  const int hi = (int)(p >> 32);
  float fr = (float)(uint32_t)(p & 0xffffffffll) * (1.0f / 4294967296.0f);
  f = (hi < 0) ? 0.f : ((hi > n - 2) ? 1.f : fr);
  i0 = min(max(hi, 0), n - 2);
}

// The 8 voxels of a stencil, requested; then interpolated.
struct LinearSample {
  Stencil st;
  float v[8];
};
__device__ __forceinline__ void request_linear(const float* __restrict__ vol, const TrainG& g, const int64_t p[3],
                                               LinearSample& s) {
  Stencil& st = s.st;
  stencil_axis(p[0], g.dims[0], st.i, st.fx);
  stencil_axis(p[1], g.dims[1], st.j, st.fy);
  stencil_axis(p[2], g.dims[2], st.k, st.fz);
  const size_t sx = 1, sy = (size_t)g.dims[0], sz = (size_t)g.dims[0] * g.dims[1];
  const size_t b = st.k * sz + st.j * sy + st.i;
  s.v[0] = vol[b], s.v[1] = vol[b + sx], s.v[2] = vol[b + sy], s.v[3] = vol[b + sy + sx];
  s.v[4] = vol[b + sz], s.v[5] = vol[b + sz + sx], s.v[6] = vol[b + sz + sy], s.v[7] = vol[b + sz + sy + sx];
}
__device__ __forceinline__ float value_linear(const LinearSample& s) {
  const float* v = s.v;
  const Stencil& st = s.st;
  return lerp_yz(fmaf(st.fx, v[1] - v[0], v[0]), fmaf(st.fx, v[3] - v[2], v[2]), fmaf(st.fx, v[5] - v[4], v[4]),
                 fmaf(st.fx, v[7] - v[6], v[6]), st.fy, st.fz);
}

__global__ __launch_bounds__(256) void train_forward_kernel(TrainG g, const CamG* __restrict__ cams,
                                                            const float* __restrict__ vol,
                                                            const float4* __restrict__ tf, float4* __restrict__ out,
                                                            float* __restrict__ out_depth, double* __restrict__ ws,
                                                            int tiles_x, int tiles_per_cam) {
  extern __shared__ float4 lds[];
  float4* tfb = lds;
  float4* tfs = lds + g.ntf;
  stage_tf(tf, g.ntf, tfb, tfs, threadIdx.x, 256);
  __syncthreads();
  const int cam_id = blockIdx.x / tiles_per_cam;
  const int tile = blockIdx.x % tiles_per_cam;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int px = (tile % tiles_x) * 16 + (wave & 1) * 8 + (lane & 7);
  const int py = (tile / tiles_x) * 16 + (wave >> 1) * 8 + (lane >> 3);
  if (px >= g.W || py >= g.H) return;
  const CamG& cam = cams[cam_id];
  const size_t ray = ((size_t)cam_id * g.H + py) * g.W + px;
  double* w = ws + ray * g.ws_stride;
  double d[3];
  camera_ray(cam, px, py, d);
  TrainRay r;
  if (!train_begin(g, cam.eye, d, r)) {
    out[ray] = make_float4(0.f, 0.f, 0.f, 0.f);
    out_depth[ray] = INFINITY;
    w[0] = 0.0;
    return;
  }
  int64_t p[3] = {r.p[0], r.p[1], r.p[2]};
  const float Ddt = g.density * g.dt_f;
  double tau_acc = 0.0;
  float tr = 1.f, cr = 0.f, cg = 0.f, cb = 0.f;
  for (int s = r.s0; s <= r.s1; ++s) {
    const int k = s - r.s0;
    if ((k & (kCkpt - 1)) == 0) w[1 + k / kCkpt] = tau_acc;
    LinearSample ls;
    request_linear(vol, g, p, ls);
    const float v = value_linear(ls);
    p[0] += r.dp[0];
    p[1] += r.dp[1];
    p[2] += r.dp[2];
    float x = (v - g.tf_lo) * g.tf_scale;
    x = fminf(fmaxf(x, 0.f), (float)(g.ntf - 1));
    const int j = min((int)x, g.ntf - 2);
    const float wl = x - (float)j;
    const float4 tb = tfb[j], ts = tfs[j];
    const float A = fmaf(wl, ts.w, tb.w);
    const float Dl = (s == r.s0) ? r.dl_first : ((s == r.s1) ? r.dl_last : Ddt);
    const float tau = Dl * A;
    if (tau > 0.f) {
      tau_acc += (double)tau;
      const float tn = __expf(-(float)tau_acc);
      const float wgt = tr - tn;
      cr = fmaf(wgt, fmaf(wl, ts.x, tb.x), cr);
      cg = fmaf(wgt, fmaf(wl, ts.y, tb.y), cg);
      cb = fmaf(wgt, fmaf(wl, ts.z, tb.z), cb);
      tr = tn;
    }
  }
  w[0] = tau_acc;
  out[ray] = make_float4(cr, cg, cb, 1.f - tr);
  out_depth[ray] = (float)r.t_in;
}

// ---- blocked copies.  In the linear layout a wave's rays meet one cache line per lane and
// row, and rows and slices a power of two apart share L2 channels: forward 8.0 ms, backward
// 23.2 ms on 256^3 with 16 cameras at 512^2.  Both kernels instead read the volume, and the
// backward adds its gradient, in the bricks' 8^3-block layout (device_common.h).  The copies cost 41 us
// and the gradient's way back 45 us there; the forward then takes 1.4 ms, the backward 5.4.
// Volumes whose copy would reach 4 GiB (32-bit offsets), or for which the scratch cannot be had,
// and calls under stream capture keep to the linear layout.

// One thread per 4-voxel run: element index 4 i of the blocked arrays, whose bits 2..8 are
// y0 z0 y1 z1 x2 y2 z2.
struct RunPos {
  int x, y, z;
};
__device__ __forceinline__ RunPos run_pos(uint32_t i, uint32_t nbx, uint32_t nby) {
  const uint32_t blk = i >> 7;
  RunPos r;
  r.x = (int)((blk % nbx) * 8 + ((i >> 2) & 4));
  r.y = (int)((blk / nbx % nby) * 8 + (i & 1) + ((i >> 1) & 2) + ((i >> 3) & 4));
  r.z = (int)((blk / nbx / nby) * 8 + ((i >> 1) & 1) + ((i >> 2) & 2) + ((i >> 4) & 4));
  return r;
}
typedef float F4u __attribute__((ext_vector_type(4), aligned(4)));

// The volume into its blocked copy (padding voxels 0); grad (or null): cleared.
__global__ __launch_bounds__(256) void block_volume_kernel(const float* __restrict__ vol, int nx, int ny, int nz,
                                                           uint32_t nbx, uint32_t nby, uint32_t n_runs,
                                                           float4* __restrict__ out, float4* __restrict__ grad) {
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n_runs; i += gridDim.x * 256) {
    const RunPos r = run_pos(i, nbx, nby);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r.y < ny && r.z < nz && r.x < nx) {
      const float* p = vol + ((size_t)r.z * ny + r.y) * nx + r.x;
      if (r.x + 4 <= nx) {
        const F4u u = *(const F4u*)p;
        v = make_float4(u.x, u.y, u.z, u.w);
      } else {
        v.x = p[0];
        if (r.x + 1 < nx) v.y = p[1];
        if (r.x + 2 < nx) v.z = p[2];
      }
    }
    out[i] = v;
    if (grad) grad[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

// grad_volume += the blocked gradient.
__global__ __launch_bounds__(256) void add_blocked_kernel(const float4* __restrict__ grad, int nx, int ny, int nz,
                                                          uint32_t nbx, uint32_t nby, uint32_t n_runs,
                                                          float* __restrict__ out) {
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n_runs; i += gridDim.x * 256) {
    const float4 g = grad[i];
    if (g.x == 0.f && g.y == 0.f && g.z == 0.f && g.w == 0.f) continue;
    const RunPos r = run_pos(i, nbx, nby);
    if (r.y >= ny || r.z >= nz || r.x >= nx) continue;
    float* p = out + ((size_t)r.z * ny + r.y) * nx + r.x;
    if (r.x + 4 <= nx) {
      F4u u = *(const F4u*)p;
      u += F4u{g.x, g.y, g.z, g.w};
      *(F4u*)p = u;
    } else {
      p[0] += g.x;
      if (r.x + 1 < nx) p[1] += g.y;
      if (r.x + 2 < nx) p[2] += g.z;
    }
  }
}

// Tile number t of queue `slot` of `queues`: 4 x 4 tiles (neighbours share cache lines) form a
// patch, and consecutive patches belong to the queues in turn (one queue per XCD: its
// workgroups are the ones whose index has its number in the low bits).  Patches go row by
// row from the middle of the image outwards, through all cameras, so that the long rays
// of a centred volume start first, and each row starts at another column, so that every
// queue has its part of the columns that the volume lies on.  False: no such tile;
// cam == n_cams: nor any later one.
__device__ __forceinline__ bool patch_tile(int t, int slot, int queues, int tiles_x, int tiles_y, int n_cams,
                                           int& cam, int& tx, int& ty) {
  const int nx = (tiles_x + 3) >> 2, ny = (tiles_y + 3) >> 2;
  const int n = (t >> 4) * queues + slot;
  const int row = n / nx;
  const int rank = row / n_cams;
  cam = rank < ny ? row % n_cams : n_cams;
  const int mid = ny >> 1;
  const int y = (rank & 1) ? mid - ((rank + 1) >> 1) : mid + (rank >> 1);
  const int x = (n % nx + 3 * row) % nx;
  tx = x * 4 + (t & 3);
  ty = y * 4 + ((t >> 2) & 3);
  return cam < n_cams && y >= 0 && tx < tiles_x && ty < tiles_y;
}
static unsigned patch_grid(int tiles_x, int tiles_y, int n_cams) {
  const long long patches = (long long)((tiles_x + 3) / 4) * ((tiles_y + 3) / 4) * n_cams;
  return (unsigned)((patches + 7) / 8 * 128);
}

// Forward on the blocked copy: four lanes per ray (march.h), an 8 x 8 pixel tile per
// workgroup, a wave per 4 x 4 pixels.  One call of the march is one checkpoint interval.
__global__ __launch_bounds__(256) void train_forward_blocked_kernel(
    SceneG sc, BrickG b, const CamG* __restrict__ cams, const float4* __restrict__ tf, float4* __restrict__ out,
    float* __restrict__ out_depth, double* __restrict__ ws, int ws_stride, int W, int H, int n_cams) {
  static_assert(kCkpt % (4 * LaneCfg<4>::R) == 0, "whole trips per checkpoint");
  extern __shared__ float4 tf_lds[];
  int cam_id, tx, ty;
  if (!patch_tile(blockIdx.x >> 3, blockIdx.x & 7, 8, (W + 7) >> 3, (H + 7) >> 3, n_cams, cam_id, tx, ty)) return;
  const int lane = threadIdx.x & 63, k = lane & 3, wave = threadIdx.x >> 6, i = lane >> 2;
  const int px = tx * 8 + (wave & 1) * 4 + (i & 3), py = ty * 8 + (wave >> 1) * 4 + (i >> 2);
  const bool in = px < W && py < H;
  const size_t ray = ((size_t)cam_id * H + py) * W + px;
  LaneRay r;
  bool hit = false;
  if (in) {
    const CamG cam = ld_uniform(cams, cam_id);
    double d[3];
    camera_ray(cam, px, py, d);
    hit = lane_begin<float, false, false, 4>(sc, b, cam.eye, d, k, r);
    if (!hit && k == 0) {
      out[ray] = make_float4(0.f, 0.f, 0.f, 0.f);
      out_depth[ray] = INFINITY;
      ws[ray * ws_stride] = 0.0;
    }
  }
  if (!__syncthreads_or(hit)) return;
  stage_tf_records(tf, sc.ntf, tf_lds, threadIdx.x, 256);
  __syncthreads();
  if (!hit) return;
  double* w = ws + ray * ws_stride;
  for (int c = 1;; ++c) {
    if (r.m + k >= 0 && k == 0) w[c] = r.acc;
    if (lane_advance<float, false, false, false, 4, true>(sc, b, tf_lds, r, kCkpt / (4 * LaneCfg<4>::R))) break;
  }
  const float4 rgba = ray_rgba<4>(r);
  if (k == 3) {
    w[0] = r.acc;
    out[ray] = rgba;
    out_depth[ray] = r.t_in;
  }
}

__device__ __forceinline__ void flush_corners(float* __restrict__ gvol, const TrainG& g, const Stencil& st,
                                              const float acc[8]) {
  const size_t sx = 1, sy = (size_t)g.dims[0], sz = (size_t)g.dims[0] * g.dims[1];
  const size_t b = st.k * sz + st.j * sy + st.i;
  const size_t off[8] = {0, sx, sy, sy + sx, sz, sz + sx, sz + sy, sz + sy + sx};
#pragma unroll
  for (int c = 0; c < 8; ++c)
    if (acc[c] != 0.f) atomicAdd(gvol + b + off[c], acc[c]);
}

// The ray's trilinear cell moved from `cur` by (dx, dy, dz), each in {-1, 0, 1}
// (a step of at most one voxel).  Corners the old and new cells share keep their
// sums, moved to their slots in the new cell (slot x + 2 y + 4 z); the others are
// added to the volume gradient.  A move along one axis thus flushes 4 corners,
// not 8.
__device__ __forceinline__ void carry_corners(float* __restrict__ gvol, const TrainG& g, const Stencil& cur,
                                              float acc[8], int dx, int dy, int dz) {
  const size_t sx = 1, sy = (size_t)g.dims[0], sz = (size_t)g.dims[0] * g.dims[1];
  const size_t b = cur.k * sz + cur.j * sy + cur.i;
  const size_t off[8] = {0, sx, sy, sy + sx, sz, sz + sx, sz + sy, sz + sy + sx};
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const bool keep = (unsigned)((c & 1) - dx) <= 1u && (unsigned)(((c >> 1) & 1) - dy) <= 1u &&
                      (unsigned)((c >> 2) - dz) <= 1u;
    if (!keep && acc[c] != 0.f) atomicAdd(gvol + b + off[c], acc[c]);
  }
  // new slot (x, y, z) <- old slot (x + dx, y + dy, z + dz), zero outside the old cell;
  // one axis at a time (slot pairs 1, 2 and 4 apart)
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int d = a == 0 ? dx : (a == 1 ? dy : dz);
    const int st = 1 << a;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      if (c & st) continue;
      const float o0 = acc[c], o1 = acc[c + st];
      acc[c] = d == 0 ? o0 : (d > 0 ? o1 : 0.f);
      acc[c + st] = d == 0 ? o1 : (d < 0 ? o0 : 0.f);
    }
  }
}

// Table-gradient sums in LDS: up to kTfRep FP64 copies (a lane's low bits pick one), copies
// fastest, so that the lanes of a wave meet in few addresses and different copies in different
// banks.  FP64 because an LDS FP32 atomic add takes 193 cycles per wave instruction on
// this chip whatever its addresses, an FP64 one 9 (doubling with every doubling of the
// lanes on one address).
constexpr int kTfRep = 4;

// Table-gradient terms of a ray's consecutive samples in one table interval, summed in
// registers (a ray through a constant region stays in one) and added to LDS when it changes.
struct TfSums {
  int j = -1;  // interval: entries j and j + 1 (-1: none yet)
  float e[8];
  bool colour = false;  // some sample had colour terms
  __device__ __forceinline__ void flush(double* copy, int reps) {
    if (j < 0) return;
    double* q = copy + (size_t)(4 * j) * reps;
    if (colour) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if ((i & 3) != 3) atomicAdd(q + i * reps, (double)e[i]);
    }
    if (e[3] != 0.f || e[7] != 0.f) {
      atomicAdd(q + 3 * reps, (double)e[3]);
      atomicAdd(q + 7 * reps, (double)e[7]);
    }
  }
  // a sample at fraction wl of interval jn: colour terms gc (wgt 0: none), opacity term gA
  __device__ __forceinline__ void add(double* copy, int reps, int jn, float wl, float wgt, float gcR, float gcG,
                                      float gcB, float gA) {
    if (jn != j) {
      flush(copy, reps);
      j = jn;
      colour = false;
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = 0.f;
    }
    const float w0 = 1.f - wl;
    if (wgt != 0.f) {  // (colour terms vanish where the sample is transparent)
      colour = true;
      e[0] = fmaf(w0, gcR, e[0]);
      e[1] = fmaf(w0, gcG, e[1]);
      e[2] = fmaf(w0, gcB, e[2]);
      e[4] = fmaf(wl, gcR, e[4]);
      e[5] = fmaf(wl, gcG, e[5]);
      e[6] = fmaf(wl, gcB, e[6]);
    }
    e[3] = fmaf(w0, gA, e[3]);
    e[7] = fmaf(wl, gA, e[7]);
  }
};

// 1 - e^-tau for tau > 0: the series up to tau^9 below 0.7 (the next term is below 1.2e-8 of
// the sum), the difference above, where e^-tau is below a half.
__device__ __forceinline__ float one_minus_exp(float tau) {
  float p = fmaf(-tau, 1.f / 362880.f, 1.f / 40320.f);
  p = fmaf(-tau, p, 1.f / 5040.f);
  p = fmaf(-tau, p, 1.f / 720.f);
  p = fmaf(-tau, p, 1.f / 120.f);
  p = fmaf(-tau, p, 1.f / 24.f);
  p = fmaf(-tau, p, 1.f / 6.f);
  p = fmaf(-tau, p, 0.5f);
  p = fmaf(-tau, p, 1.f);
  return tau < 0.7f ? tau * p : 1.f - __expf(-tau);
}

__global__ __launch_bounds__(256) void train_backward_kernel(TrainG g, const CamG* __restrict__ cams,
                                                             const float* __restrict__ vol,
                                                             const float4* __restrict__ tf,
                                                             const float4* __restrict__ grad_out,
                                                             const double* __restrict__ ws,
                                                             float* __restrict__ gvol, double* __restrict__ gtf,
                                                             int tiles_x, int tiles_per_cam, int reps) {
  extern __shared__ float4 lds[];
  float4* tfb = lds;
  float4* tfs = lds + g.ntf;
  double* gt = (double*)(lds + 2 * g.ntf);  // reps copies of 4 * ntf sums
  stage_tf(tf, g.ntf, tfb, tfs, threadIdx.x, 256);
  for (int i = threadIdx.x; i < reps * 4 * g.ntf; i += 256) gt[i] = 0.0;
  __syncthreads();
  const int cam_id = blockIdx.x / tiles_per_cam;
  const int tile = blockIdx.x % tiles_per_cam;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int px = (tile % tiles_x) * 16 + (wave & 1) * 8 + (lane & 7);
  const int py = (tile / tiles_x) * 16 + (wave >> 1) * 8 + (lane >> 3);
  const float slope_scale = g.tf_scale;
  double* my_gt = gt + (lane & (reps - 1));
  if (px < g.W && py < g.H) {
    const CamG& cam = cams[cam_id];
    const size_t ray = ((size_t)cam_id * g.H + py) * g.W + px;
    const double* w = ws + ray * g.ws_stride;
    double d[3];
    camera_ray(cam, px, py, d);
    TrainRay r;
    const float4 go = grad_out[ray];
    if (train_begin(g, cam.eye, d, r) && r.s1 >= r.s0 &&
        (go.x != 0.f || go.y != 0.f || go.z != 0.f || go.w != 0.f)) {
      const double tau_total = w[0];
      const float T_S = __expf(-(float)tau_total);
      const float Ddt = g.density * g.dt_f;
      float sr = 0.f, sg = 0.f, sb = 0.f;  // C_{>s}
      double tau_after = tau_total;
      float T_next = T_S;  // transmittance after the current segment
      Stencil cur;
      cur.i = -1;
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      // sample point of the last segment; stepping back by dp gives exactly the
      // forward's points (fixed-point integers)
      int64_t p[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) p[a] = r.p[a] + (int64_t)(r.s1 - r.s0) * r.dp[a];
      TfSums sums;
      LinearSample next;
      request_linear(vol, g, p, next);
      for (int s = r.s1; s >= r.s0; --s) {
        const int k = s - r.s0;
        const LinearSample ls = next;
        const Stencil& st = ls.st;
#pragma unroll
        for (int a = 0; a < 3; ++a) p[a] -= r.dp[a];
        // the next sample's voxels (before the first: clamped voxels, not used)
        request_linear(vol, g, p, next);
        // top of a chunk: optical depth after this segment from the forward's record
        if (((k + 1) & (kCkpt - 1)) == 0 && s != r.s1) {
          tau_after = w[1 + (k + 1) / kCkpt];
          T_next = __expf(-(float)tau_after);
        }
        const float v = value_linear(ls);
        const float xr = (v - g.tf_lo) * g.tf_scale;
        const float x = fminf(fmaxf(xr, 0.f), (float)(g.ntf - 1));
        const int j = min((int)x, g.ntf - 2);
        const float wl = x - (float)j;
        const float4 tb = tfb[j], ts = tfs[j];
        const float A = fmaf(wl, ts.w, tb.w);
        const float cR = fmaf(wl, ts.x, tb.x), cG = fmaf(wl, ts.y, tb.y), cB = fmaf(wl, ts.z, tb.z);
        const float Dl = (s == r.s0) ? r.dl_first : ((s == r.s1) ? r.dl_last : Ddt);
        const float tau = Dl * A;
        float T_s = T_next, wgt = 0.f;
        double tau_before = tau_after;
        if (tau > 0.f) {
          tau_before = tau_after - (double)tau;
          T_s = __expf(-(float)tau_before);
          // (the difference T_s - T_{s+1} would lose most of its digits at tau ~ 1e-5)
          wgt = T_s * one_minus_exp(tau);
        }
        // dL/dc_s and dL/dA_s
        const float gcR = wgt * go.x, gcG = wgt * go.y, gcB = wgt * go.z;
        const float gtau = go.x * (T_next * cR - sr) + go.y * (T_next * cG - sg) + go.z * (T_next * cB - sb) +
                           go.w * T_S;
        const float gA = gtau * Dl;
        sr = fmaf(wgt, cR, sr);
        sg = fmaf(wgt, cG, sg);
        sb = fmaf(wgt, cB, sb);
        tau_after = tau_before;
        T_next = T_s;
        sums.add(my_gt, reps, j, wl, wgt, gcR, gcG, gcB, gA);
        // sample value: zero outside the TF range (clamped u)
        const bool inside = xr >= 0.f && xr <= (float)(g.ntf - 1);
        const float gv = inside ? (gA * ts.w + gcR * ts.x + gcG * ts.y + gcB * ts.z) * slope_scale : 0.f;
        if (st.i != cur.i || st.j != cur.j || st.k != cur.k) {
          const int dx = st.i - cur.i, dy = st.j - cur.j, dz = st.k - cur.k;
          if (cur.i >= 0 && abs(dx) <= 1 && abs(dy) <= 1 && abs(dz) <= 1) {
            carry_corners(gvol, g, cur, acc, dx, dy, dz);
          } else {
            if (cur.i >= 0) flush_corners(gvol, g, cur, acc);
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = 0.f;
          }
          cur = st;
        }
        const float ux = st.fx, uy = st.fy, uz = st.fz;
        const float lx = 1.f - ux, ly = 1.f - uy, lz = 1.f - uz;
        acc[0] = fmaf(gv, lz * ly * lx, acc[0]);
        acc[1] = fmaf(gv, lz * ly * ux, acc[1]);
        acc[2] = fmaf(gv, lz * uy * lx, acc[2]);
        acc[3] = fmaf(gv, lz * uy * ux, acc[3]);
        acc[4] = fmaf(gv, uz * ly * lx, acc[4]);
        acc[5] = fmaf(gv, uz * ly * ux, acc[5]);
        acc[6] = fmaf(gv, uz * uy * lx, acc[6]);
        acc[7] = fmaf(gv, uz * uy * ux, acc[7]);
      }
      sums.flush(my_gt, reps);
      if (cur.i >= 0) flush_corners(gvol, g, cur, acc);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4 * g.ntf; i += 256) {
    double v = 0.0;
    for (int rep = 0; rep < reps; ++rep) v += gt[(size_t)i * reps + rep];
    if (v != 0.0) atomicAdd(gtf + i, v);
  }
}

// ---- backward on the blocked copies
//
// What bounds an adjoint march on this chip (measured): a global FP32 atomic costs a
// request per 64-byte line and instruction, 20.7 G/s for the whole chip, so scattered
// lanes pay one request each and 64 neighbouring floats four; an LDS FP32 atomic add takes
// 193 cycles per wave instruction whatever the addresses, an FP64 one 9 (doubling with every
// doubling of lanes on one address).  A kernel adding each left cell corner to global memory
// and every sample's table terms to FP32 LDS copies took 23.2 ms on 256^3 with 16 cameras at
// 512^2 (275 M requests; 17.6 ms without its LDS adds, 8.1 ms without both).  So:
// - both gradients are summed in LDS in FP64;
// - a wave (8 x 8 pixels, a lane per ray) walks the volume slice by slice along the axis
//   its rays are closest to: every lane does its samples in the slice, then the wave goes
//   on.  A sample of slice a touches the voxel planes a and a + 1, so two planes' patch
//   around the wave's rays is all that is open at a time; the one left behind is added to the
//   blocked global gradient row by row, where neighbouring voxels share a line;
// - the table terms of consecutive samples in one table interval are summed in registers.
// A patch is a rectangle in (w, v) = (u - sh v, v), u and v the other two axes, around a line
// through the wave's rays; sh in {-1, 0, 1} straightens the diagonal patch of an oblique
// view.  Rays whose patch is too wide are taken in halves of the wave's Morton-ordered lanes
// (down to one ray, which always fits).
//
// A persistent workgroup per CU: its 12 waves take tiles from the queue of their XCD
// (patches of 4 x 4 tiles dealt to the XCDs in turn); 8 waves where rays are taken in pieces
// (12: 370 us where 8 take 295 on 64^3 with 4 cameras at 128^2, 886 against 859 on 128^3 with
// 8 at 256^2).
//
// 256^3, 16 cameras at 512^2: 23.2 -> 5.4 ms.  In that time the vector units are issuing for
// 61% (63% of the lanes active: a ray has its samples in a slice or not), the LDS works for
// 40% and the volume's atomics (56 M requests) take 50% of their rate.
constexpr int kBwWaves = 12, kBwWavesSmall = 8;
constexpr int kBwLds = 160 * 1024;      // LDS of a CU
constexpr int kBwMinCells = 512;        // a single ray's patch takes 2 x 10 x 11

// (row shifts and row broadcasts: lane 63 ends with the minimum of all)
__device__ __forceinline__ float wave_reduce_min(float v) {
#define DPR_TRAIN_MIN(ctrl, rows)                                                                            \
  v = fminf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), ctrl, rows, 0xf, false)))
  DPR_TRAIN_MIN(0x111, 0xf);
  DPR_TRAIN_MIN(0x112, 0xf);
  DPR_TRAIN_MIN(0x114, 0xf);
  DPR_TRAIN_MIN(0x118, 0xf);
  DPR_TRAIN_MIN(0x142, 0xa);
  DPR_TRAIN_MIN(0x143, 0xc);
#undef DPR_TRAIN_MIN
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_reduce_max(float v) { return -wave_reduce_min(-v); }
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float fixed_to_float(int64_t p) {
  return fmaf((float)(uint32_t)p, 1.0f / 4294967296.0f, (float)(int)(p >> 32));
}

// Byte offset of index i along one axis of a blocked array: `stride` bytes a block, the
// in-block offsets of x or of y and z (device_common.h) shifted by sh.
__device__ __forceinline__ uint32_t axis_off(int i, uint32_t stride, bool x, int sh) {
  const uint32_t in = __builtin_amdgcn_perm(x ? 0x43424140u : 0x25242120u, x ? 0x03020100u : 0x05040100u, byte_sel(i));
  return ((uint32_t)i >> 3) * stride + (in << sh);
}

// q0, q1 or q2 by a wave-uniform index (with masks: a choice among variables would put
// them in memory)
__device__ __forceinline__ int axis_of(int a, int q0, int q1, int q2) {
  return (q0 & (a == 0 ? -1 : 0)) | (q1 & (a == 1 ? -1 : 0)) | (q2 & (a == 2 ? -1 : 0));
}
__device__ __forceinline__ float axis_of(int a, float q0, float q1, float q2) {
  return __int_as_float(axis_of(a, __float_as_int(q0), __float_as_int(q1), __float_as_int(q2)));
}

// The open patch of a wave (wave-uniform).
struct Patch {
  int A;                   // slice axis; u = (A + 1) % 3, v = (A + 2) % 3
  int sh, S;               // shear, LDS row stride
  int U, V;                // columns (w), rows (v)
  float ref, cw, kw, cv, kv;  // centre line: w = cw + kw (plane - ref), v likewise
  int Hw, Hv;
  __device__ __forceinline__ int ow(int plane) const {
    return (int)floorf(fmaf(kw, (float)plane - ref, cw)) - Hw;
  }
  __device__ __forceinline__ int ov(int plane) const {
    return (int)floorf(fmaf(kv, (float)plane - ref, cv)) - Hv;
  }
};

// Patch of the lanes with `on`, whose rays run between points pe and pb (voxel
// coordinates) with advance d.  False: it does not fit in `cells` LDS cells.
__device__ __forceinline__ bool make_patch(bool on, const float pe[3], const float pb[3], const float d[3], int cells,
                                           Patch& P) {
  const uint64_t mask = __ballot(on);
  const int lead = __ffsll((unsigned long long)mask) - 1;
  auto of_lead = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lead)); };
  const float dx = of_lead(d[0]), dy = of_lead(d[1]), dz = of_lead(d[2]);
  const float ax = fabsf(dx), ay = fabsf(dy), az = fabsf(dz);
  P.A = uniform(ax >= ay && ax >= az ? 0 : (ay >= az ? 1 : 2));
  auto pick = [&](const float q[3], int a) { return axis_of(a, q[0], q[1], q[2]); };
  const int au = P.A == 2 ? 0 : P.A + 1, av = P.A == 0 ? 2 : P.A - 1;
  const float dA = pick(d, P.A), eA = pick(pe, P.A), bA = pick(pb, P.A);
  const float inv = 1.f / dA;
  const float ku = pick(d, au) * inv, kv = pick(d, av) * inv;
  const float lA = of_lead(dA);
  // one direction along the axis, and slopes that keep the centre line near every ray
  const bool ok = !on || (dA * lA > 0.f && fabsf(ku) <= 4.f && fabsf(kv) <= 4.f);
  if (!__all(ok)) return false;
  P.ref = 0.5f * (of_lead(eA) + of_lead(bA));
  const float ur = fmaf(ku, P.ref - eA, pick(pe, au)), vr = fmaf(kv, P.ref - eA, pick(pe, av));
  auto range = [&](float q, float& lo, float& hi) {
    lo = wave_reduce_min(on ? q : INFINITY);
    hi = wave_reduce_max(on ? q : -INFINITY);
  };
  float l0, h0, l1, h1, l2, h2, lv, hv;
  range(ur, l0, h0);
  range(ur - vr, l1, h1);
  range(ur + vr, l2, h2);
  range(vr, lv, hv);
  const float r0 = h0 - l0, r1 = h1 - l1, r2 = h2 - l2;
  P.sh = uniform(r1 < r0 - 1.f && r1 <= r2 ? 1 : (r2 < r0 - 1.f ? -1 : 0));
  const float shf = (float)P.sh;
  P.cw = uniform(P.sh == 0 ? 0.5f * (l0 + h0) : (P.sh > 0 ? 0.5f * (l1 + h1) : 0.5f * (l2 + h2)));
  P.cv = uniform(0.5f * (lv + hv));
  P.kv = of_lead(kv);
  P.kw = of_lead(fmaf(-shf, kv, ku));
  // largest distance from the centre line, at the rays' ends
  float ew = 0.f, ev = 0.f;
  auto far = [&](float A, float qu, float qv) {
    ew = fmaxf(ew, fabsf(fmaf(-shf, qv, qu) - fmaf(P.kw, A - P.ref, P.cw)));
    ev = fmaxf(ev, fabsf(qv - fmaf(P.kv, A - P.ref, P.cv)));
  };
  far(eA, pick(pe, au), pick(pe, av));
  far(bA, pick(pb, au), pick(pb, av));
  // a corner's index is within 1 of its sample's coordinate (2 for u - sh v), the sample
  // within 1.5 of its plane along the axis, and clamping and rounding move it by at most 0.75
  const float Ew = wave_reduce_max(on ? ew : 0.f) + 1.5f * fabsf(P.kw) + 1.f + fabsf(shf) + 0.75f;
  const float Ev = wave_reduce_max(on ? ev : 0.f) + 1.5f * fabsf(P.kv) + 1.f + 0.75f;
  if (!(Ew < 100.f && Ev < 100.f)) return false;
  // |index - centre| <= E: from floor(centre) - floor(E) to floor(centre) + floor(E) + 1
  P.Hw = uniform((int)Ew);
  P.Hv = uniform((int)Ev);
  P.U = 2 * P.Hw + 2;
  P.V = 2 * P.Hv + 2;
  P.S = P.U | 1;
  return P.U <= 32 && 2 * P.V * P.S <= cells;
}

// The pieces that the rays of a small launch are taken in: one checkpoint interval of a
// tile each, or of a quarter of it (16 rays) where there are fewer pieces than waves.
// Measured for a whole forward and backward, whole rays / tiles / quarters:
//    64^3,  4 cameras at 128^2 ( 1024 tiles)  583 /  295 /  271 us
//   128^3,  2 cameras at 256^2 ( 2048 tiles) 1994 /  396 /  570 us
//   128^3,  8 cameras at 256^2 ( 8192 tiles) 2382 /  859 / 1665 us
//    64^3,  8 cameras at 256^2 ( 8192 tiles)  430 /  461 /  863 us
//   128^3,  4 cameras at 512^2 (16384 tiles) 1017 / 1204 / 2797 us
// (half of a launch's tiles meet the volume; its whole rays keep 3072 waves busy, all but
// the last of each, from two tiles a wave on, and need no second march).
constexpr int kPieceTiles = 8192;
constexpr size_t kPieceBytes = 1ull << 30;
constexpr int kQuarterPieces = 4096;
constexpr int kWholeTile = 4;
struct TrainPieces {
  int chunks = 1;                // intervals per ray (1: whole rays, and no list)
  const float4* col = nullptr;   // colour of interval c of a ray, at ray * chunks + c
  const uint2* list = nullptr;   // (tile, 8 * interval + quarter or kWholeTile)
  const int* count = nullptr;
};
constexpr int kHeadStride = 32;  // ints between queue heads (a cache line each)

__global__ __launch_bounds__(64 * kBwWaves) void train_backward_blocked_kernel(
    SceneG sc, BrickG b, const CamG* __restrict__ cams, const float4* __restrict__ tf,
    const float4* __restrict__ grad_out, const double* __restrict__ ws, int ws_stride, float* __restrict__ grad,
    double* __restrict__ gtf, int* __restrict__ heads, int W, int H, int n_cams, int reps, int cells, TrainPieces pieces) {
  extern __shared__ float4 lds[];
  float4* tfr = lds;
  double* gt = (double*)(lds + 2 * sc.ntf);  // table gradient: reps copies of 4 ntf, copies fastest
  double* patches = gt + (size_t)reps * 4 * sc.ntf;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double* cell = patches + wave * cells;     // this wave's two planes
  stage_tf_records(tf, sc.ntf, tfr, threadIdx.x, blockDim.x);
  for (int i = threadIdx.x; i < reps * 4 * sc.ntf + (int)(blockDim.x >> 6) * cells;
       i += blockDim.x) gt[i] = 0.0;
  __syncthreads();
  // a wave's first item is its own, so that a launch starts without thousands of atomics on
  // few counters
  const int queues = pieces.list ? 1 : 8;
  const int slot = blockIdx.x & (queues - 1);
  const int own = (int)(threadIdx.x >> 6) * (gridDim.x / queues) + blockIdx.x / queues;
  int next = uniform(own);
  const int chunks = pieces.chunks;
  const int tiles_x = (W + 7) >> 3, tiles_y = (H + 7) >> 3;
  double* my_gt = gt + (lane & (reps - 1));
  const float x_max = (float)(sc.ntf - 1);
  const float Ddt = sc.density * sc.dt_f;
  // lane -> pixel in Morton order, so that halves and quarters of the wave are compact
  const int lx8 = (lane & 1) | ((lane >> 1) & 2) | ((lane >> 2) & 4);
  const int ly8 = ((lane >> 1) & 1) | ((lane >> 2) & 2) | ((lane >> 3) & 4);

  for (;;) {
    int t = next;
    if (t < 0) {
      if (lane == 0) t = atomicAdd(heads + slot * kHeadStride, 1);
      t = uniform(t);
    }
    next = -1;
    int cam_id, tx, ty, chunk = 0, quarter = kWholeTile;
    if (pieces.list) {
      if (t >= uniform(*pieces.count)) break;
      const uint2 item = pieces.list[t];
      const int tile = uniform((int)item.x), part = uniform((int)item.y);
      tx = tile % tiles_x;
      ty = tile / tiles_x % tiles_y;
      cam_id = tile / (tiles_x * tiles_y);
      chunk = part >> 3;
      quarter = part & 7;
    } else {
      const bool tile = patch_tile(t, slot, queues, tiles_x, tiles_y, n_cams, cam_id, tx, ty);
      if (cam_id >= n_cams) break;
      if (!tile) continue;
    }
    const int px = tx * 8 + lx8, py = ty * 8 + ly8;
    const size_t ray = ((size_t)cam_id * H + py) * W + px;
    float4 go = make_float4(0.f, 0.f, 0.f, 0.f);
    RaySetup r;
    bool hit = false;
    int lo = 0, hi = -1;  // the ray's segments to do
    if (px < W && py < H && (quarter == kWholeTile || (lane >> 4) == quarter)) {
      const CamG cam = ld_uniform(cams, cam_id);
      double d[3];
      camera_ray(cam, px, py, d);
      hit = ray_begin(sc, b, cam.eye, d, r);
      if (hit) {
        lo = chunks > 1 ? r.s0 + chunk * kCkpt : r.s0;
        hi = chunks > 1 ? min(r.s1, lo + kCkpt - 1) : r.s1;
        hit = hi >= lo;
      }
      if (hit) {
        go = grad_out[ray];
        hit = go.x != 0.f || go.y != 0.f || go.z != 0.f || go.w != 0.f;
      }
    }
    if (__ballot(hit) == 0) continue;
    const double* w = ws + ray * ws_stride;
    const double tau_total = hit ? w[0] : 0.0;
    const float T_S = __expf(-(float)tau_total);
    float4 behind = make_float4(0.f, 0.f, 0.f, 0.f);  // colour of the ray's later chunks
    if (chunks > 1 && hit) {
      for (int c = (r.s1 - r.s0) / kCkpt; c > chunk; --c) {
        const float4 q = pieces.col[ray * chunks + c];
        behind.x += q.x;
        behind.y += q.y;
        behind.z += q.z;
      }
    }

    int part = 64;  // lanes taken together
    for (int m0 = 0; m0 < 64;) {
      const bool on = hit && lane >= m0 && lane < m0 + part;
      if (__ballot(on) == 0) {
        m0 += part;
        continue;
      }
      // the range's ends and the ray's advance, for the patch
      int64_t p[3] = {0, 0, 0};
      float pe[3] = {0.f, 0.f, 0.f}, pb[3] = {0.f, 0.f, 0.f}, df[3] = {0.f, 0.f, 0.f};
      if (on) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          // sample point of the last segment; stepping back by dp gives exactly the
          // forward's points (fixed-point integers)
          p[a] = r.p[a] + (int64_t)(hi - r.s0) * r.dp[a];
          pe[a] = fixed_to_float(p[a]);
          pb[a] = fixed_to_float(r.p[a] + (int64_t)(lo - r.s0) * r.dp[a]);
          df[a] = fixed_to_float(r.dp[a]);
        }
      }
      Patch P;
      if (!make_patch(on, pe, pb, df, cells, P) && part > 1) {
        part >>= 1;
        continue;
      }
      m0 += part;
      // (the rays of a patch run one way along the axis, and the march goes back along them)
      const bool down = __ballot(on && axis_of(P.A, df[0], df[1], df[2]) > 0.f) != 0;
      // cell index = j . stride + base(plane); the slice axis has stride 0 and its step
      // leads to the next plane's base
      const int sv = P.S - P.sh, PS = P.V * P.S;
      const int kx = P.A == 0 ? 0 : (P.A == 1 ? sv : 1), ky = P.A == 1 ? 0 : (P.A == 2 ? sv : 1),
                kz = P.A == 2 ? 0 : (P.A == 0 ? sv : 1);
      // byte strides of a block and shifts of the in-block offset along the three axes
      const uint32_t str[3] = {(uint32_t)kBlockVoxels * 4u, b.bsy * 4u, b.bsz * 4u};
      const uint32_t a_stride = (uint32_t)axis_of(P.A, (int)str[0], (int)str[1], (int)str[2]);
      const uint32_t u_stride = (uint32_t)axis_of(P.A, (int)str[1], (int)str[2], (int)str[0]);
      const uint32_t v_stride = (uint32_t)axis_of(P.A, (int)str[2], (int)str[0], (int)str[1]);
      const int a_sh = axis_of(P.A, 2, 4, 5), u_sh = axis_of(P.A, 4, 5, 2), v_sh = axis_of(P.A, 5, 2, 4);
      const bool u_x = P.A == 2, v_x = P.A == 1;
      auto base = [&](int plane) { return (plane & 1) * PS - P.ov(plane) * P.S - P.ow(plane); };
      auto flush = [&](int plane) {
        // (the wave's own LDS operations complete in order; the compiler keeps it too)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double* c = cell + (plane & 1) * PS;
        const int ow = P.ow(plane), ov = P.ov(plane);
        const uint32_t f_plane = axis_off(plane, a_stride, P.A == 0, a_sh);
        // 8 rows of 8 columns, 4 of 16 or 2 of 32 at once, F times (2 of 32 always, four times:
        // 260 against 248 us on 64^3 with 4 cameras at 128^2, 5.47 against 5.38 ms on 256^3)
        const int cb = P.U <= 8 ? 3 : (P.U <= 16 ? 4 : 5), rows = 64 >> cb;
        const int col = lane & ((1 << cb) - 1);
        constexpr int F = 2;
        for (int row0 = lane >> cb; row0 < P.V; row0 += rows * F) {
          double g[F];
#pragma unroll
          for (int i = 0; i < F; ++i) {
            const int row = row0 + rows * i;
            g[i] = row < P.V && col < P.U ? c[row * P.S + col] : 0.0;
          }
#pragma unroll
          for (int i = 0; i < F; ++i) {
            const int row = row0 + rows * i;
            if (g[i] != 0.0) {
              c[row * P.S + col] = 0.0;
              const int jv = row + ov, ju = col + ow + P.sh * jv;
              const uint32_t off = f_plane + axis_off(jv, v_stride, v_x, v_sh) + axis_off(ju, u_stride, u_x, u_sh);
              atomicAdd((float*)((char*)grad + off), (float)g[i]);
            }
          }
        }
      };
      float sr = behind.x, sg = behind.y, sb = behind.z;  // C_{>s}
      double tau_after = tau_total;
      float T_next = T_S;  // transmittance after the current segment
      int s = on ? hi : -1, s0 = on ? lo : 0;  // (s < s0: no samples left)
      TfSums sums;
      Sample<float> g;
      if (on) request<float, false>(b, p[0], p[1], p[2], g);
      // base cell of the lane's next sample
      auto cell_of = [&](int a) { return clamp_index((int)(p[a] >> 32), b.sdim[a] - 2); };
      int ix = cell_of(0), iy = cell_of(1), iz = cell_of(2);
      auto slice_of = [&]() { return axis_of(P.A, ix, iy, iz); };
      int sl;  // the open slice
      {
        const float q = (float)slice_of();
        sl = uniform((int)(down ? wave_reduce_max(on ? q : -INFINITY) : wave_reduce_min(on ? q : INFINITY)));
      }
      bool dirty0 = false, dirty1 = false;  // planes sl and sl + 1 hold something
      while (true) {
        const int B0 = base(sl), step = base(sl + 1) - B0;
        const int ox = P.A == 0 ? step : kx, oy = P.A == 1 ? step : ky, oz = P.A == 2 ? step : kz;
        bool added = false;
        while (true) {
          const bool now = s >= s0 && slice_of() == sl;
          if (__ballot(now) == 0) break;
          if (now) {
            const int k = s - r.s0;
            const Sample<float> h = g;
            const uint32_t a0 = mad24u(ix, kx, mad24u(iy, ky, mad24u(iz, kz, (uint32_t)B0)));
#pragma unroll
            for (int a = 0; a < 3; ++a) p[a] -= r.dp[a];
            // the next sample's voxels (before the first: clamped voxels, not used)
            request<float, false>(b, p[0], p[1], p[2], g);
            ix = cell_of(0);
            iy = cell_of(1);
            iz = cell_of(2);
            __builtin_amdgcn_sched_barrier(0);
            // top of a chunk: optical depth after this segment from the forward's record
            if (((k + 1) & (kCkpt - 1)) == 0 && s != r.s1) {
              tau_after = w[1 + (k + 1) / kCkpt];
              T_next = __expf(-(float)tau_after);
            }
            const float v = sample_value(h);
            const float xr = (v - sc.tf_lo) * sc.tf_scale;
            const float x = __builtin_amdgcn_fmed3f(xr, 0.f, x_max);
            const int j = min((int)x, sc.ntf - 2);
            const float wl = x - (float)j;
            const float4 tb = tfr[2 * j], ts = tfr[2 * j + 1];
            const float A = fmaf(wl, ts.w, tb.w);
            const float cR = fmaf(wl, ts.x, tb.x), cG = fmaf(wl, ts.y, tb.y), cB = fmaf(wl, ts.z, tb.z);
            const float Dl = (s == r.s0) ? r.dl_first : ((s == r.s1) ? r.dl_last : Ddt);
            const float tau = Dl * A;
            float T_s = T_next, wgt = 0.f;
            double tau_before = tau_after;
            if (tau > 0.f) {
              tau_before = tau_after - (double)tau;
              T_s = __expf(-(float)tau_before);
              // (the difference T_s - T_{s+1} would lose most of its digits at tau ~ 1e-5)
              wgt = T_s * one_minus_exp(tau);
            }
            // dL/dc_s and dL/dA_s
            const float gcR = wgt * go.x, gcG = wgt * go.y, gcB = wgt * go.z;
            const float gtau =
                go.x * (T_next * cR - sr) + go.y * (T_next * cG - sg) + go.z * (T_next * cB - sb) + go.w * T_S;
            const float gA = gtau * Dl;
            sr = fmaf(wgt, cR, sr);
            sg = fmaf(wgt, cG, sg);
            sb = fmaf(wgt, cB, sb);
            tau_after = tau_before;
            T_next = T_s;
            --s;
            sums.add(my_gt, reps, j, wl, wgt, gcR, gcG, gcB, gA);
            // sample value: zero outside the TF range (clamped u)
            const bool inside = xr >= 0.f && xr <= x_max;
            const float gv = inside ? (gA * ts.w + gcR * ts.x + gcG * ts.y + gcB * ts.z) * sc.tf_scale : 0.f;
            if (gv != 0.f) {
              added = true;
              const float g0 = gv * (1.f - h.fz), g1 = gv * h.fz;
              const float ly = 1.f - h.fy, lx = 1.f - h.fx;
              const float g00 = g0 * ly, g01 = g0 * h.fy, g10 = g1 * ly, g11 = g1 * h.fy;
              double* c = cell + a0;
              atomicAdd(c, (double)(g00 * lx));
              atomicAdd(c + ox, (double)(g00 * h.fx));
              atomicAdd(c + oy, (double)(g01 * lx));
              atomicAdd(c + oy + ox, (double)(g01 * h.fx));
              atomicAdd(c + oz, (double)(g10 * lx));
              atomicAdd(c + oz + ox, (double)(g10 * h.fx));
              atomicAdd(c + oz + oy, (double)(g11 * lx));
              atomicAdd(c + oz + oy + ox, (double)(g11 * h.fx));
            }
          }
        }
        if (__ballot(added) != 0) dirty0 = dirty1 = true;
        const bool last = __ballot(s >= s0) == 0;
        if (down) {
          if (dirty1) flush(sl + 1);
          dirty1 = dirty0;
          dirty0 = false;
          --sl;
        } else {
          if (dirty0) flush(sl);
          dirty0 = dirty1;
          dirty1 = false;
          ++sl;
        }
        if (last) {
          if (dirty0) flush(sl);
          if (dirty1) flush(sl + 1);
          break;
        }
      }
      sums.flush(my_gt, reps);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4 * sc.ntf; i += blockDim.x) {
    double v = 0.0;
    for (int q = 0; q < reps; ++q) v += gt[(size_t)i * reps + q];
    if (v != 0.0) atomicAdd(gtf + i, v);
  }
}

// Colour that each checkpoint interval adds to its ray's pixel, so that the backward can
// take the intervals of a ray one by one: the forward march from the interval's recorded
// optical depth.  One workgroup per (8 x 8 pixel tile, interval), a wave per quarter of the
// tile (4 x 4 pixels, the Morton quarter of the backward's lanes); lists the pieces that
// some ray reaches.
__global__ __launch_bounds__(256) void train_chunk_kernel(SceneG sc, BrickG b, const CamG* __restrict__ cams,
                                                          const float4* __restrict__ tf,
                                                          const double* __restrict__ ws, int ws_stride, int W, int H,
                                                          int n_cams, int chunks, int quarters, float4* __restrict__ col,
                                                          uint2* __restrict__ list, int* __restrict__ count) {
  extern __shared__ float4 tf_lds[];
  int cam_id, tx, ty;
  if (!patch_tile(blockIdx.x >> 3, blockIdx.x & 7, 8, (W + 7) >> 3, (H + 7) >> 3, n_cams, cam_id, tx, ty)) return;
  const int lane = threadIdx.x & 63, k = lane & 3, wave = threadIdx.x >> 6, i = lane >> 2;
  const int px = tx * 8 + (wave & 1) * 4 + (i & 3), py = ty * 8 + (wave >> 1) * 4 + (i >> 2);
  const int chunk = blockIdx.y;
  const size_t ray = ((size_t)cam_id * H + py) * W + px;
  LaneRay r;
  bool hit = false;
  if (px < W && py < H) {
    const CamG cam = ld_uniform(cams, cam_id);
    double d[3];
    camera_ray(cam, px, py, d);
    hit = lane_begin<float, false, false, 4>(sc, b, cam.eye, d, k, r);
    if (hit) {
      r.m -= chunk * kCkpt;
      hit = r.m + k >= 0;
    }
  }
  const bool any = quarters ? __ballot(hit) != 0 : __syncthreads_or(hit) != 0;
  if (any && (quarters ? lane : (int)threadIdx.x) == 0) {
    const int tiles_x = (W + 7) >> 3, tiles_y = (H + 7) >> 3;
    list[atomicAdd(count, 1)] =
        make_uint2((cam_id * tiles_y + ty) * tiles_x + tx, 8 * chunk + (quarters ? wave : kWholeTile));
  }
  // (nothing lies before the first interval)
  if (chunk == 0 || !__syncthreads_or(hit)) return;
  stage_tf_records(tf, sc.ntf, tf_lds, threadIdx.x, 256);
  __syncthreads();
  if (!hit) return;
#pragma unroll
  for (int a = 0; a < 3; ++a) r.q[a] += (int64_t)(chunk * (kCkpt / 4)) * r.d[a];
  r.acc = ws[ray * ws_stride + 1 + chunk];
  r.tr = __expf(-(float)r.acc);
  r.dl_cur = sc.density * sc.dt_f;
  lane_advance<float, false, false, false, 4, true>(sc, b, tf_lds, r, kCkpt / (4 * LaneCfg<4>::R));
  const float4 rgba = ray_rgba<4>(r);
  if (k == 0) col[ray * chunks + chunk] = rgba;
}

// clears the table sums and the tile queues behind them
__global__ void fill_f64_kernel(double* p, int n, int* heads, int first) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
  if (i < 8) heads[i * kHeadStride] = first;
  if (i == 8) heads[i * kHeadStride] = 0;  // the list's length
}

// grad_tf += the FP64 sums (rounded once to FP32)
__global__ void add_f64_to_f32_kernel(const double* __restrict__ src, float* __restrict__ dst, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] += (float)src[i];
}

static int max_segments(const int64_t dims[3], float step) {
  const double m = (double)std::max(dims[0], std::max(dims[1], dims[2]));
  const double diag = std::sqrt((double)dims[0] * dims[0] + (double)dims[1] * dims[1] + (double)dims[2] * dims[2]) / m;
  return (int)std::ceil(diag / (step / m)) + 3;
}

static dpr_status check_train(const int64_t dims[3], const dpr_camera* cams, int n, const dpr_render_params* prm,
                              int n_tf, float lo, float hi, float density) {
  if (!dims || !cams || !prm) return fail(DPR_ERR_INVALID_ARGUMENT, "training call: NULL argument");
  for (int a = 0; a < 3; ++a)
    if (dims[a] < 2 || dims[a] > (1 << 16)) return fail(DPR_ERR_INVALID_ARGUMENT, "training call: dims[%d]", a);
  if (n < 1) return fail(DPR_ERR_INVALID_ARGUMENT, "training call: n = %d", n);
  for (int c = 0; c < n; ++c) {
    dpr_status s = check_camera(&cams[c]);
    if (s != DPR_OK) return s;
    if (cams[c].width != cams[0].width || cams[c].height != cams[0].height)
      return fail(DPR_ERR_INVALID_ARGUMENT, "training call: all cameras must share one image size");
  }
  if (!(prm->step_voxels > 0.f && prm->step_voxels <= 1.f))
    return fail(DPR_ERR_INVALID_ARGUMENT, "training call: step_voxels %g", prm->step_voxels);
  if (n_tf < 2 || n_tf > kMaxTF) return fail(DPR_ERR_INVALID_ARGUMENT, "training call: n_tf %d", n_tf);
  if (!(hi > lo)) return fail(DPR_ERR_INVALID_ARGUMENT, "training call: value range");
  if (!(density >= 0.f)) return fail(DPR_ERR_INVALID_ARGUMENT, "training call: density");
  return DPR_OK;
}

static TrainG make_train(const int64_t dims[3], const dpr_camera* cams, int n, const dpr_render_params* prm, int n_tf,
                         float lo, float hi, float density) {
  TrainG g{};
  int64_t m = std::max(dims[0], std::max(dims[1], dims[2]));
  for (int a = 0; a < 3; ++a) g.dims[a] = (int)dims[a];
  g.h = 1.0 / (double)m;
  g.inv_h = (double)m;
  g.dt = (double)prm->step_voxels * g.h;
  g.dt_f = (float)g.dt;
  g.density = density;
  g.tf_lo = lo;
  g.tf_scale = (float)(n_tf - 1) / (hi - lo);
  g.ntf = n_tf;
  g.W = cams[0].width;
  g.H = cams[0].height;
  g.n_cams = n;
  g.ws_stride = 1 + (max_segments(dims, prm->step_voxels) + kCkpt - 1) / kCkpt;
  return g;
}

// ---- scratch of the training calls (the blocked copies, the FP64 table sums), kept by the
// device and grown on demand.  A call on another stream than the last one's waits for it
// on the GPU.  (A call under capture takes the table sums only, in the caller's ordering.)
static dpr_status scratch_begin(dpr_device dev) {
  if (dev->train_stream_set && dev->train_stream != dev->stream && dev->train_ev) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    DPR_HIP(hipStreamIsCapturing(dev->stream, &cs));
    if (cs == hipStreamCaptureStatusNone) DPR_HIP(hipStreamWaitEvent(dev->stream, dev->train_ev, 0));
  }
  return DPR_OK;
}
static dpr_status scratch_end(dpr_device dev) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  DPR_HIP(hipStreamIsCapturing(dev->stream, &cs));
  if (cs != hipStreamCaptureStatusNone) return DPR_OK;
  if (!dev->train_ev) DPR_HIP(hipEventCreateWithFlags(&dev->train_ev, hipEventDisableTiming));
  DPR_HIP(hipEventRecord(dev->train_ev, dev->stream));
  dev->train_stream = dev->stream;
  dev->train_stream_set = true;
  return DPR_OK;
}

// The blocked copies of a volume, where they can be had: below 4 GiB (32-bit offsets), when
// the memory is there, and outside stream capture.  Else the kernels on the linear layout
// run, and where they are the faster ones (train_small, train_coarse).
struct TrainBlocks {
  float* vol = nullptr;
  float* grad = nullptr;
  uint32_t nb[3] = {0, 0, 0};
  uint32_t n_runs = 0;
};
// Scratch buffer i of at least `bytes`; null where it cannot be had.
static void* train_buffer(dpr_device dev, int i, size_t bytes) {
  if (dev->train_cap[i] < bytes) {
    dev_free(dev->train_buf[i]);  // (waits for the device)
    dev->train_buf[i] = nullptr;
    dev->train_cap[i] = 0;
    if (dev_alloc(&dev->train_buf[i], bytes, "training scratch") != DPR_OK) return nullptr;
    dev->train_cap[i] = bytes;
  }
  return dev->train_buf[i];
}
static bool train_blocks(dpr_device dev, const TrainG& g, bool grad, TrainBlocks& t) {
  uint64_t n = kBlockVoxels;
  for (int a = 0; a < 3; ++a) {
    t.nb[a] = (uint32_t)(g.dims[a] + 7) / 8;
    n *= t.nb[a];
  }
  if (n * 4 > 0xffffffffull) return false;
  // (a graph may be replayed after the scratch has grown, and beside other calls)
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(dev->stream, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return false;
  const size_t bytes = (size_t)n * 4 + kPairSlack;
  t.vol = (float*)train_buffer(dev, 0, bytes);
  if (grad) t.grad = (float*)train_buffer(dev, 1, bytes);
  if (!t.vol || (grad && !t.grad)) return false;
  t.n_runs = (uint32_t)(n / 4);
  return true;
}

// Where the kernels on the linear layout are the faster ones, by the work in ray-voxels (rays
// times the longest extent).  Measured, a forward and backward on the blocked copies / with
// the linear backward / with both linear:
// - a launch so small that the copies' kernels cost more than they save:
//    33^3,  1 camera  at  65^2 (0.14 M)  200 /  183 /  173 us
//    40^3,  1 camera  at 100^2 (0.4 M)   188 /  182 /  173 us
//    64^3,  4 cameras at  65^2 (1.1 M)   264 /  307 /  359 us
// - the backward of many rays that lie voxels apart (at the volume's centre): they share no
//   cells, and a patch around them is mostly empty, but few rays fill the chip only that way:
//    64^3, 12 cameras at  65^2 (2.8 voxels, 3.2 M)   286 /  340 us
//   200^3,  2 cameras at 100^2 (5.7 voxels, 4.0 M)   725 / 1214 us
//   128^3,  4 cameras at 100^2 (3.6 voxels, 5.1 M)   985 /  669 us
//   128^3, 12 cameras at  65^2 (5.6 voxels, 6.5 M)  1680 /  748 us
//   200^3,  6 cameras at 200^2 (2.8 voxels, 48 M)   1434 / 1512 us
//   128^3,  4 cameras at 181^2 (2.0 voxels, 17 M)    583 /  730 us
constexpr double kSmallWork = 0.6e6, kCoarsePitch = 2.4, kCoarseWork = 4.5e6;
static double train_work(const TrainG& g) {
  return (double)g.n_cams * g.W * g.H * std::max(g.dims[0], std::max(g.dims[1], g.dims[2]));
}
static bool train_small(const TrainG& g) { return train_work(g) <= kSmallWork; }
static bool train_coarse(const TrainG& g, const dpr_camera* cams) {
  if (train_work(g) < kCoarseWork) return false;
  double sum = 0.0;  // pixel pitches at the centre
  for (int c = 0; c < g.n_cams; ++c) {
    double d2 = 0.0;
    for (int a = 0; a < 3; ++a) {
      const double d = cams[c].eye[a] - 0.5 * g.dims[a] * g.h;
      d2 += d * d;
    }
    sum += std::sqrt(d2) * 2.0 * std::tan(cams[c].fovy_deg * M_PI / 360.0) / g.H;
  }
  return sum * g.inv_h >= kCoarsePitch * g.n_cams;
}

static SceneG train_scene(const TrainG& g) {
  SceneG s{};
  for (int a = 0; a < 3; ++a) s.dims[a] = g.dims[a];
  s.h = g.h;
  s.inv_h = g.inv_h;
  s.dt = g.dt;
  s.dt_f = g.dt_f;
  s.density = g.density;
  s.ert = 2.f;
  s.ert_t = -1.f;
  s.tf_lo = g.tf_lo;
  s.tf_scale = g.tf_scale;
  s.ntf = g.ntf;
  return s;
}

// The whole volume as one brick over its blocked copy.
static BrickG train_brick(const TrainG& g, const TrainBlocks& t) {
  BrickG b{};
  b.data = t.vol;
  for (int a = 0; a < 3; ++a) {
    b.sdim[a] = g.dims[a];
    b.ohi[a] = g.dims[a];
    b.mdim[a] = 1;
  }
  b.nbx = t.nb[0];
  b.nbxy = t.nb[0] * t.nb[1];
  b.bsy = kBlockVoxels * b.nbx;
  b.bsz = kBlockVoxels * b.nbxy;
  return b;
}

static unsigned run_grid(uint32_t n_runs, int cu_count) {
  return (unsigned)std::min<uint64_t>(((uint64_t)n_runs + 255) / 256, (uint64_t)cu_count * 16);
}

// Camera tables of the training calls, cached per device by content.
struct CamCacheEntry {
  dpr_device dev;
  int hip_device;
  std::vector<dpr_camera> cams;
  CamG* table;
};

static dpr_status cam_table(dpr_device dev, const dpr_camera* cams, int n, CamG** out) {
  static thread_local std::vector<CamCacheEntry> cache;
  for (auto& e : cache)
    if (e.dev == dev && e.hip_device == dev->dev && (int)e.cams.size() == n &&
        memcmp(e.cams.data(), cams, n * sizeof(dpr_camera)) == 0) {
      *out = e.table;
      return DPR_OK;
    }
  std::vector<CamG> h(n);
  for (int c = 0; c < n; ++c) h[c] = make_cam(cams[c]);
  CamG* d = nullptr;
  dpr_status s = dev_alloc((void**)&d, n * sizeof(CamG), "training cameras");
  if (s != DPR_OK) return s;
  DPR_HIP(hipMemcpyAsync(d, h.data(), n * sizeof(CamG), hipMemcpyHostToDevice, dev->stream));
  DPR_HIP(hipStreamSynchronize(dev->stream));
  if (cache.size() >= 16) {
    DPR_HIP(hipStreamSynchronize(dev->stream));
    dev_free(cache.front().table);
    cache.erase(cache.begin());
  }
  cache.push_back({dev, dev->dev, std::vector<dpr_camera>(cams, cams + n), d});
  *out = d;
  return DPR_OK;
}

}  // namespace dpr

using namespace dpr;

extern "C" {

dpr_status dpr_train_workspace_size(const int64_t dims[3], const dpr_camera* cams, int32_t n, float step,
                                    size_t* bytes) {
  if (!dims || !cams || !bytes) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_train_workspace_size: NULL argument");
  dpr_render_params p{step, 2.f, 16, 0u};
  dpr_status s = check_train(dims, cams, n, &p, 2, 0.f, 1.f, 0.f);
  if (s != DPR_OK) return s;
  TrainG g = make_train(dims, cams, n, &p, 2, 0.f, 1.f, 0.f);
  *bytes = (size_t)n * g.W * g.H * g.ws_stride * sizeof(double);
  return DPR_OK;
}

dpr_status dpr_render_train_forward(dpr_device dev, const float* volume, const int64_t dims[3], const float* tf,
                                    int32_t n_tf, float lo, float hi, float density, const dpr_render_params* prm,
                                    const dpr_camera* cams, int32_t n, float* out_rgba, float* out_depth,
                                    void* ws, size_t ws_bytes) {
  if (!dev || !volume || !tf || !out_rgba || !out_depth || !ws)
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_train_forward: NULL argument");
  dpr_status s = check_train(dims, cams, n, prm, n_tf, lo, hi, density);
  if (s != DPR_OK) return s;
  TrainG g = make_train(dims, cams, n, prm, n_tf, lo, hi, density);
  size_t need = (size_t)n * g.W * g.H * g.ws_stride * sizeof(double);
  if (ws_bytes < need)
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_train_forward: workspace %zu < %zu bytes", ws_bytes, need);
  CamG* dc = nullptr;
  if ((s = cam_table(dev, cams, n, &dc)) != DPR_OK) return s;
  const int tx = (g.W + 15) / 16, ty = (g.H + 15) / 16;
  dim3 grid((unsigned)(tx * ty * n));
  size_t lds = 2 * sizeof(float4) * (size_t)n_tf;
  TrainBlocks t;
  if (!train_small(g) && train_blocks(dev, g, false, t)) {
    if ((s = scratch_begin(dev)) != DPR_OK) return s;
    hipLaunchKernelGGL(block_volume_kernel, dim3(run_grid(t.n_runs, dev->cu_count)), dim3(256), 0, dev->stream, volume,
                       g.dims[0], g.dims[1], g.dims[2], t.nb[0], t.nb[1], t.n_runs, (float4*)t.vol, (float4*)nullptr);
    hipLaunchKernelGGL(train_forward_blocked_kernel, dim3(patch_grid((g.W + 7) / 8, (g.H + 7) / 8, n)), dim3(256), lds,
                       dev->stream, train_scene(g), train_brick(g, t), dc, (const float4*)tf, (float4*)out_rgba,
                       out_depth, (double*)ws, g.ws_stride, g.W, g.H, n);
    DPR_HIP(hipGetLastError());
    return scratch_end(dev);
  }
  hipLaunchKernelGGL(train_forward_kernel, grid, dim3(256), lds, dev->stream, g, dc, volume, (const float4*)tf,
                     (float4*)out_rgba, out_depth, (double*)ws, tx, tx * ty);
  DPR_HIP(hipGetLastError());
  return DPR_OK;
}

dpr_status dpr_render_backward(dpr_device dev, const float* volume, const int64_t dims[3], const float* tf,
                               int32_t n_tf, float lo, float hi, float density, const dpr_render_params* prm,
                               const dpr_camera* cams, int32_t n, const float* grad_rgba, const void* ws,
                               size_t ws_bytes, float* grad_volume, float* grad_tf) {
  if (!dev || !volume || !tf || !grad_rgba || !ws || !grad_volume || !grad_tf)
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_backward: NULL argument");
  dpr_status s = check_train(dims, cams, n, prm, n_tf, lo, hi, density);
  if (s != DPR_OK) return s;
  TrainG g = make_train(dims, cams, n, prm, n_tf, lo, hi, density);
  size_t need = (size_t)n * g.W * g.H * g.ws_stride * sizeof(double);
  if (ws_bytes < need)
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_backward: workspace %zu < %zu bytes", ws_bytes, need);
  CamG* dc = nullptr;
  if ((s = cam_table(dev, cams, n, &dc)) != DPR_OK) return s;
  const int tx = (g.W + 15) / 16, ty = (g.H + 15) / 16;
  dim3 grid((unsigned)(tx * ty * n));
  if (!dev->tf_grad64 && (s = dev_alloc((void**)&dev->tf_grad64, 4 * kMaxTF * sizeof(double) + 9 * kHeadStride * sizeof(int),
                                           "transfer-function gradient sums")) != DPR_OK)
    return s;
  const int nt = 4 * n_tf;
  int* heads = (int*)(dev->tf_grad64 + 4 * kMaxTF);
  if ((s = scratch_begin(dev)) != DPR_OK) return s;
  TrainBlocks t;
  const bool blocked = !train_small(g) && !train_coarse(g, cams) && train_blocks(dev, g, true, t);
  // Rays in pieces where whole ones would leave the chip's waves idle: up to kPieceTiles
  // tiles, while the intervals' colours take no more than kPieceBytes.
  TrainPieces pieces;
  float4* col = nullptr;
  uint2* list = nullptr;
  const int tiles_x = (g.W + 7) / 8, tiles_y = (g.H + 7) / 8;
  const long long tiles = (long long)tiles_x * tiles_y * n;
  const int max_chunks = g.ws_stride - 1;
  const size_t col_bytes = (size_t)n * g.W * g.H * max_chunks * sizeof(float4);
  if (blocked && tiles <= kPieceTiles && col_bytes <= kPieceBytes) {
    col = (float4*)train_buffer(dev, 2, col_bytes + (size_t)tiles * 4 * max_chunks * sizeof(uint2));
    if (col) {
      list = (uint2*)((char*)col + col_bytes);
      pieces.chunks = max_chunks;
      pieces.col = col;
      pieces.list = list;
      pieces.count = heads + 8 * kHeadStride;
    }
  }
  const int quarters = tiles * max_chunks <= kQuarterPieces;
  const int waves = list ? kBwWavesSmall : kBwWaves;
  const int queues = list ? 1 : 8;
  const int blocks = std::max(queues, dev->cu_count / queues * queues);
  hipLaunchKernelGGL(fill_f64_kernel, dim3((nt + 255) / 256), dim3(256), 0, dev->stream, dev->tf_grad64, nt, heads,
                     blocks / queues * waves);
  if (blocked) {
    const dim3 rgrid(run_grid(t.n_runs, dev->cu_count));
    hipLaunchKernelGGL(block_volume_kernel, rgrid, dim3(256), 0, dev->stream, volume, g.dims[0], g.dims[1], g.dims[2],
                       t.nb[0], t.nb[1], t.n_runs, (float4*)t.vol, (float4*)t.grad);
    if (list)
      hipLaunchKernelGGL(train_chunk_kernel, dim3(patch_grid(tiles_x, tiles_y, n), pieces.chunks), dim3(256),
                         2 * sizeof(float4) * (size_t)n_tf, dev->stream, train_scene(g), train_brick(g, t), dc,
                         (const float4*)tf, (const double*)ws, g.ws_stride, g.W, g.H, n, pieces.chunks, quarters, col, list,
                         heads + 8 * kHeadStride);
    // table records, copies of the table gradient (each 8 bytes an entry and channel), and the
    // rest for the waves' patches
    const int left = kBwLds - 32 * n_tf;
    int reps = kTfRep;
    while (reps > 1 && left - reps * 32 * n_tf < waves * 960 * 8) reps >>= 1;
    const int cells = std::min(2048, (left - reps * 32 * n_tf) / (waves * 8));
    const size_t blds = 32 * (size_t)n_tf * (1 + reps) + (size_t)waves * cells * 8;
    // (more dynamic LDS than a launch takes by default)
    DPR_HIP(hipFuncSetAttribute((const void*)train_backward_blocked_kernel,
                                hipFuncAttributeMaxDynamicSharedMemorySize, kBwLds));
    static_assert((kBwLds - 64 * kMaxTF) / (kBwWaves * 8) >= kBwMinCells, "one ray's patch fits with the largest table");
    hipLaunchKernelGGL(train_backward_blocked_kernel, dim3(blocks), dim3(64 * waves), blds, dev->stream,
                       train_scene(g), train_brick(g, t), dc, (const float4*)tf, (const float4*)grad_rgba,
                       (const double*)ws, g.ws_stride, t.grad, dev->tf_grad64, heads, g.W, g.H, n, reps, cells,
                       pieces);
    hipLaunchKernelGGL(add_blocked_kernel, rgrid, dim3(256), 0, dev->stream, (const float4*)t.grad, g.dims[0],
                       g.dims[1], g.dims[2], t.nb[0], t.nb[1], t.n_runs, grad_volume);
  } else {
    int reps = kTfRep;  // as many copies as 64 KiB hold beside the table
    while (32 * n_tf * (1 + reps) > 64 * 1024) reps >>= 1;
    hipLaunchKernelGGL(train_backward_kernel, grid, dim3(256), 32 * (size_t)n_tf * (1 + reps), dev->stream, g, dc,
                       volume, (const float4*)tf, (const float4*)grad_rgba, (const double*)ws, grad_volume,
                       dev->tf_grad64, tx, tx * ty, reps);
  }
  hipLaunchKernelGGL(add_f64_to_f32_kernel, dim3((nt + 255) / 256), dim3(256), 0, dev->stream, dev->tf_grad64,
                     grad_tf, nt);
  DPR_HIP(hipGetLastError());
  return scratch_end(dev);
}

}  // extern "C"
