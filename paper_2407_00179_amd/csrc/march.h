// Resumable per-ray emission-absorption march through one brick.
//
// Sample points advance in exact 32.32 fixed point, so the point of segment s is the
// same integer whichever way the ray got there: by one lane or four, in one call or in
// budgeted slices (persistent kernel), with or without skipping.
//
// Iso-surfaces (ISO): the sides (v >= v_iso) of consecutive samples are compared
// at every lattice point the brick owns (those in [t_in, t_out)); the first change
// of side is an opaque surface, lit at the linearly interpolated crossing with the
// gradient of the trilinear patch there, and closes the ray.  A macrocell is then
// skipped only when its majorant is 0, its value range lies on one side of v_iso,
// and that side is the previous sample's (classes encoded in the majorant: 0 below,
// -1 at or above, positive: sample it).
#pragma once

#include "device_common.h"

namespace dpr {

constexpr double kFix = 4294967296.0;  // 2^32

// A ray clipped to a brick.
struct RaySetup {
  int64_t p[3];          // sample point of segment s0, 32.32 fixed point (global voxel-centre coords)
  int64_t dp[3];         // advance per segment
  double t_in, t_out;    // clipped parametric range (world units)
  int s0, s1;            // first and last segment
  float dl_first, dl_last;  // D * clipped length of the first / last segment
};

constexpr int kIsoSide = 1, kIsoPair = 2, kIsoKnown = 4;

// Clip the ray against the brick's owned box and set up its march.  Returns false
// on a miss (zero-length chords included).
__device__ __forceinline__ bool ray_begin(const SceneG& sc, const BrickG& b, const double o[3], const double d[3],
                                          RaySetup& r) {
  double lo[3], hi[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    lo[a] = b.olo[a] * sc.h;
    hi[a] = b.ohi[a] * sc.h;
  }
  if (!clip_box(o, d, lo, hi, r.t_in, r.t_out)) return false;
  const double dt = sc.dt;
  int s0 = (int)floor(r.t_in / dt);
  int s1 = (int)ceil(r.t_out / dt) - 1;
  // lengths of the clipped end segments; a non-positive one is dropped
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
  // (s1 < s0 only through rounding at a vanishing chord: a hit with no samples)
  r.s0 = s0;
  r.s1 = s1;
  r.dl_first = sc.density * (float)lf;
  r.dl_last = sc.density * (float)ll;
  const double tm = (s0 + 0.5) * dt;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double dv = d[a] * sc.inv_h;
    const double g = fma(tm, dv, o[a] * sc.inv_h - 0.5);
    r.p[a] = __double2ll_rn(g * kFix);
    r.dp[a] = __double2ll_rn(dt * dv * kFix);
  }
  return true;
}

// Voxel index (stored, relative to the brick) and fraction along one axis of a
// 32.32 fixed-point sample point, clamped to the global domain [0, n - 1].
__device__ __forceinline__ int axis_index(int64_t p, int n, int slo, int sdim) {
  const int hi = (int)(p >> 32);
  const int i0 = min(max(hi, 0), n - 2);
  // commit guarantees i0 - slo lies in [0, sdim - 2]; the clamp only guards memory
  return min(max(i0 - slo, 0), sdim - 2);
}
__device__ __forceinline__ float axis_frac(int64_t p, int n) {
  const int hi = (int)(p >> 32);
  const float fr = (float)(uint32_t)(p & 0xffffffffll) * (1.0f / 4294967296.0f);
  return (hi < 0) ? 0.f : ((hi > n - 2) ? 1.f : fr);
}

template <typename T>
struct Gather {
  float v[8];
  float fx, fy, fz;
};

// The loaded voxels of a sample's 8-voxel footprint, before decoding (FP16: the
// four voxel pairs as loaded), so a request in flight holds as few registers as
// possible.
template <typename T, bool WIDE = false>
struct Voxels {  // FP32, 32- and 64-bit offsets
  float v[8];
};
template <>
struct Voxels<__half, false> {
  uint32_t c[4];
};
// FP16 voxels without pairs: what lies from voxel x on and, where x ends a 4-voxel run, voxel
// x + 1 from where the next run is.  They are put together only where the sample is used,
// which is what waits for the loads: merged when requested, the march of an 8 GB brick at
// 3840 x 2160 waited for each sample's voxels before it went on (9.7 ms with its commit; 8.7).
template <>
struct Voxels<__half, true> {
  uint32_t c[4], next[4];
  uint32_t sel;  // byte selector of the pair
};
__device__ __forceinline__ uint32_t voxel_pair(const Voxels<__half, false>& g, int k) { return g.c[k]; }
__device__ __forceinline__ uint32_t voxel_pair(const Voxels<__half, true>& g, int k) {
  return __builtin_amdgcn_perm(g.next[k], g.c[k], g.sel);
}

// Load the 8 voxels around base voxel (lx, ly, lz) (stored indices).  Byte offsets from
// the brick base: 32-bit sums for bricks below 4 GiB; WIDE (the blocked array is 4 GiB
// or more, or 64-bit offsets were asked for): 32-bit element indices (a brick holds
// fewer than 2^32 elements), widened and scaled once per load.  Either way the loads
// are global loads.  An FP16 brick is stored as voxel pairs when addressed with 32-bit
// offsets and as 2-byte voxels when addressed with 64-bit offsets (the commit picks
// the layout and the addressing together).
//
// In two parts.  Where an x-pair can straddle two 4-voxel runs, the lanes at a run's end read
// their voxels lx + 1 on their own (load_run_ends), and only if a wave has such lanes.  A
// wave waits for a sample by the number of loads issued after it, and the compiler has to
// take the smallest possible: with a sample's second part between the next one's request and
// its use, waiting for a sample meant waiting for most of the next one.  So a march asks
// for the next sample's first part, waits for the present one (arrived), asks for the
// next one's second part and goes on: eight partial frames of 256^3 FP32 bricks at 1024^2
// 1.23 -> 0.99 ms, four frames of all of them 2.24 -> 2.04 ms.  (Requests two samples ahead
// instead of one are slower: 1.12 and 2.14 ms.)
struct Footed {
  Foot f;
  int lx;
};
template <typename T, bool WIDE>
constexpr int kOffsetShift = WIDE ? 0 : 2;  // footprint's SH
template <typename T, bool WIDE>
__device__ __forceinline__ auto byte_offset(uint32_t e) {
  if constexpr (WIDE)
    return (uint64_t)e * sizeof(T);
  else
    return e;
}
template <typename T, bool WIDE, bool UNI>
__device__ __forceinline__ Footed load_footprint(const BrickG& b, int lx, int ly, int lz, Voxels<T, WIDE>& g) {
  using GC = const char __attribute__((address_space(1)))*;
  const Foot f = footprint<kOffsetShift<T, WIDE>, UNI>(b, lx, ly, lz, in_block_x(lx));
  const uint32_t a[4] = {f.a, f.a + f.dy, f.a + f.dz, f.a + f.dz + f.dy};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const auto o = byte_offset<T, WIDE>(a[k]);
    if constexpr (sizeof(T) == 4) {
      // voxel lx + 1 follows voxel lx in memory unless lx ends a 4-voxel x-run, so each
      // x-pair is one 8-byte load
      const float2 c = load_pair_f32(b.data, o);
      g.v[2 * k] = c.x;
      g.v[2 * k + 1] = c.y;
    } else if constexpr (WIDE) {
      // FP16 voxels (2 bytes: the layout of bricks addressed with 64-bit offsets): likewise
      typedef uint32_t U2 __attribute__((aligned(2)));
      g.c[k] = *(const U2 __attribute__((address_space(1)))*)((GC)b.data + o);
    } else {
      // FP16 voxel pairs (4 bytes, the layout of bricks below 4 GiB): each element
      // holds the voxels (x, x + 1), one aligned 4-byte load per pair
      g.c[k] = *(const uint32_t __attribute__((address_space(1)))*)((GC)b.data + o);
    }
  }
  return {f, lx};
}
__device__ __forceinline__ void load_run_ends(const BrickG&, const Footed&, Voxels<__half, false>&) {}
template <typename T, bool WIDE>
__device__ __forceinline__ void load_run_ends(const BrickG& b, const Footed& p, Voxels<T, WIDE>& g) {
  if constexpr (sizeof(T) == 2) {
    g.sel = 0x03020100u;
    // (not read unless lx ends a run)
    asm("" : "=v"(g.next[0]), "=v"(g.next[1]), "=v"(g.next[2]), "=v"(g.next[3]));
  }
  if ((p.lx & 3) == 3) {
    // from element 3 of a run to the block's second run, or to the next block
    constexpr int SH = kOffsetShift<T, WIDE>;
    const uint32_t e = p.f.a + ((p.lx & 4) ? (512u - 67u) << SH : (64u - 3u) << SH);
    const uint32_t a[4] = {e, e + p.f.dy, e + p.f.dz, e + p.f.dz + p.f.dy};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const auto o = byte_offset<T, WIDE>(a[k]);
      if constexpr (sizeof(T) == 4)
        g.v[2 * k + 1] = load_voxel_b<T>(b.data, o);
      else
        g.next[k] = *(const uint16_t __attribute__((address_space(1)))*)(
            (const char __attribute__((address_space(1)))*)b.data + o);
    }
    if constexpr (sizeof(T) == 2) g.sel = 0x05040100u;
  }
}
// Waits for a sample's voxels.
template <bool WIDE>
__device__ __forceinline__ void arrived(Voxels<float, WIDE>& g) {
  asm volatile("" : "+v"(g.v[0]), "+v"(g.v[1]), "+v"(g.v[2]), "+v"(g.v[3]), "+v"(g.v[4]), "+v"(g.v[5]), "+v"(g.v[6]),
               "+v"(g.v[7]));
}
__device__ __forceinline__ void arrived(Voxels<__half, false>& g) {
  asm volatile("" : "+v"(g.c[0]), "+v"(g.c[1]), "+v"(g.c[2]), "+v"(g.c[3]));
}
__device__ __forceinline__ void arrived(Voxels<__half, true>& g) {
  asm volatile("" : "+v"(g.c[0]), "+v"(g.c[1]), "+v"(g.c[2]), "+v"(g.c[3]), "+v"(g.next[0]), "+v"(g.next[1]),
               "+v"(g.next[2]), "+v"(g.next[3]));
}

// Load the 8 voxels around a sample point.
template <typename T, bool WIDE>
__device__ __forceinline__ void load_voxels(const SceneG& sc, const BrickG& b, const int64_t p[3], Voxels<T, WIDE>& g) {
  load_run_ends(b,
                         load_footprint<T, WIDE, false>(b, axis_index(p[0], sc.dims[0], b.slo[0], b.sdim[0]),
                                                        axis_index(p[1], sc.dims[1], b.slo[1], b.sdim[1]),
                                                        axis_index(p[2], sc.dims[2], b.slo[2], b.sdim[2]), g),
                         g);
}

// The 8 footprint voxels as FP32: (x0, x1) at (y0, z0), (y1, z0), (y0, z1), (y1, z1).
template <typename T, bool WIDE>
__device__ __forceinline__ void decode_voxels(const Voxels<T, WIDE>& g, float v[8]) {
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = g.v[k];
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float2 c = unpack_pair_f16(voxel_pair(g, k));
      v[2 * k] = c.x;
      v[2 * k + 1] = c.y;
    }
  }
}

// Trilinear fractions of a sample point.
__device__ __forceinline__ void sample_frac(const SceneG& sc, const int64_t p[3], float& fx, float& fy, float& fz) {
  fx = axis_frac(p[0], sc.dims[0]);
  fy = axis_frac(p[1], sc.dims[1]);
  fz = axis_frac(p[2], sc.dims[2]);
}

// Gather the 8 voxels around a sample point and its trilinear fractions.
template <typename T, bool WIDE>
__device__ __forceinline__ void gather(const SceneG& sc, const BrickG& b, const int64_t p[3], Gather<T>& g) {
  sample_frac(sc, p, g.fx, g.fy, g.fz);
  Voxels<T, WIDE> raw;
  load_voxels<T, WIDE>(sc, b, p, raw);
  decode_voxels(raw, g.v);
}

template <typename T>
__device__ __forceinline__ float trilerp(const Gather<T>& g) {
  const float c00 = fmaf(g.fx, g.v[1] - g.v[0], g.v[0]), c01 = fmaf(g.fx, g.v[3] - g.v[2], g.v[2]);
  const float c10 = fmaf(g.fx, g.v[5] - g.v[4], g.v[4]), c11 = fmaf(g.fx, g.v[7] - g.v[6], g.v[6]);
  const float c0 = fmaf(g.fy, c01 - c00, c00), c1 = fmaf(g.fy, c11 - c10, c10);
  return fmaf(g.fz, c1 - c0, c0);
}


// ---------------------------------------------------------------- the march
// L lanes per ray, one or the four of a DPP quad; each takes every L-th sample.
//
// A ray is a serial chain: with one lane per ray a launch takes at least its longest
// ray's samples times the time a wave needs for one, and its last rays leave most of
// the chip idle.  With four lanes the chain is a quarter as long, and a wave's loads
// cover 16 rays over two voxels of depth, which is fewer cache lines than 64 rays at
// one depth.  Per four samples the lanes gather, interpolate and look up their own
// one; the optical depth before each is a scan over the quad, and a lane keeps the colour
// sum of its own samples, added up at the ray's end.  One lane per ray works in the same
// groups of four samples with the same sums, so one and four lanes give the same bits.
// (Sums in sample order in every lane of the quad, on broadcast values, take 20 more
// instructions a sample, a sixth of all: 27 FP16 bricks, four cameras at 2048^2, 11.7 ms
// against 10.5; 512^3 FP32, four frames at 1024^2, 2.03 against 1.95.)  The batched renderer uses four lanes (times in
// k_batch.hip), the plain launch, which also counts a ray's samples, one.
//
// The lattice is walked in trips of R steps of L samples.  A gather buffer per step in
// flight, the next NB - 1 steps' voxels requested ahead; the majorant of the next
// trip's first samples is requested with them.  (One lane skips whole groups of four only.)  If every lane's next sample lies in an
// empty macrocell the steps that all of them make inside their own are skipped (a
// sample of zero opacity changes nothing, so any part of a run may be skipped or
// sampled with the same bits).  Steps past a ray's last segment, or after it ended,
// have length 0, which leaves every sum as it is, so a trip's body has no exits.
//
// Every branch condition is the same in the lanes of a ray.
constexpr int kRayDone = -(1 << 29);  // LaneRay::m of a ray that ended early

template <int L>
struct LaneCfg {
  static constexpr int NB = 2, R = L == 4 ? 2 : 4;
};

struct LaneRay {
  int64_t q[3];  // this lane's next sample point, 32.32 fixed point, in stored voxel indices of the brick
  int64_t d[3];  // advance of L segments
  double acc;    // optical depth before the next L samples
  float tr;      // transmittance after this lane's last sample (the last lane's: after the last L samples)
  float cr[4], cg[4], cb[4];  // colour sums: (four lanes) [0], of this lane's samples, (one lane) of every fourth
  float dl_cur, dl_last;  // D * length of this lane's next segment unless it is the ray's last / of the last
  float t_in;
  int m;         // last segment minus this lane's next one
  int n;         // (one lane) logical samples processed, once the ray has ended
  float pv;      // iso-surfaces: value of the sample before q
  int pst;       // iso-surfaces: bit 0 side of that sample, bit 1 the next sample closes a tested
                 // pair, bit 2 pv holds the value
};

template <int CTRL>
__device__ __forceinline__ float quad_perm(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int quad_perm(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int K>
__device__ __forceinline__ float quad_bcast(float v) {
  return quad_perm<K * 0x55>(v);
}
template <int K>
__device__ __forceinline__ double quad_bcast(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)quad_perm<K * 0x55>((int)(uint32_t)u);
  const uint32_t hi = (uint32_t)quad_perm<K * 0x55>((int)(uint32_t)(u >> 32));
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ float masked(float v, int mask) { return __int_as_float(__float_as_int(v) & mask); }
__device__ __forceinline__ float quad_max(float v) {
  v = fmaxf(v, quad_perm<0xB1>(v));
  return fmaxf(v, quad_perm<0x4E>(v));
}
__device__ __forceinline__ int quad_min(int v) {
  v = min(v, quad_perm<0xB1>(v));
  return min(v, quad_perm<0x4E>(v));
}

// A ray's colour: its four sums, in the same order for one lane and four.
template <int L>
__device__ __forceinline__ float4 ray_rgba(const LaneRay& r) {
  auto sum = [](const float c[4]) {
    if constexpr (L == 1) return (c[0] + c[1]) + (c[2] + c[3]);
    float v = c[0];
    v += quad_perm<0xB1>(v);
    return v + quad_perm<0x4E>(v);
  };
  return make_float4(sum(r.cr), sum(r.cg), sum(r.cb), 1.f - r.tr);
}

// min(max(i, 0), top) for a wave-uniform top >= 0
__device__ __forceinline__ int clamp_index(int i, int top) {
  int r;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(r) : "v"(i), "s"(top));
  return r;
}

// Base voxel and fraction along one axis of a point in stored voxel indices, clamped
// to the stored range [0, top + 1] (top = stored extent - 2).  The commit guarantees
// that a ray's own samples leave the stored range only through a global face, where
// this is the clamp of the sampling rule.
__device__ __forceinline__ int local_axis(int64_t p, int top, float& f) {
  const int hi = (int)(p >> 32);
  const int i = clamp_index(hi, top);
  // i == hi: the fraction; hi below or above the range: 0 or 1
  f = __builtin_amdgcn_fmed3f(fmaf((float)(uint32_t)p, 1.0f / 4294967296.0f, (float)(hi - i)), 0.f, 1.f);
  return i;
}

// A requested sample: its voxels and trilinear fractions.
template <typename T, bool WIDE = false>
struct Sample {
  Voxels<T, WIDE> v;
  float fx, fy, fz;
};

// Interpolate a requested sample (the lerps of trilerp).  FP16: the difference of a
// pair's halves is one mixed-precision FMA, exact like the FP32 difference of the
// converted halves, and the halves themselves are FMA operands.
__device__ __forceinline__ float pair_diff(uint32_t c) {
  float d;
  asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(c));
  return d;
}
__device__ __forceinline__ float lerp_yz(float c00, float c01, float c10, float c11, float fy, float fz) {
  const float c0 = fmaf(fy, c01 - c00, c00), c1 = fmaf(fy, c11 - c10, c10);
  return fmaf(fz, c1 - c0, c0);
}
template <bool WIDE>
__device__ __forceinline__ float sample_value(const Sample<float, WIDE>& s) {
  const float* v = s.v.v;
  return lerp_yz(fmaf(s.fx, v[1] - v[0], v[0]), fmaf(s.fx, v[3] - v[2], v[2]), fmaf(s.fx, v[5] - v[4], v[4]),
                 fmaf(s.fx, v[7] - v[6], v[6]), s.fy, s.fz);
}
template <bool WIDE>
__device__ __forceinline__ float sample_value(const Sample<__half, WIDE>& s) {
  auto lerp_x = [&](uint32_t c) {
    return fmaf(s.fx, pair_diff(c), __half2float(__ushort_as_half((unsigned short)(c & 0xffffu))));
  };
  return lerp_yz(lerp_x(voxel_pair(s.v, 0)), lerp_x(voxel_pair(s.v, 1)), lerp_x(voxel_pair(s.v, 2)),
                 lerp_x(voxel_pair(s.v, 3)), s.fy, s.fz);
}

// Request the 8 voxels around a point in stored voxel indices of a wave-uniform brick: the
// first part; all.
template <typename T, bool WIDE>
__device__ __forceinline__ Footed request_first(const BrickG& b, int64_t x, int64_t y, int64_t z, Sample<T, WIDE>& g) {
  const int lx = local_axis(x, b.sdim[0] - 2, g.fx);
  const int ly = local_axis(y, b.sdim[1] - 2, g.fy);
  const int lz = local_axis(z, b.sdim[2] - 2, g.fz);
  return load_footprint<T, WIDE, true>(b, lx, ly, lz, g.v);
}
template <typename T, bool WIDE>
__device__ __forceinline__ void request(const BrickG& b, int64_t x, int64_t y, int64_t z, Sample<T, WIDE>& g) {
  load_run_ends(b, request_first<T, WIDE>(b, x, y, z, g), g.v);
}

// Set up lane k's part of a ray: ray_begin, then the points of segments s0 + k,
// s0 + k + L, ... relative to the brick's first stored voxel (exact integers).  For
// iso-surfaces, the pair at the brick entry: when the first processed segment starts
// exactly at t_in its lattice point is this brick's, and the sample half a step before
// the entry opens the pair.
template <typename T, bool WIDE, bool ISO, int L>
__device__ __forceinline__ bool lane_begin(const SceneG& sc, const BrickG& b, const double o[3], const double d[3],
                                           int k, LaneRay& r) {
  RaySetup f;
  if (!ray_begin(sc, b, o, d, f)) return false;
  int64_t p[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    p[a] = f.p[a] - ((int64_t)b.slo[a] << 32);
    r.q[a] = p[a] + (int64_t)k * f.dp[a];
    r.d[a] = L * f.dp[a];
  }
  r.acc = 0.0;
  r.tr = 1.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) r.cr[i] = r.cg[i] = r.cb[i] = 0.f;
  r.t_in = (float)f.t_in;
  r.m = f.s1 - f.s0 - k;
  r.n = f.s1 - f.s0 + 1;
  r.dl_cur = k == 0 ? f.dl_first : sc.density * sc.dt_f;
  r.dl_last = f.s0 == f.s1 ? f.dl_first : f.dl_last;
  if constexpr (ISO) {
    r.pv = 0.f;
    r.pst = 0;
    if ((double)f.s0 * sc.dt >= f.t_in) {
      Sample<T, WIDE> s;
      request<T, WIDE>(b, p[0] - f.dp[0], p[1] - f.dp[1], p[2] - f.dp[2], s);
      r.pv = sample_value(s);
      r.pst = kIsoPair | kIsoKnown | (r.pv >= sc.iso ? kIsoSide : 0);
    }
  }
  return true;
}

// The opaque surface between samples s - 1 and s (value vs; q: the point of sample s,
// dq: advance per segment): crossing by linear interpolation, normal = gradient of the
// trilinear patch there, colour = TF colour at v_iso * (k_a + k_d |cos|).  Adds it to
// the colour behind transmittance tr.
template <typename T, bool WIDE>
__device__ __forceinline__ void iso_hit(const SceneG& sc, const BrickG& b, const float4* tfr, const int64_t q[3],
                                        const int64_t dq[3], float vs, int pst, float pv, float tr, float& cr,
                                        float& cg, float& cb) {
  const int64_t qp[3] = {q[0] - dq[0], q[1] - dq[1], q[2] - dq[2]};
  float vp = pv;
  if (!(pst & kIsoKnown)) {  // the previous sample was skipped: its value now
    Sample<T, WIDE> g;
    request<T, WIDE>(b, qp[0], qp[1], qp[2], g);
    vp = sample_value(g);
  }
  const float f = (sc.iso - vp) / (vs - vp);
  int64_t qh[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) qh[a] = qp[a] + __double2ll_rn((double)f * (double)dq[a]);
  Sample<T, WIDE> g;
  request<T, WIDE>(b, qh[0], qh[1], qh[2], g);
  float v[8];
  decode_voxels(g.v, v);
  // d/dx, d/dy, d/dz of the patch: the edge differences, interpolated in the other two axes
  const float x0 = fmaf(g.fy, (v[3] - v[2]) - (v[1] - v[0]), v[1] - v[0]);
  const float x1 = fmaf(g.fy, (v[7] - v[6]) - (v[5] - v[4]), v[5] - v[4]);
  const float gx = fmaf(g.fz, x1 - x0, x0);
  const float y0 = fmaf(g.fx, (v[3] - v[1]) - (v[2] - v[0]), v[2] - v[0]);
  const float y1 = fmaf(g.fx, (v[7] - v[5]) - (v[6] - v[4]), v[6] - v[4]);
  const float gy = fmaf(g.fz, y1 - y0, y0);
  const float z0 = fmaf(g.fx, (v[5] - v[1]) - (v[4] - v[0]), v[4] - v[0]);
  const float z1 = fmaf(g.fx, (v[7] - v[3]) - (v[6] - v[2]), v[6] - v[2]);
  const float gz = fmaf(g.fy, z1 - z0, z0);
  // the ray direction is parallel to the per-segment advance.  Every product and
  // sum is spelled out (fmaf, __fmul_rn): left to contraction, the compiler may
  // associate these sums differently in different kernels, and the skip and
  // no-skip marches would then differ in the last bit
  const float dx = (float)dq[0], dy = (float)dq[1], dz = (float)dq[2];
  const float nn = fmaf(gz, gz, fmaf(gy, gy, __fmul_rn(gx, gx)));
  const float dd = fmaf(dz, dz, fmaf(dy, dy, __fmul_rn(dx, dx)));
  const float dot = fmaf(gz, dz, fmaf(gy, dy, __fmul_rn(gx, dx)));
  const float cosv = nn > 0.f ? fabsf(dot) / sqrtf(__fmul_rn(nn, dd)) : 1.f;
  float x = (sc.iso - sc.tf_lo) * sc.tf_scale;
  x = fminf(fmaxf(x, 0.f), (float)(sc.ntf - 1));
  const int j = min((int)x, sc.ntf - 2);
  const float w = x - (float)j;
  const float4 tb = tfr[2 * j], ts = tfr[2 * j + 1];
  const float lit = fmaf(sc.iso_kd, fminf(cosv, 1.f), sc.iso_ka);
  cr = fmaf(tr, __fmul_rn(fmaf(w, ts.x, tb.x), lit), cr);
  cg = fmaf(tr, __fmul_rn(fmaf(w, ts.y, tb.y), lit), cg);
  cb = fmaf(tr, __fmul_rn(fmaf(w, ts.z, tb.z), lit), cb);
}

// RAW: the table's values are not known to be finite (a sample of no optical depth adds
// nothing, whatever its colour).
// March until the ray ends (true) or max_trips trips have passed.  b is wave-uniform.
template <typename T, bool SKIP, bool WIDE, bool ISO, int L, bool RAW = false>
__device__ __forceinline__ bool lane_advance(const SceneG& sc, const BrickG& b, const float4* tfr, LaneRay& r,
                                             int max_trips) {
  static_assert(L == 1 || L == 4, "one lane, or a DPP quad");
  constexpr int NB = LaneCfg<L>::NB, R = LaneCfg<L>::R;
  static_assert(R % NB == 0 && NB >= 2, "a trip ends with the buffers as it found them");
  static_assert(L == 4 || R == 4, "one lane: a trip is a group of four samples");
  const int lane = threadIdx.x & 63, k = lane & (L - 1);
  const int from1 = k >= 1 ? -1 : 0, from2 = k >= 2 ? -1 : 0;
  const float x_max = (float)(sc.ntf - 1);
  const float Ddt = sc.density * sc.dt_f;
  int64_t q0 = r.q[0], q1 = r.q[1], q2 = r.q[2];
  const int64_t d0 = r.d[0], d1 = r.d[1], d2 = r.d[2];
  double acc = r.acc;
  constexpr int NC = L == 1 ? 4 : 1;
  float tr = r.tr, cr[NC], cg[NC], cb[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    cr[i] = r.cr[i];
    cg[i] = r.cg[i];
    cb[i] = r.cb[i];
  }
  float t4[NC], r4[NC], g4[NC], b4[NC];  // (one lane) the group's optical depths and colours
  float dl_cur = r.dl_cur;
  int m = r.m;
  int pst = ISO ? r.pst : 0;
  float pv = ISO ? r.pv : 0.f, vh = 0.f;
  int hit = -1;  // iso-surfaces: L * (step of the trip) + (lane of the ray) of the sample behind the surface

  // the next L samples, in order; i: step of the trip
  auto step = [&](const Sample<T, WIDE>& s, int i) {
    const float v = sample_value(s);
    const float x = __builtin_amdgcn_fmed3f((v - sc.tf_lo) * sc.tf_scale, 0.f, x_max);
    // (the last record has no slope: x = ntf - 1 gives its entry)
    const int j = (int)x;
    const float w = __builtin_amdgcn_fractf(x);
    const float4 tb = tfr[2 * j], ts = tfr[2 * j + 1];
    float Dl = m > 0 ? dl_cur : (m == 0 ? r.dl_last : 0.f);
    dl_cur = Ddt;
    int surf = L;  // lane of the first sample behind the surface
    if constexpr (ISO) {
      // a change of side against the sample before ends the ray on the surface
      const int side = v >= sc.iso ? kIsoSide : 0;
      int prev = pst;
      if constexpr (L == 4) {
        const int ps = quad_perm<0x90>(side);
        prev = k == 0 ? pst : (ps | kIsoPair);
      }
      const bool cross = m >= 0 && (prev & kIsoPair) && side != (prev & kIsoSide);
      bool hit_now = L == 1 ? cross || hit >= 0 : cross;
      if constexpr (L == 4) {
        const uint64_t cm = __ballot(cross);
        const uint32_t nib = cm ? (uint32_t)(cm >> (lane & 60)) & 15u : 0u;
        hit_now = nib != 0;
        if (hit_now) surf = __ffs(nib) - 1;
      }
      if (hit_now) {
        if constexpr (L == 1) {
          surf = 0;
          if (hit < 0) vh = v;
        } else {
          vh = __shfl(v, (lane & 60) + surf);
          const float vb = __shfl(v, (lane & 60) + max(surf - 1, 0));
          if (surf > 0) {
            pv = vb;
            pst |= kIsoKnown;
          }
        }
        if (k >= surf) Dl = 0.f;  // no emission from the crossing segment on
        if (L == 4 || hit < 0) hit = L * i + surf;
      } else if (hit < 0) {
        pst = kIsoPair | kIsoKnown | (L == 4 ? quad_perm<0xFF>(side) : side);
        pv = L == 4 ? quad_bcast<3>(v) : v;
      }
    }
    m -= L;
    const float tau = fmaxf(Dl * fmaf(w, ts.w, tb.w), 0.f);
    float r0 = fmaf(w, ts.x, tb.x), g0 = fmaf(w, ts.y, tb.y), b0 = fmaf(w, ts.z, tb.z);
    if (RAW && !(tau > 0.f)) r0 = g0 = b0 = 0.f;
    if constexpr (L == 1) {
      t4[i] = tau;
      r4[i] = r0;
      g4[i] = g0;
      b4[i] = b0;
      if (i < 3) return;
      const double t01 = (double)t4[1] + (double)t4[0], t12 = (double)t4[2] + (double)t4[1],
                   t23 = (double)t4[3] + (double)t4[2];
      const double a4[4] = {acc + (double)t4[0], acc + t01, acc + (t12 + (double)t4[0]), acc + (t23 + t01)};
      float tn[4];
      int first = 4;  // first sample after which the ray is opaque enough
#pragma unroll
      for (int n = 3; n >= 0; --n) {
        tn[n] = __expf(-(float)a4[n]);
        if (tn[n] <= sc.ert_t) first = n;
      }
      float before = tr;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const float wgt = n > first ? 0.f : before - tn[n];
        before = tn[n];
        cr[n] = fmaf(wgt, r4[n], cr[n]);
        cg[n] = fmaf(wgt, g4[n], cg[n]);
        cb[n] = fmaf(wgt, b4[n], cb[n]);
        if (n == 0 || n <= first) {
          acc = a4[n];
          tr = tn[n];
        }
      }
      if (ISO && first < 4 && hit > first) hit = -1;  // it ended before the surface
      const int end = min(first, ISO && hit >= 0 ? hit : 4);
      if (end < 4 && m > kRayDone / 2) {
        r.n -= m + 4 - end;
        m = kRayDone;
      }
    } else {
      // optical depth after this lane's sample: a scan over the quad
      const float t1 = masked(quad_perm<0x90>(tau), from1);
      const double s1 = (double)tau + (double)t1;
      const uint64_t u = (uint64_t)__double_as_longlong(s1);
      const uint32_t lo = (uint32_t)(quad_perm<0x40>((int)(uint32_t)u) & from2);
      const uint32_t hi = (uint32_t)(quad_perm<0x40>((int)(uint32_t)(u >> 32)) & from2);
      double a = acc + (s1 + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo)));
      float tn = __expf(-(float)a);
      // transmittance before it: the previous lane's, or what lane 3 left four samples ago
      float wgt = quad_perm<0x93>(k == 3 ? tr : tn) - tn;
      const uint64_t term = __ballot(tn <= sc.ert_t);
      if (term) {  // some ray of the wave ends early: its later samples of these four do not count
        const uint32_t nib = (uint32_t)(term >> (lane & 60)) & 15u;
        if (nib) {
          const int first = __ffs(nib) - 1, src = (lane & 60) + first;
          if (k > first) wgt = 0.f;
          a = __shfl(a, src);
          tn = __shfl(tn, src);
          m = kRayDone;
          if (ISO && first < surf && hit >= L * i) hit = -1;  // it ended before the surface
        }
      }
      if (ISO && hit >= 0) m = kRayDone;
      acc = quad_bcast<3>(a);
      tr = tn;
      cr[0] = fmaf(wgt, r0, cr[0]);
      cg[0] = fmaf(wgt, g0, cg[0]);
      cb[0] = fmaf(wgt, b0, cb[0]);
      // (the step ends here: left alone, the compiler puts its end behind the wait for the next
      // sample's voxels, and FP32 frames take 5% longer)
      asm volatile("" : "+v"(cr[0]), "+v"(cg[0]), "+v"(cb[0]));
    }
  };
  // macrocell of a point: cell = floor(g + 1/2), in cells from the brick's first owned one
  const int64_t c0 = 0x80000000ll - ((int64_t)(b.olo[0] - b.slo[0]) << 32);
  const int64_t c1 = 0x80000000ll - ((int64_t)(b.olo[1] - b.slo[1]) << 32);
  const int64_t c2 = 0x80000000ll - ((int64_t)(b.olo[2] - b.slo[2]) << 32);
  auto macrocell = [&](int64_t cell, int a) {
    return clamp_index((int)(cell >> 32) >> b.mc_shift, b.mdim[a] - 1);
  };
  auto majorant = [&](int64_t x, int64_t y, int64_t z) {
    const int mx = macrocell(x + c0, 0), my = macrocell(y + c1, 1), mz = macrocell(z + c2, 2);
    return ld_global(b.majorant, (uint32_t)((mz * b.mdim[1] + my) * b.mdim[0] + mx));
  };
  // the samples at the lanes' next points all lie in macrocells that can be skipped
  auto empty_at = [&](float mj) {
    if constexpr (ISO) {
      // transparent, and on the side of the previous sample: classes 0 below, -1 at or above
      const float hi = L == 4 ? quad_max(mj) : mj, lo = L == 4 ? -quad_max(-mj) : mj;
      return hi <= 0.f && lo == hi && (!(pst & kIsoPair) || (hi < 0.f) == (bool)(pst & kIsoSide));
    } else {
      return (L == 4 ? quad_max(mj) : mj) == 0.f;
    }
  };

  Sample<T, WIDE> g[NB];
  bool pre = false;      // g[0 .. NB - 2] hold the samples at q, q + d, ...
  float mj_next = 0.f;
  bool have_mj = false;  // mj_next is the majorant at q
  bool done = m + k < 0;
  for (int trip = 0; !done && trip < max_trips; ++trip) {
    if constexpr (SKIP) {
      float mj = mj_next;
      if (!have_mj) {
        mj = majorant(q0, q1, q2);
        // (waits here, and not for the voxels requested ahead where the majorant was, too)
        asm volatile("" : "+v"(mj));
      }
      if (empty_at(mj)) {
        // the steps each lane makes inside its own macrocell.  A macrocell's range covers
        // half a voxel around the samples it holds, so the rounding of these distances
        // cannot matter.
        auto steps = [&](int64_t cell, int64_t dd, int a) {
          const int c = (int)(cell >> 32) - (macrocell(cell, a) << b.mc_shift);
          const float in = fmaf((float)(uint32_t)cell, 1.0f / 4294967296.0f, (float)c);
          const float v = fmaf((float)(uint32_t)dd, 1.0f / 4294967296.0f, (float)(int)(dd >> 32));
          const float dist = v > 0.f ? (float)(1 << b.mc_shift) - in : in;
          return dist * __builtin_amdgcn_rcpf(fabsf(v));
        };
        const float t = fminf(steps(q0 + c0, d0, 0), fminf(steps(q1 + c1, d1, 1), steps(q2 + c2, d2, 2)));
        int n = 1 + (int)fminf(fmaxf(t, 0.f), (float)(1 << 20));
        if constexpr (L == 4) n = quad_min(n);
        const int left = (m + k) / L + 1;
        n = n >= left ? left : (L == 1 ? n & ~3 : n);  // (one lane: whole groups of four)
        if (L == 4 || n > 0) {
          if constexpr (ISO) pst = kIsoPair | (mj < 0.f ? kIsoSide : 0);
          m -= L * n;
          dl_cur = Ddt;
          q0 += (int64_t)n * d0;
          q1 += (int64_t)n * d1;
          q2 += (int64_t)n * d2;
          pre = false;
          have_mj = false;
          done = m + k < 0;
          continue;
        }
      }
    }
    int64_t x = q0, y = q1, z = q2;  // the next point to request
    if (!pre) {
#pragma unroll
      for (int i = 0; i < NB - 1; ++i)
        request<T, WIDE>(b, q0 + i * d0, q1 + i * d1, q2 + i * d2, g[i]);
    }
    x += (NB - 1) * d0;
    y += (NB - 1) * d1;
    z += (NB - 1) * d2;
    int64_t n0 = 0, n1 = 0, n2 = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (i + NB - 1 == R) {  // the next trip's first samples
        n0 = x;
        n1 = y;
        n2 = z;
        if constexpr (SKIP) {
          mj_next = majorant(x, y, z);
          have_mj = true;
        }
      }
      Sample<T, WIDE>& ahead = g[(i + NB - 1) % NB];
      const Footed foot = request_first<T, WIDE>(b, x, y, z, ahead);
      // (a chain of additions: left alone, the compiler keeps every multiple of d in registers)
      x += d0;
      y += d1;
      z += d2;
      asm("" : "+v"(x), "+v"(y), "+v"(z));
      __builtin_amdgcn_sched_barrier(0);
      arrived(g[i % NB].v);
      load_run_ends(b, foot, ahead.v);
      __builtin_amdgcn_sched_barrier(0);
      step(g[i % NB], i);
    }
    if (ISO && hit >= 0) {
      // the point of the sample behind the surface, from this lane's point at the trip's start
      const int64_t dq[3] = {d0 / L, d1 / L, d2 / L};
      const int off = hit - k;
      const int64_t qs[3] = {q0 + off * dq[0], q1 + off * dq[1], q2 + off * dq[2]};
      const float t_hit = L == 4 ? quad_bcast<3>(tr) : tr;
      float c0 = cr[NC - 1], c1 = cg[NC - 1], c2 = cb[NC - 1];
      iso_hit<T, WIDE>(sc, b, tfr, qs, dq, vh, pst, pv, t_hit, c0, c1, c2);
      if (L == 1 || k == 3) {  // (one of the four sums takes it)
        cr[NC - 1] = c0;
        cg[NC - 1] = c1;
        cb[NC - 1] = c2;
      }
      tr = 0.f;
    }
    q0 = n0;
    q1 = n1;
    q2 = n2;
    pre = true;
    done = m + k < 0;
  }
  r.q[0] = q0;
  r.q[1] = q1;
  r.q[2] = q2;
  r.acc = acc;
  r.tr = tr;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    r.cr[i] = cr[i];
    r.cg[i] = cg[i];
    r.cb[i] = cb[i];
  }
  r.dl_cur = dl_cur;
  r.m = m;
  if constexpr (ISO) {
    r.pst = pst;
    r.pv = pv;
  }
  return done;
}

// The table as interleaved (entry, next - entry) records: one LDS address per lookup.
__device__ __forceinline__ void stage_tf_records(const float4* __restrict__ tf, int ntf, float4* rec, int tid,
                                                 int nthreads) {
  for (int i = tid; i < ntf; i += nthreads) {
    const float4 a = tf[i];
    const float4 b = (i + 1 < ntf) ? tf[i + 1] : a;
    rec[2 * i] = a;
    rec[2 * i + 1] = make_float4(b.x - a.x, b.y - a.y, b.z - a.z, b.w - a.w);
  }
}

// Element i (wave-uniform) of an array that no kernel writes, into scalar registers.
template <typename V>
__device__ __forceinline__ V ld_uniform(const V* p, int i) {
  static_assert(sizeof(V) % 4 == 0, "whole words");
  using C = const uint32_t __attribute__((address_space(4)))*;
  const C q = (C)(uintptr_t)(p + i);
  union {
    uint32_t w[sizeof(V) / 4];
    V v;
  } u;
#pragma unroll
  for (size_t j = 0; j < sizeof(V) / 4; ++j) u.w[j] = q[j];
  return u.v;
}

// Stage the TF as (entry, next - entry) pairs so a lookup is one FMA per channel.
__device__ __forceinline__ void stage_tf(const float4* __restrict__ tf, int ntf, float4* base, float4* slope,
                                         int tid, int nthreads) {
  for (int i = tid; i < ntf; i += nthreads) {
    float4 a = tf[i];
    float4 b = (i + 1 < ntf) ? tf[i + 1] : a;
    base[i] = a;
    slope[i] = make_float4(b.x - a.x, b.y - a.y, b.z - a.z, b.w - a.w);
  }
}

}  // namespace dpr
