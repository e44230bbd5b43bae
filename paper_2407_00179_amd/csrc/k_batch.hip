// Batched rendering of many cameras over uneven bricks.
//
// One persistent launch walks a queue of (camera, brick, screen tile) items.
// Each workgroup pops an item's 8 x 8 pixels with one atomic; each of its waves takes a
// chunk of them, 16 rays, at a time and marches them to their ends, four lanes per ray.
// A tile compositor then merges, per camera tile, the fragments of
// every item covering it.  The queue is built on the device (queue_kernel) from the
// bricks' screen rectangles, so a frame of a moving camera costs the host a few
// microseconds and no synchronization.  Repeated frames replay a HIP graph of march and
// composite.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "composite.h"
#include "march.h"
#include "runtime.hpp"

namespace dpr {

struct BatchItem {
  int cam, brick, tx, ty;
  int slot;  // where its fragments go, in tiles
};

// The tiles that one brick's screen rectangle covers in one camera's image.  Their items'
// fragments lie in raster order from slot `first` on, and their items take the same
// range of the queue, in another order.
struct BatchGroup {
  int x0, y0, w, h;  // tiles (w = h = 0: none)
  int first, cam, brick;
};

struct BatchG {
  const CamG* cams;
  const BrickG* bricks;
  const BatchGroup* groups;  // of camera c: groups_per_cam from c * groups_per_cam on
  int n_cams, groups_per_cam;
  const BatchItem* items;
  int n_items;
  int tile_w, tile_h;
  float4* frag_rgba;
  float* frag_depth;
  int* head;  // chunks popped by this launch; 0 between launches
  int* item_count;  // coverage counters (DPR_FLAG_QUEUE_COVERAGE), else null
  int* slot_count;
};

// Chunks that a workgroup takes from the queue at a time: one for each of its waves, so that
// they march side by side and meet in the CU's L1 (a wave on its own: 37% more L1 misses on
// the multi-camera batch of 27 FP16 bricks, 14.2 ms against 11.7).  Twice as many, or
// workgroups of 8 or 16 waves, are slower (12.4 ms), and so are neighbouring tiles for the
// waves of an XCD, which have half the L2 misses but crowd the same L2 channels (15.9 ms).
constexpr int kShareChunks = 4;

__global__ void zero_counts_kernel(int* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}

// A wave marches the queue's rays with the four lanes of a quad per ray (march.h), 16 at a
// time: 4 x 4 pixel patches of a tile where the tile's shape allows.  What bounds it: the
// chain of a launch's longest ray where a frame has few rays (one 256^3 brick at 1024^2:
// 0.56 ms with one lane per ray, 0.14 ms with four), else the texture path, which is busy over
// 80% of the time: a load of 64 scattered lanes takes 17 to 24 cycles whatever its width, and
// L1 misses wait.  A wave's 16 rays end together as a rule: handing the lanes of those that
// ended to others (once half had: 7.5 ms on two cameras at 2048^2 of 27 FP16 bricks; once an
// eighth was left: 7.2; not at all: 7.0) costs more in ray set-up, in 64 bits and for few
// lanes at a time, than it saves.  With 80 to 91 registers five or six waves run on a SIMD
// (ISO: four); more by force only spills.  More workgroups than have a share of the queue
// only cost their start.
template <typename T, bool SKIP, bool WIDE, bool ISO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void batch_march_kernel(
    SceneG sc, BatchG bg, const float4* __restrict__ tf) {
  extern __shared__ float4 tf_lds[];
  stage_tf_records(tf, sc.ntf, tf_lds, threadIdx.x, 256);
  // the workgroup's share of the queue: chunks [next, end), taken under a lock
  __shared__ int lock, share_next, share_end;
  if (threadIdx.x == 0) {
    lock = 0;
    share_next = blockIdx.x * kShareChunks;
    share_end = share_next + kShareChunks;
  }
  __syncthreads();

  constexpr int L = 4;
  const int lane = threadIdx.x & 63, k = lane & (L - 1);
  const int tp = bg.tile_w * bg.tile_h;
  const bool patches = ((bg.tile_w | bg.tile_h) & 3) == 0;
  const int patches_x = bg.tile_w >> 2;
  const bool squares = ((bg.tile_w | bg.tile_h) & 7) == 0;
  const int squares_x = bg.tile_w >> 3;

  // the queue's unit is a chunk of the rays of a wave (it divides every tile's pixels)
  constexpr int kChunkRays = 64 / L;
  const int per_item = tp / kChunkRays, n_chunks = bg.n_items * per_item;

  for (;;) {
    int c = 0;
    if (lane == 0) {
      // (the holder's work is finite and needs no other wave, so every wait ends)
      while (__hip_atomic_exchange(&lock, 1, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) __builtin_amdgcn_s_sleep(1);
      c = __hip_atomic_load(&share_next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (c == __hip_atomic_load(&share_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) && c < n_chunks) {
        c = (atomicAdd(bg.head, 1) + gridDim.x) * kShareChunks;
        __hip_atomic_store(&share_end, c + kShareChunks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      // (past the queue's end nothing more is taken)
      __hip_atomic_store(&share_next, c < n_chunks ? c + 1 : c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_store(&lock, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    // wave-uniform: the item, and so the camera and the brick, live in scalar registers
    c = __builtin_amdgcn_readfirstlane(c);
    if (c >= n_chunks) break;
    const int it = c / per_item, first = (c % per_item) * kChunkRays;
    if (bg.item_count && lane == 0 && first == 0) atomicAdd(bg.item_count + it, 1);
    const BatchItem I = ld_uniform(bg.items, it);
    const int i = first + lane / L;
    int ux, uy;  // pixel inside the tile
    if (squares) {
      const int p = i >> 6, s = i >> 4;  // 8 x 8 pixels of four patches
      ux = (p % squares_x) * 8 + (s & 1) * 4 + (i & 1) + ((i >> 1) & 2);
      uy = (p / squares_x) * 8 + (s & 2) * 2 + ((i >> 1) & 1) + ((i >> 2) & 2);
    } else if (patches) {
      const int p = i >> 4;
      ux = (p % patches_x) * 4 + (i & 3);
      uy = (p / patches_x) * 4 + ((i >> 2) & 3);
    } else {
      ux = i % bg.tile_w;
      uy = i / bg.tile_w;
    }
    const int px = I.tx * bg.tile_w + ux, py = I.ty * bg.tile_h + uy;
    const CamG cam = ld_uniform(bg.cams, I.cam);
    float4 rgba = make_float4(0.f, 0.f, 0.f, 0.f);
    float z = INFINITY;
    if (px < cam.W && py < cam.H) {
      double d[3];
      camera_ray(cam, px, py, d);
      LaneRay r;
      if (lane_begin<T, WIDE, ISO, L>(sc, ld_uniform(bg.bricks, I.brick), cam.eye, d, k, r)) {
        lane_advance<T, SKIP, WIDE, ISO, L>(sc, ld_uniform(bg.bricks, I.brick), tf_lds, r, 0x7fffffff);
        rgba = ray_rgba<L>(r);
        z = r.t_in;
      }
    }
    if (k == L - 1) {
      const size_t slot = (size_t)I.slot * tp + uy * bg.tile_w + ux;
      bg.frag_rgba[slot] = rgba;
      bg.frag_depth[slot] = z;
      if (bg.slot_count) atomicAdd(bg.slot_count + slot, 1);
    }
  }
}

// Builds a launch's queue: groups in order, inside a group the tiles by decreasing chord of
// their centre ray through the brick, so that the longest rays start first and the rays
// still marching when a group (or the whole queue) runs out are short ones.  Workgroup j of
// the J that a group of T tiles takes has the tiles j, j + J, ...: it sorts them (a
// counting sort over kChordBuckets lengths) and writes its p-th to place p J + j, so the J
// sorted lists together are nearly a sorted one and no pass goes over the whole group.
// Also copies the launch's descriptors from host memory (src) to the device (dst) and
// clears the queue's head.  Latency-bound (descriptors read over the bus, two barriers): 7.5 us
// for eight bricks at 1024^2.  Lists built and sorted on the host, uploaded with a wait each
// and captured into a new graph took 0.9 ms a frame there, and 0.2 ms at 256^2.
constexpr int kQueueTiles = 2048, kChordBuckets = 64;
struct QueueG {
  const uint4* src;
  uint4* dst;
  int words;
  const CamG* cams;  // in src
  const BrickG* bricks;
  const BatchGroup* groups;
  int n_groups;      // 0: the copy only
  int tile_w, tile_h;
  double h;
  float inv_diag;    // 1 / the longest chord
  BatchItem* items;
  int* head;
};
__global__ __launch_bounds__(256) void queue_kernel(QueueG q) {
  __shared__ int count[kChordBuckets];
  const int tid = threadIdx.x;
  for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * 256 + tid; i < q.words; i += gridDim.x * gridDim.y * 256)
    q.dst[i] = q.src[i];
  if (q.n_groups && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *q.head = 0;
  for (int gi = blockIdx.y; gi < q.n_groups; gi += gridDim.y) {
    const BatchGroup g = q.groups[gi];
    const int T = g.w * g.h, J = (T + kQueueTiles - 1) / kQueueTiles;
    for (int j = blockIdx.x; j < J; j += gridDim.x) {
      const CamG& cam = q.cams[g.cam];
      const BrickG& b = q.bricks[g.brick];
      if (tid < kChordBuckets) count[tid] = 0;
      __syncthreads();
      float lo[3], hi[3];  // the brick's faces from the eye
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lo[a] = (float)(b.olo[a] * q.h - cam.eye[a]);
        hi[a] = (float)(b.ohi[a] * q.h - cam.eye[a]);
      }
      const float mx = 2.f * (float)cam.sx / (float)cam.W, my = -2.f * (float)cam.sy / (float)cam.H;
      constexpr int U = kQueueTiles / 256;
      int bucket[U], rank[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = (u * 256 + tid) * J + j;
        bucket[u] = -1;
        if (t < T) {
          const float x = ((float)((g.x0 + t % g.w) * q.tile_w) + 0.5f * (float)q.tile_w) * mx - (float)cam.sx;
          const float y = ((float)((g.y0 + t / g.w) * q.tile_h) + 0.5f * (float)q.tile_h) * my + (float)cam.sy;
          float tn = 0.f, tf = INFINITY, dd = 0.f;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const float d = (float)cam.f[a] + x * (float)cam.r[a] + y * (float)cam.u[a];
            dd += d * d;
            const float inv = 1.f / d, t0 = lo[a] * inv, t1 = hi[a] * inv;  // (an infinity or NaN only misplaces a tile)
            tn = fmaxf(tn, fminf(t0, t1));
            tf = fminf(tf, fmaxf(t0, t1));
          }
          const float chord = fmaxf(tf - tn, 0.f) * sqrtf(dd) * q.inv_diag;  // 0 .. 1
          bucket[u] = min(max((int)((1.f - chord) * kChordBuckets), 0), kChordBuckets - 1);
          rank[u] = atomicAdd(&count[bucket[u]], 1);
        }
      }
      __syncthreads();
      if (tid < kChordBuckets) {  // (one wave) counts -> places
        const int n = count[tid];
        int sum = n;
        for (int o = 1; o < kChordBuckets; o <<= 1) {
          const int v = __shfl_up(sum, o);
          if (tid >= o) sum += v;
        }
        count[tid] = sum - n;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (bucket[u] < 0) continue;
        const int t = (u * 256 + tid) * J + j;
        q.items[g.first + (count[bucket[u]] + rank[u]) * J + j] =
            BatchItem{g.cam, g.brick, g.x0 + t % g.w, g.y0 + t / g.w, g.first + t};
      }
      __syncthreads();
    }
  }
}

// The bricks that cover a tile of camera c, in brick order: their fragments' slots and
// brick numbers (the wave looks at 64 groups at a time).  Returns how many.
template <int KMAX>
struct TileSources {
  int slot[KMAX], brick[KMAX];
};
template <int KMAX>
__device__ __forceinline__ int tile_sources(TileSources<KMAX>& s, const BatchG& bg, int c, int tx, int ty) {
  const int lane = threadIdx.x;
  const BatchGroup* gs = bg.groups + (size_t)c * bg.groups_per_cam;
  int n = 0;
  for (int k0 = 0; k0 < bg.groups_per_cam; k0 += 64) {
    BatchGroup g;
    bool in = false;
    if (k0 + lane < bg.groups_per_cam) {
      g = gs[k0 + lane];
      in = (unsigned)(tx - g.x0) < (unsigned)g.w && (unsigned)(ty - g.y0) < (unsigned)g.h;
    }
    const uint64_t m = __ballot(in);
    const int i = n + __popcll(m & ~(~0ull << lane));
    if (in && i < KMAX) {
      s.slot[i] = g.first + (ty - g.y0) * g.w + tx - g.x0;
      s.brick[i] = g.brick;
    }
    n += __popcll(m);
  }
  __syncthreads();
  return min(n, KMAX);
}

// Per camera tile: composite the fragments of the items that cover it.  One wave
// per 64 pixels of a tile.
template <int KMAX>
__global__ __launch_bounds__(64) void tile_composite_kernel(BatchG bg, float4* const* __restrict__ out_rgba,
                                                            float* const* __restrict__ out_depth, int chunks) {
  __shared__ CompLDS<KMAX> s;
  __shared__ TileSources<KMAX> src;
  const int g = blockIdx.x / chunks;
  const int q = blockIdx.x % chunks;
  const int lane = threadIdx.x;
  const int tp = bg.tile_w * bg.tile_h;
  const int pix = q * 64 + lane;
  if (blockIdx.x == 0 && blockIdx.y == 0 && lane == 0) *bg.head = 0;  // for the next launch
  for (int c = blockIdx.y; c < bg.n_cams; c += gridDim.y) {
    const int W = bg.cams[c].W, H = bg.cams[c].H;
    const int tiles_x = (W + bg.tile_w - 1) / bg.tile_w;
    const int tx = g % tiles_x, ty = g / tiles_x;
    if (ty * bg.tile_h >= H) continue;
    const int px = tx * bg.tile_w + pix % bg.tile_w;
    const int py = ty * bg.tile_h + pix / bg.tile_w;
    const bool live_px = pix < tp && px < W && py < H;
    const int K = tile_sources<KMAX>(src, bg, c, tx, ty);
    float4 col = make_float4(0.f, 0.f, 0.f, 0.f);
    float z = INFINITY;
    if (K > 0) {
      composite_wave<KMAX>(
          s, K, live_px, [&](int k) { return bg.frag_depth[(size_t)src.slot[k] * tp + pix]; },
          [&](int k) { return bg.frag_rgba[(size_t)src.slot[k] * tp + pix]; },
          [&](int k) { return src.brick[k]; }, col, z);
    }
    if (live_px) {
      const size_t p = (size_t)py * W + px;
      out_rgba[c][p] = col;
      out_depth[c][p] = z;
    }
    __syncthreads();
  }
}

// Deep-frame target of the tile pass (dpr_render_deep): per pixel the count and
// the sorted fragments, layer-major (layer i of pixel p at i * P + p).
struct DeepOut {
  int* counts;
  float4* rgba;
  float* depth;
  int* ids;
  size_t P;
  int rank;
};

// Per camera tile: sort each pixel's fragments of the items covering the tile by
// (depth, brick) and write them as the pixel's deep-frame layers.  One wave per 64
// pixels of a tile; one camera.
template <int KMAX>
__global__ __launch_bounds__(64) void tile_deep_kernel(BatchG bg, DeepOut dout, int chunks) {
  __shared__ CompLDS<KMAX> s;
  __shared__ TileSources<KMAX> src;
  const int g = blockIdx.x / chunks;
  const int q = blockIdx.x % chunks;
  const int lane = threadIdx.x;
  if (blockIdx.x == 0 && lane == 0) *bg.head = 0;  // for the next launch
  const int W = bg.cams[0].W, H = bg.cams[0].H;
  const int tp = bg.tile_w * bg.tile_h;
  const int tiles_x = (W + bg.tile_w - 1) / bg.tile_w;
  const int tx = g % tiles_x, ty = g / tiles_x;
  const int pix = q * 64 + lane;
  const int px = tx * bg.tile_w + pix % bg.tile_w;
  const int py = ty * bg.tile_h + pix / bg.tile_w;
  const bool live_px = pix < tp && px < W && py < H;
  const int K = tile_sources<KMAX>(src, bg, 0, tx, ty);
  int n = 0;
  if (K > 0)
    n = sort_wave<KMAX>(
        s, K, live_px, [&](int k) { return bg.frag_depth[(size_t)src.slot[k] * tp + pix]; },
        [&](int k) { return src.brick[k]; });
  if (live_px) {
    const size_t p = (size_t)py * W + px;
    dout.counts[p] = n;
    for (int i = 0; i < n; ++i) {
      const int k = s.lst[i][lane];
      dout.rgba[(size_t)i * dout.P + p] = bg.frag_rgba[(size_t)src.slot[k] * tp + pix];
      dout.depth[(size_t)i * dout.P + p] = s.zs[k][lane];
      dout.ids[(size_t)i * dout.P + p] = dout.rank * 65536 + src.brick[k];
    }
  }
}

// A buffer kept for the next frames: a first one of the size asked for, a later one with a
// quarter to spare where that can be had, so that a moving camera seldom allocates; one of
// more than 64 MiB is given back when a sixteenth of it would do.
struct GrowBuffer {
  void* p = nullptr;
  size_t cap = 0;
  dpr_status need(size_t bytes, const char* what) {
    if (p && bytes <= cap && (cap <= (64u << 20) || bytes > cap / 16)) return DPR_OK;
    const bool again = p != nullptr && bytes > cap;
    release();
    bytes = std::max<size_t>(bytes, 256);
    const size_t spare = bytes + bytes / 4;
    if (again && dev_alloc(&p, spare, what) == DPR_OK) {
      cap = spare;
      return DPR_OK;
    }
    dpr_status s = dev_alloc(&p, bytes, what);
    if (s == DPR_OK) cap = bytes;
    return s;
  }
  void release() {
    dev_free(p);  // (waits for the device)
    p = nullptr;
    cap = 0;
  }
};

struct BatchState {
  // key
  std::vector<dpr_camera> cams;
  std::vector<dpr_frame> outs;
  std::vector<const void*> out_ptrs;
  int tile_w = 0, tile_h = 0;
  int brick_sel = -1;  // the one brick rendered (dpr_render_partial), or -1 for all
  uint64_t geo_version = 0;
  bool skip = true;
  // deep-frame target (dpr_render_deep) instead of flat frames, and its buffers
  dpr_deep_frame deep = nullptr;
  const void* deep_ptrs[4] = {nullptr, nullptr, nullptr, nullptr};
  int deep_rank = -1;
  // brick views last brought to the device, and the scene arguments and TF table
  // baked into the captured graph
  std::vector<BrickG> h_bricks;
  SceneG cap_scene{};
  const float4* cap_tf = nullptr;
  // the launch's descriptors: cameras, bricks, groups, output pointers, in one device
  // buffer that queue_kernel fills from pinned host memory (kStages copies in turn, each
  // with an event after its last reader)
  static constexpr int kStages = 4;
  GrowBuffer desc, queue, fragments, fragment_depths;
  char* stage = nullptr;
  size_t stage_cap = 0;  // of one copy
  int next_stage = 0;
  hipEvent_t stage_ev[kStages] = {nullptr, nullptr, nullptr, nullptr};
  size_t off_cams = 0, off_bricks = 0, off_groups = 0, off_rgba = 0, off_depth = 0, desc_bytes = 0;
  std::vector<char> h_desc;   // what the device buffer holds (or will, in stream order)
  bool built = false;
  int uses = 0;               // renders since the descriptors or an argument last changed
  bool used = false;          // last_stream is set
  hipStream_t last_stream = nullptr;
  int* item_count = nullptr;  // queue-coverage counters, allocated on first use
  int* slot_count = nullptr;
  bool counted = false;       // the last render counted
  int n_items = 0, n_groups = 0, groups_per_cam = 0, max_k = 0, queue_blocks = 0;
  unsigned tiles = 0;    // of the largest image
  int grid[2] = {0, 0};  // persistent grid of the march kernel without / with iso-surface
  const void* grid_fn[2] = {nullptr, nullptr};  // and what it was worked out for
  size_t grid_lds = 0;
  hipStream_t cap = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipEvent_t ev[3] = {nullptr, nullptr, nullptr};  // before march, after march, after composite
  bool timed = false;                               // events were recorded by the last render
  // plain per-brick path
  std::vector<dpr_frame> plain_parts;

  int* head() const { return (int*)desc.p; }
  template <typename V>
  V* dev_at(size_t off) const { return (V*)((char*)desc.p + off); }
  void drop_counts() {
    dev_free(item_count);
    dev_free(slot_count);
    item_count = slot_count = nullptr;
    counted = false;
  }
  // 64-bit offsets for every brick if any brick the launch reads needs them
  bool wide() const {
    if (brick_sel >= 0) return brick_sel < (int)h_bricks.size() && h_bricks[brick_sel].wide;
    for (const auto& g : h_bricks)
      if (g.wide) return true;
    return false;
  }
  void drop_graph() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    exec = nullptr;
    graph = nullptr;
  }
  ~BatchState() {
    drop_graph();
    drop_counts();
    for (auto* b : {&desc, &queue, &fragments, &fragment_depths}) b->release();
    host_free(stage);
    for (auto e : stage_ev)
      if (e) (void)hipEventDestroy(e);
    for (auto f : plain_parts) dpr_frame_release(f);
    if (cap) (void)hipStreamDestroy(cap);
    for (auto e : ev)
      if (e) (void)hipEventDestroy(e);
  }
};

void batch_state_free(BatchState* s) { delete s; }

// Conservative screen rectangle (pixel indices, inclusive) of a box's projection.
static void brick_screen_rect(const CamG& c, const double lo[3], const double hi[3], int& x0, int& y0, int& x1,
                              int& y1) {
  double mnx = 1e300, mny = 1e300, mxx = -1e300, mxy = -1e300;
  for (int i = 0; i < 8; ++i) {
    double p[3] = {(i & 1) ? hi[0] : lo[0], (i & 2) ? hi[1] : lo[1], (i & 4) ? hi[2] : lo[2]};
    double v[3] = {p[0] - c.eye[0], p[1] - c.eye[1], p[2] - c.eye[2]};
    double z = v[0] * c.f[0] + v[1] * c.f[1] + v[2] * c.f[2];
    if (!(z > 1e-9)) {  // a corner at or behind the eye: take the whole screen
      x0 = 0;
      y0 = 0;
      x1 = c.W - 1;
      y1 = c.H - 1;
      return;
    }
    double x = (v[0] * c.r[0] + v[1] * c.r[1] + v[2] * c.r[2]) / z;
    double y = (v[0] * c.u[0] + v[1] * c.u[1] + v[2] * c.u[2]) / z;
    double px = (x / c.sx + 1.0) * 0.5 * c.W - 0.5;
    double py = (1.0 - y / c.sy) * 0.5 * c.H - 0.5;
    mnx = std::min(mnx, px);
    mxx = std::max(mxx, px);
    mny = std::min(mny, py);
    mxy = std::max(mxy, py);
  }
  x0 = (int)std::max(0.0, std::floor(mnx) - 1.0);
  y0 = (int)std::max(0.0, std::floor(mny) - 1.0);
  x1 = (int)std::min((double)c.W - 1, std::ceil(mxx) + 1.0);
  y1 = (int)std::min((double)c.H - 1, std::ceil(mxy) + 1.0);
}

template <typename T, bool SKIP, bool ISO>
static const void* march_fn_t(bool wide) {
  return wide ? (const void*)batch_march_kernel<T, SKIP, true, ISO>
              : (const void*)batch_march_kernel<T, SKIP, false, ISO>;
}

template <typename T, bool SKIP>
static const void* march_fn_s(bool wide, bool iso) {
  return iso ? march_fn_t<T, SKIP, true>(wide) : march_fn_t<T, SKIP, false>(wide);
}

static const void* march_fn(bool f16, bool skip, bool wide, bool iso) {
  if (f16) return skip ? march_fn_s<__half, true>(wide, iso) : march_fn_s<__half, false>(wide, iso);
  return skip ? march_fn_s<float, true>(wide, iso) : march_fn_s<float, false>(wide, iso);
}

static hipError_t enqueue_batch(dpr_world w, BatchState* b, hipStream_t st, bool timed, bool count = false) {
  SceneG sc = make_scene(w);
  BatchG g{};
  g.cams = b->dev_at<CamG>(b->off_cams);
  g.bricks = b->dev_at<BrickG>(b->off_bricks);
  g.groups = b->dev_at<BatchGroup>(b->off_groups);
  g.n_cams = (int)b->cams.size();
  g.groups_per_cam = b->groups_per_cam;
  g.items = (const BatchItem*)b->queue.p;
  g.n_items = b->n_items;
  g.tile_w = b->tile_w;
  g.tile_h = b->tile_h;
  g.frag_rgba = (float4*)b->fragments.p;
  g.frag_depth = (float*)b->fragment_depths.p;
  g.head = b->head();
  if (count) {
    const size_t slots = (size_t)b->n_items * b->tile_w * b->tile_h;
    g.item_count = b->item_count;
    g.slot_count = b->slot_count;
    hipLaunchKernelGGL(zero_counts_kernel, dim3(256), dim3(256), 0, st, b->item_count, (size_t)b->n_items);
    hipLaunchKernelGGL(zero_counts_kernel, dim3(1024), dim3(256), 0, st, b->slot_count, slots);
  }
  const bool f16 = w->bricks[b->brick_sel >= 0 ? b->brick_sel : 0].dtype == DPR_F16;
  size_t lds = 2 * sizeof(float4) * (size_t)sc.ntf;
  const int iso = sc.iso_on ? 1 : 0;
  if (timed) (void)hipEventRecord(b->ev[0], st);
  const void* fn = march_fn(f16, b->skip, b->wide(), iso);
  void* args[] = {(void*)&sc, (void*)&g, (void*)&w->tf_dev};
  // no more workgroups than have a share of the queue
  const size_t shares = ((size_t)b->n_items * (b->tile_w * b->tile_h / 16) + kShareChunks - 1) / kShareChunks;
  const unsigned grid = (unsigned)std::min<size_t>(b->grid[iso], std::max<size_t>(shares, 1));
  const hipError_t le = hipLaunchKernel(fn, dim3(grid), dim3(256), args, lds, st);
  if (le != hipSuccess) return le;
  if (timed) (void)hipEventRecord(b->ev[1], st);
  const int tp = b->tile_w * b->tile_h;
  const int chunks = (tp + 63) / 64;
  const dim3 cgrid(b->tiles * chunks, (unsigned)std::min<size_t>(b->cams.size(), 65535));
  if (b->deep) {
    const dpr_deep_frame d = b->deep;
    DeepOut dout{d->counts, d->rgba, d->depth, d->ids, (size_t)d->w * d->h, b->deep_rank};
    if (b->max_k <= 16)
      hipLaunchKernelGGL(tile_deep_kernel<16>, cgrid, dim3(64), 0, st, g, dout, chunks);
    else if (b->max_k <= 64)
      hipLaunchKernelGGL(tile_deep_kernel<64>, cgrid, dim3(64), 0, st, g, dout, chunks);
    else
      hipLaunchKernelGGL(tile_deep_kernel<256>, cgrid, dim3(64), 0, st, g, dout, chunks);
  } else {
    float4* const* orgba = b->dev_at<float4*>(b->off_rgba);
    float* const* odepth = b->dev_at<float*>(b->off_depth);
    if (b->max_k <= 16)
      hipLaunchKernelGGL(tile_composite_kernel<16>, cgrid, dim3(64), 0, st, g, orgba, odepth, chunks);
    else if (b->max_k <= 64)
      hipLaunchKernelGGL(tile_composite_kernel<64>, cgrid, dim3(64), 0, st, g, orgba, odepth, chunks);
    else
      hipLaunchKernelGGL(tile_composite_kernel<256>, cgrid, dim3(64), 0, st, g, orgba, odepth, chunks);
  }
  if (timed) (void)hipEventRecord(b->ev[2], st);
  return hipGetLastError();
}

// Waits for the state's frames in flight, also on another stream than the present one.
static dpr_status wait_frames(dpr_world w, BatchState* b) {
  if (b->used && b->last_stream != w->dev->stream)
    DPR_HIP(hipDeviceSynchronize());
  else
    DPR_HIP(hipStreamSynchronize(w->dev->stream));
  return DPR_OK;
}

// Brings h_desc to the device, and builds the queue from it where `sort` is set.  Nothing
// waits, unless the state was last used on another stream.
static dpr_status enqueue_desc(dpr_world w, BatchState* b, bool sort) {
  hipStream_t st = w->dev->stream;
  // (a graph of the caller's would copy from a stage that later frames rewrite)
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  DPR_HIP(hipStreamIsCapturing(st, &cs));
  if (cs != hipStreamCaptureStatusNone) return hip_fail(hipErrorStreamCaptureUnsupported, "batched render: new descriptors");
  dpr_status s;
  if (b->used && b->last_stream != st && (s = wait_frames(w, b)) != DPR_OK) return s;
  if (b->desc_bytes > b->stage_cap) {
    DPR_HIP(hipStreamSynchronize(st));
    host_free(b->stage);
    b->stage = nullptr;
    b->stage_cap = 0;
    if ((s = host_alloc((void**)&b->stage, b->desc_bytes * BatchState::kStages, "batch descriptors")) != DPR_OK) return s;
    b->stage_cap = b->desc_bytes;
  }
  const int i = b->next_stage;
  b->next_stage = (i + 1) % BatchState::kStages;
  if (!b->stage_ev[i])
    DPR_HIP(hipEventCreateWithFlags(&b->stage_ev[i], hipEventDisableTiming));
  else
    DPR_HIP(hipEventSynchronize(b->stage_ev[i]));
  char* src = b->stage + (size_t)i * b->stage_cap;
  memcpy(src, b->h_desc.data(), b->desc_bytes);
  const SceneG sc = make_scene(w);
  QueueG q{};
  q.src = (const uint4*)src;
  q.dst = (uint4*)b->desc.p;
  q.words = (int)(b->desc_bytes / sizeof(uint4));
  q.cams = (const CamG*)(src + b->off_cams);
  q.bricks = (const BrickG*)(src + b->off_bricks);
  q.groups = (const BatchGroup*)(src + b->off_groups);
  q.n_groups = sort ? b->n_groups : 0;
  q.tile_w = b->tile_w;
  q.tile_h = b->tile_h;
  q.h = sc.h;
  q.inv_diag = (float)(1.0 / (sc.h * std::sqrt((double)sc.dims[0] * sc.dims[0] + (double)sc.dims[1] * sc.dims[1] +
                                               (double)sc.dims[2] * sc.dims[2])));
  q.items = (BatchItem*)b->queue.p;
  q.head = b->head();
  const dim3 grid(sort ? b->queue_blocks : 1, sort ? std::min(b->n_groups, 65535) : 4);
  hipLaunchKernelGGL(queue_kernel, grid, dim3(256), 0, st, q);
  DPR_HIP(hipGetLastError());
  DPR_HIP(hipEventRecord(b->stage_ev[i], st));
  b->uses = 0;
  return DPR_OK;
}

// Most rectangles of a camera's groups that share a tile.  The corner (x0, y0) of some two
// of them lies in as many as any tile does; per x0, the rows are counted with a
// difference array.
static int max_overlap(const BatchGroup* g, int n) {
  int rows = 0, best = 0;
  for (int i = 0; i < n; ++i) rows = std::max(rows, g[i].y0 + g[i].h);
  std::vector<int> diff(rows + 1);
  for (int i = 0; i < n; ++i) {
    if (g[i].w == 0) continue;
    std::fill(diff.begin(), diff.end(), 0);
    for (int j = 0; j < n; ++j)
      if (g[j].w && g[j].x0 <= g[i].x0 && g[i].x0 < g[j].x0 + g[j].w) {
        ++diff[g[j].y0];
        --diff[g[j].y0 + g[j].h];
      }
    int sum = 0;
    for (int v : diff) best = std::max(best, sum += v);
  }
  return best;
}

// (Re)build the descriptors, the queue and the fragment storage for these cameras.
static dpr_status build_batch(dpr_world w, BatchState* b, const dpr_camera* cams, int n, const dpr_frame* outs,
                              int tw, int th, int brick_sel) {
  b->built = false;
  b->drop_counts();
  dpr_status s;
  if (b->exec) {
    if ((s = wait_frames(w, b)) != DPR_OK) return s;
    b->drop_graph();
  }
  b->cams.assign(cams, cams + n);
  b->outs.assign(outs, outs + n);
  b->out_ptrs.clear();
  for (int c = 0; c < n; ++c) {
    b->out_ptrs.push_back(outs[c] ? outs[c]->rgba : nullptr);
    b->out_ptrs.push_back(outs[c] ? outs[c]->depth : nullptr);
  }
  b->tile_w = tw;
  b->tile_h = th;
  b->brick_sel = brick_sel;
  b->geo_version = w->geo_version;
  b->skip = !(w->params.flags & DPR_FLAG_NO_SKIP);
  const SceneG sc = make_scene(w);
  b->h_bricks.clear();
  for (const auto& br : w->bricks)
    b->h_bricks.push_back(br.device_view(b->skip, w->params.flags & DPR_FLAG_WIDE_OFFSETS));
  const int K = brick_sel >= 0 ? 1 : (int)w->bricks.size();
  b->groups_per_cam = K;
  b->n_groups = n * K;
  auto place = [](size_t& end, size_t bytes) {
    const size_t at = end;
    end = (end + bytes + 127) / 128 * 128;
    return at;
  };
  size_t end = 128;  // the queue's head
  b->off_cams = place(end, n * sizeof(CamG));
  b->off_bricks = place(end, b->h_bricks.size() * sizeof(BrickG));
  b->off_groups = place(end, (size_t)b->n_groups * sizeof(BatchGroup));
  b->off_rgba = place(end, n * sizeof(float4*));
  b->off_depth = place(end, n * sizeof(float*));
  b->desc_bytes = end;
  b->h_desc.assign(end, 0);
  CamG* cg = (CamG*)(b->h_desc.data() + b->off_cams);
  BatchGroup* groups = (BatchGroup*)(b->h_desc.data() + b->off_groups);
  memcpy(b->h_desc.data() + b->off_bricks, b->h_bricks.data(), b->h_bricks.size() * sizeof(BrickG));
  int first = 0, max_k = 1, largest = 1;
  b->tiles = 0;
  for (int c = 0; c < n; ++c) {
    cg[c] = make_cam(cams[c]);
    ((float4**)(b->h_desc.data() + b->off_rgba))[c] = outs[c] ? (float4*)outs[c]->rgba : nullptr;
    ((float**)(b->h_desc.data() + b->off_depth))[c] = outs[c] ? outs[c]->depth : nullptr;
    b->tiles = std::max(b->tiles, (unsigned)((cams[c].width + tw - 1) / tw) * (unsigned)((cams[c].height + th - 1) / th));
    for (int i = 0; i < K; ++i) {
      const int k = brick_sel >= 0 ? brick_sel : i;
      const Brick& br = w->bricks[k];
      double lo[3], hi[3];
      for (int a = 0; a < 3; ++a) {
        lo[a] = br.olo[a] * sc.h;
        hi[a] = br.ohi[a] * sc.h;
      }
      int x0, y0, x1, y1;
      brick_screen_rect(cg[c], lo, hi, x0, y0, x1, y1);
      BatchGroup& g = groups[(size_t)c * K + i];
      g = BatchGroup{0, 0, 0, 0, first, c, k};
      if (x1 < x0 || y1 < y0) continue;
      g.x0 = x0 / tw;
      g.y0 = y0 / th;
      g.w = x1 / tw - g.x0 + 1;
      g.h = y1 / th - g.y0 + 1;
      first += g.w * g.h;
      largest = std::max(largest, g.w * g.h);
    }
    max_k = std::max(max_k, K <= 16 ? K : max_overlap(groups + (size_t)c * K, K));
  }
  if (max_k > kMaxFrags) return fail(DPR_ERR_UNSUPPORTED, "dpr_render_batch: %d bricks cover one tile", max_k);
  b->n_items = first;
  b->max_k = max_k;
  b->queue_blocks = std::min((largest + kQueueTiles - 1) / kQueueTiles, 4096);
  const size_t frags = (size_t)b->n_items * tw * th;
  if ((s = b->desc.need(b->desc_bytes, "batch descriptors")) != DPR_OK) return s;
  if ((s = b->queue.need((size_t)b->n_items * sizeof(BatchItem), "batch items")) != DPR_OK) return s;
  if ((s = b->fragments.need(frags * sizeof(float4), "batch fragments")) != DPR_OK) return s;
  if ((s = b->fragment_depths.need(frags * sizeof(float), "batch fragment depths")) != DPR_OK) return s;
  for (auto& e : b->ev)
    if (!e) DPR_HIP(hipEventCreate(&e));
  // persistent grid: as many 256-thread workgroups as fit on the GPU at once
  const bool f16 = w->bricks[brick_sel >= 0 ? brick_sel : 0].dtype == DPR_F16;
  const size_t lds = 2 * sizeof(float4) * (size_t)sc.ntf;
  for (int iso = 0; iso < 2; ++iso) {
    const void* fn = march_fn(f16, b->skip, b->wide(), iso);
    if (fn == b->grid_fn[iso] && lds == b->grid_lds) continue;
    int per_cu = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, lds);
    if (e != hipSuccess || per_cu < 1) per_cu = 1;
    b->grid[iso] = w->dev->cu_count * per_cu;
    b->grid_fn[iso] = fn;
  }
  b->grid_lds = lds;
  if ((s = enqueue_desc(w, b, true)) != DPR_OK) return s;
  b->built = true;
  return DPR_OK;
}

static dpr_status capture_graph(dpr_world w, BatchState* b) {
  if (!b->cap) DPR_HIP(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
  DPR_HIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
  hipError_t e = enqueue_batch(w, b, b->cap, false);
  hipGraph_t g = nullptr;
  hipError_t e2 = hipStreamEndCapture(b->cap, &g);
  if (e != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return hip_fail(e, "dpr_render_batch: capture");
  }
  if (e2 != hipSuccess) return hip_fail(e2, "hipStreamEndCapture");
  b->graph = g;
  DPR_HIP(hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0));
  b->cap_scene = make_scene(w);
  b->cap_tf = w->tf_dev;
  return DPR_OK;
}

// The queue depends only on geometry (bricks, cameras, tile shape); data
// recommits and transfer-function changes only touch the brick views (device
// pointers, macrocell grids) and the scene arguments, which are refreshed here
// without rebuilding: brick views are brought to the device again when they changed, and
// the captured graph is dropped when an argument baked into it changed.
static dpr_status refresh_batch(dpr_world w, BatchState* b) {
  std::vector<BrickG> bg;
  for (const auto& br : w->bricks) bg.push_back(br.device_view(b->skip, w->params.flags & DPR_FLAG_WIDE_OFFSETS));
  const bool moved = bg.size() != b->h_bricks.size() || memcmp(bg.data(), b->h_bricks.data(), bg.size() * sizeof(BrickG)) != 0;
  bool stale = moved;
  if (b->exec) {
    const SceneG sc = make_scene(w);
    stale |= memcmp(&sc, &b->cap_scene, sizeof(SceneG)) != 0 || b->cap_tf != w->tf_dev;
    if (stale) {
      dpr_status s = wait_frames(w, b);
      if (s != DPR_OK) return s;
      b->drop_graph();
      b->uses = 0;
    }
  }
  if (moved) {
    b->h_bricks = bg;
    memcpy(b->h_desc.data() + b->off_bricks, bg.data(), bg.size() * sizeof(BrickG));
    b->built = false;
    dpr_status s = enqueue_desc(w, b, false);
    if (s != DPR_OK) return s;
    b->built = true;
  }
  return DPR_OK;
}

static void deep_key(dpr_deep_frame d, const void* ptrs[4]) {
  ptrs[0] = d ? d->counts : nullptr;
  ptrs[1] = d ? d->rgba : nullptr;
  ptrs[2] = d ? d->depth : nullptr;
  ptrs[3] = d ? d->ids : nullptr;
}

static bool same_key(const BatchState* b, dpr_world w, const dpr_camera* cams, int n, const dpr_frame* outs, int tw,
                     int th, dpr_deep_frame deep, int rank, int brick_sel) {
  if (!b || b->tile_w != tw || b->tile_h != th || (int)b->cams.size() != n || b->brick_sel != brick_sel) return false;
  const void* dp[4];
  deep_key(deep, dp);
  if (b->deep != deep || b->deep_rank != rank || memcmp(b->deep_ptrs, dp, sizeof(dp)) != 0) return false;
  if (b->geo_version != w->geo_version || b->skip != !(w->params.flags & DPR_FLAG_NO_SKIP)) return false;
  if (memcmp(b->cams.data(), cams, n * sizeof(dpr_camera)) != 0) return false;
  for (int c = 0; c < n; ++c)
    if (b->outs[c] != outs[c] || (outs[c] && (b->out_ptrs[2 * c] != outs[c]->rgba ||
                                              b->out_ptrs[2 * c + 1] != outs[c]->depth)))
      return false;
  return b->built;
}

static dpr_status check_batch_args(dpr_world w, const dpr_camera* cams, int n, const dpr_frame* outs) {
  if (!w || !cams || !outs) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_batch: NULL argument");
  if (n < 1) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_batch: n = %d", n);
  if (!w->committed) return fail(DPR_ERR_INVALID_STATE, "dpr_render_batch: world not committed");
  if (!w->tf_set) return fail(DPR_ERR_INVALID_STATE, "dpr_render_batch: no transfer function set");
  for (int c = 0; c < n; ++c) {
    dpr_status s = check_camera(&cams[c]);
    if (s != DPR_OK) return s;
    if (!outs[c]) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_batch: frame %d is NULL", c);
    if (outs[c]->w != cams[c].width || outs[c]->h != cams[c].height)
      return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_batch: frame %d size differs from its camera", c);
    if (outs[c]->dev != w->dev) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_batch: frame of another device");
  }
  for (const auto& b : w->bricks)
    if (b.dtype != w->bricks[0].dtype)
      return fail(DPR_ERR_UNSUPPORTED, "dpr_render_batch: bricks of mixed dtypes");
  if ((int)w->bricks.size() > kMaxFrags)
    return fail(DPR_ERR_UNSUPPORTED, "dpr_render_batch: more than %d bricks", kMaxFrags);
  return DPR_OK;
}

// Baseline: per camera, one plain launch per brick into full partial frames, then
// the K-frame compositor.
static dpr_status render_plain(dpr_world w, const dpr_camera* cams, int n, dpr_frame* outs) {
  if (!w->batch) w->batch = new BatchState;
  BatchState* b = w->batch;
  const int K = (int)w->bricks.size();
  const bool skip = !(w->params.flags & DPR_FLAG_NO_SKIP);
  SceneG sc = make_scene(w);
  std::vector<int32_t> ids(K);
  std::iota(ids.begin(), ids.end(), 0);
  for (int c = 0; c < n; ++c) {
    bool resize = (int)b->plain_parts.size() != K;
    for (auto f : b->plain_parts) resize |= f->w != cams[c].width || f->h != cams[c].height;
    if (resize) {
      DPR_HIP(hipStreamSynchronize(w->dev->stream));
      for (auto f : b->plain_parts) dpr_frame_release(f);
      b->plain_parts.clear();
      for (int i = 0; i < K; ++i) {
        dpr_frame f = nullptr;
        dpr_status s = dpr_frame_create(w->dev, cams[c].width, cams[c].height, &f);
        if (s != DPR_OK) return s;
        b->plain_parts.push_back(f);
      }
    }
    CamG cg = make_cam(cams[c]);
    for (int i = 0; i < K; ++i) {
      const Brick& br = w->bricks[i];
      DPR_HIP(launch_march(sc, br.device_view(skip, w->params.flags & DPR_FLAG_WIDE_OFFSETS), cg, w->tf_dev, br.dtype == DPR_F16, skip,
                           (float4*)b->plain_parts[i]->rgba, b->plain_parts[i]->depth, nullptr, w->dev->stream));
    }
    dpr_status s = composite_frames(w->dev, b->plain_parts.data(), ids.data(), K, outs[c]);
    if (s != DPR_OK) return s;
  }
  return DPR_OK;
}

static dpr_status render_batch_state(dpr_world w, BatchState* b, const dpr_camera* cams, int n, dpr_frame* outs,
                                     uint32_t flags, int tw, int th, dpr_deep_frame deep, int rank, int brick_sel) {
  dpr_status s = ensure_majorants(w);
  if (s != DPR_OK) return s;
  if (!same_key(b, w, cams, n, outs, tw, th, deep, rank, brick_sel)) {
    s = build_batch(w, b, cams, n, outs, tw, th, brick_sel);
    if (s != DPR_OK) return s;
    b->deep = deep;
    b->deep_rank = rank;
    deep_key(deep, b->deep_ptrs);
  } else {
    s = refresh_batch(w, b);
    if (s != DPR_OK) return s;
  }
  w->last_batch = b;
  b->counted = false;
  b->last_stream = w->dev->stream;
  b->used = true;
  const bool again = b->uses++ > 0;
  if (flags & DPR_FLAG_QUEUE_COVERAGE) {
    if (!b->item_count) {
      const size_t slots = (size_t)b->n_items * b->tile_w * b->tile_h;
      s = dev_alloc((void**)&b->item_count, std::max<size_t>(1, b->n_items) * sizeof(int), "queue coverage counters");
      if (s != DPR_OK) return s;
      s = dev_alloc((void**)&b->slot_count, std::max<size_t>(1, slots) * sizeof(int), "queue coverage counters");
      if (s != DPR_OK) return s;
    }
    DPR_HIP(enqueue_batch(w, b, w->dev->stream, true, true));
    b->timed = true;
    b->counted = true;
    return DPR_OK;
  }
  if (flags & DPR_FLAG_NO_GRAPH) {
    DPR_HIP(enqueue_batch(w, b, w->dev->stream, true));
    b->timed = true;
    return DPR_OK;
  }
  // a graph from the second frame on: capturing one takes as long as many frames (0.1 ms or
  // more), which a moving camera's would not earn back
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (!b->exec && again) DPR_HIP(hipStreamIsCapturing(w->dev->stream, &cs));
  if (!b->exec && (!again || cs != hipStreamCaptureStatusNone)) {
    DPR_HIP(enqueue_batch(w, b, w->dev->stream, false));
    b->timed = false;
    return DPR_OK;
  }
  if (!b->exec) {
    s = capture_graph(w, b);
    if (s != DPR_OK) return s;
  }
  DPR_HIP(hipGraphLaunch(b->exec, w->dev->stream));
  b->timed = false;
  return DPR_OK;
}

static dpr_status render_batch_tiled(dpr_world w, const dpr_camera* cams, int n, dpr_frame* outs, uint32_t flags,
                                     int tw, int th, dpr_deep_frame deep = nullptr, int rank = -1) {
  if (!w->batch) w->batch = new BatchState;
  return render_batch_state(w, w->batch, cams, n, outs, flags, tw, th, deep, rank, -1);
}

// render-parameter flags the batched paths take from the world
constexpr uint32_t kBatchFlags = DPR_FLAG_NO_GRAPH | DPR_FLAG_QUEUE_COVERAGE;

// One brick's partial frame through the persistent kernel: items of that brick
// only (one cached state per brick), every camera tile written by the tile pass
// (tiles the brick does not cover come out empty).
dpr_status render_partial_batched(dpr_world w, int id, dpr_frame out) {
  if ((int)w->partial_batch.size() < (int)w->bricks.size()) w->partial_batch.resize(w->bricks.size(), nullptr);
  if (!w->partial_batch[id]) w->partial_batch[id] = new BatchState;
  return render_batch_state(w, w->partial_batch[id], &w->cam, 1, &out, w->params.flags & kBatchFlags,
                            w->batch_tile_w, w->batch_tile_h, nullptr, -1, id);
}

dpr_status render_frame_batched(dpr_world w, dpr_frame out) {
  return render_batch_tiled(w, &w->cam, 1, &out, w->params.flags & kBatchFlags, w->batch_tile_w,
                            w->batch_tile_h);
}

static dpr_status render_deep(dpr_world w, int rank, dpr_deep_frame out) {
  dpr_frame none = nullptr;
  dpr_status s = render_batch_tiled(w, &w->cam, 1, &none, w->params.flags & kBatchFlags, w->batch_tile_w,
                                    w->batch_tile_h, out, rank);
  if (s != DPR_OK) return s;
  out->rank = rank;
  return DPR_OK;
}

}  // namespace dpr

using namespace dpr;

extern "C" {

dpr_status dpr_render_batch(dpr_world w, const dpr_camera* cams, int32_t n, dpr_frame* outs, uint32_t flags) {
  dpr_status s = check_batch_args(w, cams, n, outs);
  if (s != DPR_OK) return s;
  if (flags & DPR_FLAG_PLAIN) {
    s = ensure_majorants(w);
    if (s != DPR_OK) return s;
    return render_plain(w, cams, n, outs);
  }
  return render_batch_tiled(w, cams, n, outs, flags, w->batch_tile_w, w->batch_tile_h);
}

dpr_status dpr_render_deep(dpr_world w, int32_t rank, dpr_deep_frame out) {
  if (!w || !out) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_deep: NULL argument");
  if (!w->committed) return fail(DPR_ERR_INVALID_STATE, "dpr_render_deep: world not committed");
  if (!w->tf_set) return fail(DPR_ERR_INVALID_STATE, "dpr_render_deep: no transfer function set");
  if (!w->cam_set) return fail(DPR_ERR_INVALID_STATE, "dpr_render_deep: no camera set");
  if (rank < 0 || rank >= 32768) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_deep: rank %d", rank);
  if (out->dev != w->dev) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_deep: frame of another device");
  if (out->w != w->cam.width || out->h != w->cam.height)
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_deep: frame %dx%d != camera %dx%d", out->w, out->h,
                w->cam.width, w->cam.height);
  if (out->cap < (int)w->bricks.size())
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_render_deep: capacity %d < %d bricks", out->cap,
                (int)w->bricks.size());
  for (const auto& b : w->bricks)
    if (b.dtype != w->bricks[0].dtype) return fail(DPR_ERR_UNSUPPORTED, "dpr_render_deep: bricks of mixed dtypes");
  return render_deep(w, rank, out);
}

dpr_status dpr_batch_timings(dpr_world w, float* march_ms, float* composite_ms) {
  if (!w) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_batch_timings: NULL world");
  BatchState* b = w->last_batch;
  if (!b || !b->timed || !b->ev[0])
    return fail(DPR_ERR_INVALID_STATE, "dpr_batch_timings: the last batched render was not enqueued directly");
  DPR_HIP(hipEventSynchronize(b->ev[2]));
  float a = 0.f, c = 0.f;
  DPR_HIP(hipEventElapsedTime(&a, b->ev[0], b->ev[1]));
  DPR_HIP(hipEventElapsedTime(&c, b->ev[1], b->ev[2]));
  if (march_ms) *march_ms = a;
  if (composite_ms) *composite_ms = c;
  return DPR_OK;
}

dpr_status dpr_batch_coverage(dpr_world w, int64_t out[4]) {
  if (!w || !out) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_batch_coverage: NULL argument");
  BatchState* b = w->last_batch;
  if (!b || !b->counted)
    return fail(DPR_ERR_INVALID_STATE, "dpr_batch_coverage: the last batched render did not count its queue");
  const size_t slots = (size_t)b->n_items * b->tile_w * b->tile_h;
  std::vector<int> items(b->n_items), marks(slots);
  DPR_HIP(hipStreamSynchronize(w->dev->stream));
  if (b->n_items > 0) {
    DPR_HIP(hipMemcpy(items.data(), b->item_count, items.size() * sizeof(int), hipMemcpyDeviceToHost));
    DPR_HIP(hipMemcpy(marks.data(), b->slot_count, marks.size() * sizeof(int), hipMemcpyDeviceToHost));
  }
  out[0] = (int64_t)items.size();
  out[1] = std::count(items.begin(), items.end(), 1);
  out[2] = (int64_t)marks.size();
  out[3] = std::count(marks.begin(), marks.end(), 1);
  return DPR_OK;
}

dpr_status dpr_set_batch_tile(dpr_world w, int32_t tw, int32_t th) {
  if (!w) return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_set_batch_tile: NULL world");
  if (tw < 1 || th < 1 || (tw * th) % 64 != 0 || tw * th > 1024)
    return fail(DPR_ERR_INVALID_ARGUMENT, "dpr_set_batch_tile: %dx%d is not a multiple of 64 pixels <= 1024", tw, th);
  w->batch_tile_w = tw;
  w->batch_tile_h = th;
  return DPR_OK;
}

dpr_status dpr_autotune_batch(dpr_world w, const dpr_camera* cams, int32_t n, dpr_frame* outs, int32_t* tw_out,
                              int32_t* th_out) {
  dpr_status s = check_batch_args(w, cams, n, outs);
  if (s != DPR_OK) return s;
  // the persisted choice for this device and shape of work, if any
  const char* cache = getenv("DPR_TUNE_CACHE");
  std::string key;
  if (cache && cache[0]) {
    const Brick& b0 = w->bricks[0];
    key = "gfx950 cu" + std::to_string(w->dev->cu_count) +
          (b0.dtype == DPR_F16 ? (b0.half16 ? " f16-2byte" : " f16-pairs") : " f32") + " bricks";
    for (const auto& br : w->bricks)
      key += " " + std::to_string(br.sdim[0]) + "x" + std::to_string(br.sdim[1]) + "x" + std::to_string(br.sdim[2]);
    key += " cameras";
    for (int c = 0; c < n; ++c) key += " " + std::to_string(cams[c].width) + "x" + std::to_string(cams[c].height);
    char prm[128];
    snprintf(prm, sizeof prm, " step %g ert %g mc %d flags %u", w->params.step_voxels, w->params.ert_threshold,
             w->params.macrocell_cells, w->params.flags & (DPR_FLAG_NO_SKIP | DPR_FLAG_WIDE_OFFSETS));
    key += prm;
    int32_t found = 0, cw = 0, ch = 0;
    s = dpr_tune_cache_lookup(cache, key.c_str(), &found, &cw, &ch);
    if (s != DPR_OK) return s;
    if (found && dpr_set_batch_tile(w, cw, ch) == DPR_OK) {
      s = render_batch_tiled(w, cams, n, outs, 0, cw, ch);  // leave the chosen shape built
      if (s != DPR_OK) return s;
      if (tw_out) *tw_out = cw;
      if (th_out) *th_out = ch;
      return DPR_OK;
    }
  }
  static const int cand[][2] = {{8, 8}, {16, 8}, {16, 16}, {32, 16}, {32, 32}};
  hipEvent_t e0, e1;
  DPR_HIP(hipEventCreate(&e0));
  DPR_HIP(hipEventCreate(&e1));
  float best = 1e30f;
  int bw = w->batch_tile_w, bh = w->batch_tile_h;
  for (const auto& c : cand) {
    s = render_batch_tiled(w, cams, n, outs, 0, c[0], c[1]);  // build
    if (s != DPR_OK) break;
    s = render_batch_tiled(w, cams, n, outs, 0, c[0], c[1]);  // capture + warm-up
    if (s != DPR_OK) break;
    DPR_HIP(hipEventRecord(e0, w->dev->stream));
    for (int r = 0; r < 3; ++r) {
      s = render_batch_tiled(w, cams, n, outs, 0, c[0], c[1]);
      if (s != DPR_OK) break;
    }
    DPR_HIP(hipEventRecord(e1, w->dev->stream));
    DPR_HIP(hipEventSynchronize(e1));
    float ms = 0.f;
    DPR_HIP(hipEventElapsedTime(&ms, e0, e1));
    if (log_enabled()) fprintf(stderr, "[dpr] autotune tile %dx%d: %.3f ms\n", c[0], c[1], ms / 3);
    if (ms < best) {
      best = ms;
      bw = c[0];
      bh = c[1];
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (s != DPR_OK) return s;
  w->batch_tile_w = bw;
  w->batch_tile_h = bh;
  s = render_batch_tiled(w, cams, n, outs, 0, bw, bh);  // leave the chosen shape built
  if (s != DPR_OK) return s;
  if (!key.empty()) {
    s = dpr_tune_cache_store(cache, key.c_str(), bw, bh);
    if (s != DPR_OK) return s;
  }
  if (tw_out) *tw_out = bw;
  if (th_out) *th_out = bh;
  return DPR_OK;
}

}  // extern "C"
