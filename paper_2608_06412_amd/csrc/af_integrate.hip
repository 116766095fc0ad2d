// Per-frame integration kernels: quantisation, block allocation in the hash
// map, scan-centric cube accumulation (Section 3.2), ray-cleared band
// (Section 3.4, "Arm path checking"), surface points (Section 3.1), the fold
// with the weight cap (Section 3.6) and the brick grid used by scoring.
#include "af_internal.h"

#include <algorithm>

#pragma clang fp contract(off)

namespace af {
namespace {

constexpr int kThreads = 256;

__device__ inline int lane_id() { return (int)(threadIdx.x & 63u); }

// Insert `key`; returns its slot (fresh = newly inserted) or -1 if full.
__device__ int32_t hash_insert(HashTable t, int64_t key, bool &fresh) {
  uint32_t s = slot_of(key, t.mask);
  for (uint32_t i = 0; i <= t.mask; ++i) {
    // (a cached read: a key, once there, stays for the whole kernel, and where
    // the read still says "free" the exchange below has the last word)
    int64_t cur = __hip_atomic_load(&t.keys[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    if (cur == key) {
      fresh = false;
      return (int32_t)s;
    }
    if (cur == kEmpty) {
      unsigned long long prev = atomicCAS((unsigned long long *)&t.keys[s],
                                          (unsigned long long)kEmpty,
                                          (unsigned long long)key);
      if ((int64_t)prev == kEmpty) {
        fresh = true;
        return (int32_t)s;
      }
      if ((int64_t)prev == key) {
        fresh = false;
        return (int32_t)s;
      }
    }
    s = (s + 1) & t.mask;
  }
  fresh = false;
  return -1;
}

// Exact floor(sqrt(n)) for 0 <= n < 2^62.
__device__ inline int64_t isqrt64(int64_t n) {
  if (n <= 0) return 0;
  uint64_t u = (uint64_t)n;
  uint64_t r = (uint64_t)__builtin_sqrt((double)n);
  while (r * r > u) --r;
  while ((r + 1) * (r + 1) <= u) ++r;
  return (int64_t)r;
}

// a / b to nearest, halves away from zero (b > 0), for |a / b| < 2^12 and
// b < 2^30.  The quotient of doubles truncates right: 2 |a| + b < 2^43 is
// exact, and a quotient below an integer is so by at least 1 / 2b > 2^-32,
// far more than a double's last bit.  (A 64-bit division takes some 150
// instructions, this one 20; a return needs up to 54.)
__device__ inline int64_t div_round(int64_t a, int64_t b) {
  int64_t m = a < 0 ? -a : a;
  int64_t q = (int64_t)((double)(2 * m + b) / (double)(2 * b));
  return a < 0 ? -q : q;
}

__device__ inline int64_t div_floor(int64_t a, int64_t b) {
  int64_t q = a / b;
  if ((a % b != 0) && ((a < 0) != (b < 0))) --q;
  return q;
}

__device__ inline void wave_count(unsigned long long *ctr, bool flag) {
  unsigned long long b = __ballot(flag);
  if (lane_id() == 0 && b) atomicAdd(ctr, (unsigned long long)__popcll(b));
}

// Blocks per axis that a cube of 2 R + 1 voxels can span.
__host__ __device__ inline int span_side(int R) { return (2 * R + 7) / 8 + 1; }

// Band samples of a return: distances tau + 128 (j + 1) up to 2.25 tau.
__device__ inline int band_samples(int tau_u) {
  int j = 0;
  while (j < kMaxBand && 4 * ((int64_t)tau_u + 128 * (j + 1)) <= 9 * (int64_t)tau_u) ++j;
  return j;
}

__device__ inline bool in_box(int32_t bx, int32_t by, int32_t bz, int3 lo, int3 hi) {
  return bx >= lo.x && bx <= hi.x && by >= lo.y && by <= hi.y && bz >= lo.z && bz <= hi.z;
}

// The per-return kernels (prep, touch, bin) run kParts waves per 64 returns:
// lane = return, and the waves share out its cube's blocks and its band
// samples.  A return's chain of dependent map reads is what they wait for, and
// a frame of 20,000 returns is 313 waves with one thread a return, one wave a
// CU.  Entry i of return r lies at [i * cap + r], so a wave reads lines.
constexpr int kParts = 8;
constexpr int kPartThreads = 64 * kParts;

// --------------------------------------------------------------- prep
// Quantise each return, insert the blocks of its cube and of its band
// samples, and insert its voxel into the point set.  (20,000 returns, a tree
// frame: 60 -> 18 us.)
__global__ void __launch_bounds__(kPartThreads)
k_frame_prep(const float *__restrict__ xyz, const FrameArgs *fa, Params p, MapDev m,
             PointsDev pts, FrameScratch fs, FrameCounters *c) {
  const int64_t n = fa->n, cap = fs.cap;
  const int3 Q = fa->Q;
  const int3 wlo = fa->wlo, whi = fa->whi;
  const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t r = (int64_t)blockIdx.x * 64 + lane_id();
  const bool in = r < n;
  bool ok = in;
  int P[3] = {0, 0, 0};
  if (in) {
    for (int i = 0; i < 3; ++i) {
      double t = (double)xyz[3 * r + i] * p.scale;
      if (!(fabs(t) <= (double)kCoordLim))
        ok = false;
      else
        P[i] = (int)__builtin_rint(t);
    }
    if (ok && P[0] == Q.x && P[1] == Q.y && P[2] == Q.z) ok = false;
  }
  if (part == 0) {
    wave_count(&c->n_valid, ok);
    wave_count(&c->n_dropped, in && !ok);
  }
  if (!in) return;
  int64_t g[3] = {(int64_t)Q.x - P[0], (int64_t)Q.y - P[1], (int64_t)Q.z - P[2]};
  const int64_t L = ok ? isqrt64(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]) : 0;
  if (part == 0) fs.P[r] = make_int4(P[0], P[1], P[2], (int)L);

  bool full = false;
  // blocks of the cube (-1: none, or outside the window)
  const int side = span_side(p.R);
  int lo[3], hi[3];
  for (int a = 0; a < 3; ++a) {
    lo[a] = ((P[a] >> 8) - p.R) >> 3;
    hi[a] = ((P[a] >> 8) + p.R) >> 3;
  }
  for (int i = part; i < side * side * side; i += kParts) {
    const int bx = lo[0] + i % side, by = lo[1] + i / side % side, bz = lo[2] + i / (side * side);
    int32_t s = -1;
    if (ok && bx <= hi[0] && by <= hi[1] && bz <= hi[2] && in_box(bx, by, bz, wlo, whi)) {
      bool fresh;
      s = hash_insert(m.h, pack_key(bx, by, bz), fresh);
      if (s < 0) full = true;
      if (fresh) fs.new_blocks[atomicAdd(&c->n_new_blocks, 1)] = s;
    }
    fs.span[i * cap + r] = s;
  }
  // band samples: (tau, 2.25 tau] back towards the sensor, every v/2
  const int nband = band_samples(p.tau_u);
  for (int j = part; j < nband; j += kParts) {
    const int64_t lam = (int64_t)p.tau_u + 128 * (j + 1);
    int32_t s = -2;   // no sample, or outside the window: neither marked nor counted
    if (lam < L) {
      const int vx = (int)((P[0] + div_round(lam * g[0], L)) >> 8);
      const int vy = (int)((P[1] + div_round(lam * g[1], L)) >> 8);
      const int vz = (int)((P[2] + div_round(lam * g[2], L)) >> 8);
      if (in_box(vx >> 3, vy >> 3, vz >> 3, wlo, whi)) {
        bool fresh;
        s = hash_insert(m.h, pack_key(vx >> 3, vy >> 3, vz >> 3), fresh);
        if (s < 0) full = true;
        if (fresh) fs.new_blocks[atomicAdd(&c->n_new_blocks, 1)] = s;
        fs.band[(2 * j + 1) * cap + r] = (vx & 7) | ((vy & 7) << 3) | ((vz & 7) << 6);
      }
    }
    fs.band[2 * j * cap + r] = s;
  }
  // the return's voxel is a surface point (inside the window)
  if (part == kParts - 1 && ok) {
    int32_t ps = -1;
    if (in_box(P[0] >> 11, P[1] >> 11, P[2] >> 11, wlo, whi)) {
      const int64_t key = pack_key(P[0] >> 8, P[1] >> 8, P[2] >> 8);
      bool fresh;
      ps = hash_insert(pts.h, key, fresh);
      if (ps < 0) full = true;
      if (fresh) {
        int at = atomicAdd(&c->n_new_points, 1);
        fs.new_keys[at] = key;
        fs.new_kslot[at] = ps;
      }
    }
    fs.pslot[r] = ps;
  }
  if (full) atomicOr(&c->status, kStatusHashFull);
}

// The frame's arguments (fa_new.n >= 0: an eager frame's; a recorded frame
// has them already) and zeroed counters.
__global__ void k_reset_counters(FrameCounters *c, MapDev m, PointsDev pts, FrameArgs *fa,
                                 FrameArgs fa_new) {
  if (threadIdx.x < 3 * kStatSlots) c->fold[threadIdx.x / 3][threadIdx.x % 3] = 0ull;
  if (threadIdx.x != 0) return;
  if (fa_new.n >= 0) *fa = fa_new;
  c->n_valid = c->n_dropped = c->pairs_applied = c->pairs_excluded = 0;
  c->band_marks = c->voxels_folded = 0;
  c->n_new_blocks = c->n_touched = c->n_new_points = c->status = 0;
  c->n_changed = c->n_binned = c->held = 0;
  for (int i = 0; i < 3; ++i) {
    c->bmin[i] = 0x7fffffff;
    c->bmax[i] = -0x7fffffff - 1;
  }
  c->blocks_before = *m.n_blocks;
  c->points_before = *pts.n_points;
  c->free_before = m.n_free ? *m.n_free : 0;
}

// One workgroup per new block: assign its id and clear its voxels.
__global__ void __launch_bounds__(kThreads)
k_assign_blocks(MapDev m, FrameScratch fs, FrameCounters *c, const FrameArgs *fa, int3 glo, int3 ghi) {
  const int32_t frame = fa->frame;
  int n_new = c->n_new_blocks;
  int64_t base = *m.n_blocks;
  const int nfree = c->free_before;   // evicted ids first (sliding window)
  for (int i = blockIdx.x; i < n_new; i += gridDim.x) {
    int32_t slot = fs.new_blocks[i];
    int64_t id = i < nfree ? (int64_t)m.free_ids[nfree - 1 - i] : base + (i - nfree);
    if (id >= m.max_blocks) {
      if (threadIdx.x == 0) {
        m.h.vals[slot] = -1;
        atomicOr(&c->status, kStatusBlockOverflow);
      }
      continue;
    }
    if (threadIdx.x == 0) {
      m.h.vals[slot] = (int32_t)id;
      int64_t k = m.h.keys[slot];
      m.bkey[id] = k;
      m.touched[id] = -1;
      m.tpos[id] = 0;
      int32_t b[3];
      unpack_key(k, b[0], b[1], b[2]);
      for (int a = 0; a < 3; ++a) {
        atomicMin(&c->bmin[a], b[a]);
        atomicMax(&c->bmax[a], b[a]);
      }
      if (!in_box(b[0], b[1], b[2], glo, ghi)) atomicOr(&c->held, 1);
    }
    for (int t = threadIdx.x; t < kBlockVox; t += kThreads) {
      m.S[id * kBlockVox + t] = 0;
      m.W[id * kBlockVox + t] = 0;
    }
    if (threadIdx.x < 16) {
      m.clr[id * 16 + threadIdx.x] = 0;
      m.surf[id * 16 + threadIdx.x] = 0;
    }
  }
}

// Lanes with the same id >= 0 share one add on its counter: atomics on one
// address take turns, some 13 ns each.  A lane's leader is the last lane that
// entered itself at the id's place in a table of the wave's (a lane that finds
// another id there leads itself: two groups of one id only cost an add).
// Returns the lane's own rank; first: its block's first return of the frame.
// (Going through the wave's distinct ids one by one took 64 turns where a
// frame's returns come in no order: cluster frame of 40,000 48 -> 43 us, tree frame 32 -> 26.)
__device__ inline int grouped_add(int32_t *counter, int32_t id, bool &first, int *table, int *sizes) {
  const int lane = lane_id();
  const auto order = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  const int place = (int)(((uint32_t)id * 0x9E3779B1u) >> 26);
  sizes[lane] = 0;
  if (id >= 0) __hip_atomic_store(&table[place], lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  order();
  int leader = id >= 0 ? __hip_atomic_load(&table[place], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : lane;
  const int32_t theirs = __shfl(id, leader);
  leader = theirs == id ? leader : lane;
  const int own = id >= 0 ? atomicAdd(&sizes[leader], 1) : 0;
  order();
  const int size = __hip_atomic_load(&sizes[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  int base = 0;
  if (id >= 0 && leader == lane) base = atomicAdd(&counter[id], size);
  base = __shfl(base, leader);
  first = base + own == 0;
  return base + own;
}

// Mark every block of the frame touched (once), rank each return among those
// of each block of its cube, and set the band's cleared bits.  m.tpos counts a
// block's returns here (0 between frames), then holds the start of its bin.
// The blocks' ids replace their slots in fs.span.  Marks and cleared bits that
// are there already (a cached read tells) take no atomic.  (A cluster frame of
// 40,000 returns: touch 123 and bin count 46 -> 43 us.)
__global__ void __launch_bounds__(kPartThreads)
k_touch_band(const FrameArgs *fa, Params p, MapDev m, FrameScratch fs, FrameCounters *c) {
  const int64_t n = fa->n, cap = fs.cap;
  const int32_t frame = fa->frame;
  const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t r = (int64_t)blockIdx.x * 64 + lane_id();
  if (((int64_t)blockIdx.x * 64 >= n) | (c->held != 0)) return;
  __shared__ int32_t s_new[64 * (kMaxSpan + kMaxBand)];   // blocks this workgroup touched first
  __shared__ int s_count[3];                              // those, their place in the list, marks
  __shared__ int s_group[kParts][2][64];                  // see grouped_add
  if (threadIdx.x < 3) s_count[threadIdx.x] = 0;
  __syncthreads();
  auto touch = [&](int32_t id) {
    if (__hip_atomic_load(&m.touched[id], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT) == frame ||
        atomicExch(&m.touched[id], frame) == frame)
      return;
    s_new[atomicAdd(&s_count[0], 1)] = id;
  };
  const int side = span_side(p.R);
  for (int i = part; i < side * side * side; i += kParts) {
    const int32_t s = r < n ? fs.span[i * cap + r] : -1;
    const int32_t id = s >= 0 ? m.h.vals[s] : -1;
    bool first;
    const int rank = grouped_add(m.tpos, id, first, s_group[part][0], s_group[part][1]);
    if (r < n) {
      fs.span[i * cap + r] = id;
      fs.rank[i * cap + r] = rank;
    }
    if (id >= 0 && first) touch(id);
  }
  const int nband = band_samples(p.tau_u);
  int marks = 0;
  for (int j = part; j < nband; j += kParts) {
    const int32_t s = r < n ? fs.band[2 * j * cap + r] : -2;
    marks += (int)__popcll(__ballot(s != -2));
    const int32_t id = s >= 0 ? m.h.vals[s] : -1;
    if (id < 0) continue;
    const int vi = fs.band[(2 * j + 1) * cap + r];
    uint32_t *w = &m.clr[(int64_t)id * 16 + (vi >> 5)];
    const uint32_t bit = 1u << (vi & 31);
    if (!(__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT) & bit))
      atomicOr(w, bit);
    touch(id);
  }
  if (lane_id() == 0 && marks) atomicAdd(&s_count[2], marks);
  __syncthreads();
  const int found = s_count[0];
  if (threadIdx.x == 0) {
    if (found) s_count[1] = atomicAdd(&c->n_touched, found);
    if (s_count[2]) atomicAdd(&c->band_marks, (unsigned long long)s_count[2]);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < found; i += kPartThreads) fs.touched[s_count[1] + i] = s_new[i];
}

// ---------------------------------------------------------------- points
// New point keys of the frame get ids in ascending key order (rank by
// counting smaller keys), are initialised and flagged in their block.
// New points are appended in key order.  Each workgroup first sorts its
// tile of (distinct) new keys in LDS with Batcher's bitonic network; a key's
// rank among all new keys is then the sum of its lower bounds in the tiles.
__global__ void __launch_bounds__(kThreads)
k_sort_new_tiles(FrameScratch fs, const FrameCounters *c) {
  static_assert((kThreads & (kThreads - 1)) == 0, "bitonic tile needs a power of two");
  __shared__ int64_t v[kThreads];
  const int m = c->n_new_points;
  const int base = blockIdx.x * kThreads;
  if ((base >= m) | (c->held != 0)) return;
  const int t = threadIdx.x;
  v[t] = base + t < m ? fs.new_keys[base + t] : (int64_t)0x7fffffffffffffffLL;
  __syncthreads();
  for (int k = 2; k <= kThreads; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int q = t ^ j;
      if (q > t) {
        const int64_t a = v[t], b = v[q];
        if ((a > b) == ((t & k) == 0)) {
          v[t] = b;
          v[q] = a;
        }
      }
      __syncthreads();
    }
  fs.new_sorted[base + t] = v[t];
}

// 64 keys a workgroup, its waves sharing out the tiles (each a search of 8
// dependent reads): with every thread going through all the tiles the search
// of a tree frame's keys took 19.5 us, now 8.6.
constexpr int kAppendWaves = 16;
__global__ void __launch_bounds__(64 * kAppendWaves)
k_points_append(MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c, const FrameArgs *fa) {
  const int32_t frame = fa->frame;
  __shared__ int s_rank[kAppendWaves][64];
  const int mcount = c->n_new_points;
  const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
  const int i = blockIdx.x * 64 + lane;
  if (((int)(blockIdx.x * 64) >= mcount) | (c->held != 0)) return;
  const int64_t key = fs.new_keys[i < mcount ? i : 0];
  int part = 0;
  for (int base = wave * kThreads; base < mcount; base += kAppendWaves * kThreads) {
    int lo = 0, hi = mcount - base < kThreads ? mcount - base : kThreads;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (fs.new_sorted[base + mid] < key) lo = mid + 1;
      else hi = mid;
    }
    part += lo;
  }
  s_rank[wave][lane] = part;
  __syncthreads();
  if (wave != 0 || i >= mcount) return;
  int rank = 0;
  for (int w = 0; w < kAppendWaves; ++w) rank += s_rank[w][lane];
  int64_t id = (int64_t)*pts.n_points + rank;
  int32_t slot = fs.new_kslot[i];
  if (id >= pts.max_points) {
    pts.h.vals[slot] = -1;
    atomicOr(&c->status, kStatusPointOverflow);
    return;
  }
  pts.h.vals[slot] = (int32_t)id;
  pts.key[id] = key;
  pts.first[id] = frame;
  pts.last[id] = -1;
  pts.nvp[id] = 0;
  pts.head[id] = 0;
  pts.nq[id] = 0;
  pts.sumq[3 * id] = pts.sumq[3 * id + 1] = pts.sumq[3 * id + 2] = 0;
  pts.has_normal[id] = -1;
  int32_t x, y, z;
  unpack_key(key, x, y, z);
  int32_t bs = hash_find(m.h, pack_key(x >> 3, y >> 3, z >> 3));
  int32_t bid = bs >= 0 ? m.h.vals[bs] : -1;
  int vi = (x & 7) | ((y & 7) << 3) | ((z & 7) << 6);
  pts.addr[id] = bid >= 0 ? bid * kBlockVox + vi : -1;
  if (bid >= 0) atomicOr(&m.surf[(int64_t)bid * 16 + (vi >> 5)], 1u << (vi & 31));
}

// Once per (point, frame): running sensor sum and the viewpoint ring.
__device__ inline void point_view(int64_t r, int3 Q, int32_t frame, const Params &p,
                                  const PointsDev &pts, const FrameScratch &fs) {
  if (fs.P[r].w == 0) return;
  int32_t s = fs.pslot[r];
  int32_t id = s >= 0 ? pts.h.vals[s] : -1;
  if (id < 0 || atomicExch(&pts.last[id], frame) == frame) return;
  pts.sumq[3 * (int64_t)id] += Q.x;
  pts.sumq[3 * (int64_t)id + 1] += Q.y;
  pts.sumq[3 * (int64_t)id + 2] += Q.z;
  pts.nq[id] += 1;
  int cnt = pts.nvp[id], head = pts.head[id];
  bool store = true;
  if (cnt > 0) {
    int last = (head + p.n_vp - 1) % p.n_vp;
    const int32_t *v = pts.vp + ((int64_t)id * kMaxVp + last) * 3;
    int64_t d0 = (int64_t)Q.x - v[0], d1 = (int64_t)Q.y - v[1], d2 = (int64_t)Q.z - v[2];
    store = d0 * d0 + d1 * d1 + d2 * d2 > p.dmin2;
  }
  if (store) {
    int32_t *v = pts.vp + ((int64_t)id * kMaxVp + head) * 3;
    v[0] = Q.x;
    v[1] = Q.y;
    v[2] = Q.z;
    pts.head[id] = (head + 1) % p.n_vp;
    pts.nvp[id] = cnt < p.n_vp ? cnt + 1 : cnt;
  }
}

// ------------------------------------------------------------ fold/bricks
// Two-bit code of one voxel: bit 0 TSDF < r_c, bit 1 unknown and not cleared.
__device__ inline uint32_t voxel_code(const Params &p, int32_t S, int32_t W, bool cleared) {
  bool occ = W > 0 && (int64_t)S < (int64_t)p.rc_u * W;
  bool unk = W == 0 && !cleared;
  return (occ ? 1u : 0u) | (unk ? 2u : 0u);
}

// Bit i of the low 16 to bit 2 i.
__device__ inline uint32_t spread16(uint32_t x) {
  x = (x | (x << 8)) & 0x00FF00FFu;
  x = (x | (x << 4)) & 0x0F0F0F0Fu;
  x = (x | (x << 2)) & 0x33333333u;
  return (x | (x << 1)) & 0x55555555u;
}

// The workgroups that walk blocks have kFoldThreads threads: thread t holds
// the voxels t + kFoldThreads h (h < kFoldVox), a wave whole z slices.
constexpr int kFoldThreads = 512, kFoldVox = kBlockVox / kFoldThreads;
constexpr int kFoldWaves = kFoldThreads / 64;

// A block written to its brick of the grid.  A wave holds z slices (64
// voxels, lane = x | y << 3), so every plane's words come from its ballots;
// only the octant bits need the other waves: s_occ4 is workgroup scratch that
// the caller zeroed (thread 0) before its last barrier, and that thread 0
// alone reads here.  clrw is the block's cleared-bit word of this thread's
// voxels, surfw (threads 32..47) its surface word t - 32, both loaded by the
// caller (early, so the loads overlap other work); bkey its key.
__device__ inline void write_brick(const Params &p, GridDev g, const int32_t S[kFoldVox],
                                   const int32_t W[kFoldVox], uint32_t *s_occ4,
                                   const uint32_t clrw[kFoldVox], uint32_t surfw, int64_t bkey) {
  const int t = threadIdx.x, lane = lane_id();
  int32_t b[3];
  unpack_key(bkey, b[0], b[1], b[2]);
  const int x = b[0] - g.g0[0], y = b[1] - g.g0[1], z = b[2] - g.g0[2];
  const bool inside = (unsigned)x < (unsigned)g.gd[0] && (unsigned)y < (unsigned)g.gd[1] &&
                      (unsigned)z < (unsigned)g.gd[2];
  const int64_t brick = ((int64_t)z * g.gd[1] + y) * g.gd[0] + x;
  for (int h = 0; h < kFoldVox; ++h) {
    const int slice = (t >> 6) + kFoldWaves * h;
    const uint32_t cd = voxel_code(p, S[h], W[h], (clrw[h] >> (t & 31)) & 1u);
    const uint64_t occ = __ballot(cd & 1u), unk = __ballot(cd & 2u);
    // the slice's four 4 x 4 quadrants: the low or high half of the brick's octants
    const uint32_t nib = (uint32_t)((occ & 0x000000000F0F0F0Full) != 0) |
                         ((uint32_t)((occ & 0x00000000F0F0F0F0ull) != 0) << 1) |
                         ((uint32_t)((occ & 0x0F0F0F0F00000000ull) != 0) << 2) |
                         ((uint32_t)((occ & 0xF0F0F0F000000000ull) != 0) << 3);
    if (lane == 0 && nib) atomicOr(s_occ4, nib << (4 * (slice >> 2)));
    if (!inside) continue;
    if (lane < 4) {   // 16 voxels a word
      const uint32_t lo = (uint32_t)(occ >> (16 * lane)) & 0xFFFFu;
      const uint32_t hi = (uint32_t)(unk >> (16 * lane)) & 0xFFFFu;
      g.pred[brick * 32 + 4 * slice + lane] = spread16(lo) | (spread16(hi) << 1);
    } else if (lane < 6) {
      g.occ1[brick * 16 + 2 * slice + (lane - 4)] = (uint32_t)(occ >> (32 * (lane - 4)));
    }
  }
  if (inside && t >= 32 && t < 48) g.surf[brick * 16 + (t - 32)] = surfw;
  __syncthreads();
  if (inside && t == 0) {
    const uint32_t any = *s_occ4, bit = 1u << (brick & 31);
    if (any)
      atomicOr(&g.occ_any[brick >> 5], bit);
    else
      atomicAnd(&g.occ_any[brick >> 5], ~bit);
    g.occ4[brick] = (uint8_t)any;
  }
}

// ---------------------------------------------------- binned integration
// Section 3.2 as a gather: every (return, block of its cube) pair is binned
// by block; one workgroup per touched block then sums the clamped distances
// of the block's returns (cone test, isqrt) in LDS.  The fold with the weight
// cap (Section 3.6) and the block's brick follow in the same workgroup, so
// the map sees one plain store per voxel and no atomics.

// The ids that k_assign_blocks gave out become part of the map.
__device__ inline void commit_blocks(const MapDev &m, const FrameCounters *c) {
  int64_t add = c->n_new_blocks, at = *m.n_blocks;
  const int64_t nfree = c->free_before;
  if (m.n_free) *m.n_free = (int32_t)(add < nfree ? nfree - add : 0);
  add = add > nfree ? add - nfree : 0;
  if (at + add > m.max_blocks) add = m.max_blocks - at;
  *m.n_blocks = (int32_t)(at + add);
}

// The bins' places: any order will do, so each wave takes room for 64 blocks
// at once.  (A prefix sum in one workgroup took 15 us on a tree frame, this 4.)
// The frame's new ids also become part of the map here: nothing between the
// assignment and this kernel reads the counts as they were, nothing after.
__global__ void __launch_bounds__(kThreads)
k_bin_place(MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c) {
  const int nt = c->n_touched;   // (0 in a frame that is held)
  const int lane = lane_id();
  for (int j0 = (blockIdx.x * kThreads + threadIdx.x) & ~63; j0 < nt; j0 += gridDim.x * kThreads) {
    const int j = j0 + lane;
    const int32_t id = j < nt ? fs.touched[j] : 0;
    const int cnt = j < nt ? m.tpos[id] : 0;
    int incl = cnt;
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    int base = 0;
    if (lane == 63) base = atomicAdd(&c->n_binned, incl);
    base = __shfl(base, 63) + incl - cnt;
    if (j < nt) {
      fs.bin[j] = make_int2(base, cnt);
      m.tpos[id] = base;
    }
  }
  if (blockIdx.x != 0 || threadIdx.x != 0 || c->held) return;
  commit_blocks(m, c);
  int64_t at = *pts.n_points, add = c->n_new_points;
  if (at + add > pts.max_points) add = pts.max_points - at;
  *pts.n_points = (int32_t)(at + add);
}

// Each return into the bins of its blocks, and its viewpoint to its point.
__global__ void __launch_bounds__(kPartThreads)
k_bin_fill(const FrameArgs *fa, Params p, MapDev m, PointsDev pts, FrameScratch fs,
           const FrameCounters *c) {
  const int64_t n = fa->n, cap = fs.cap;
  const int part = (int)(threadIdx.x >> 6);
  const int64_t r = (int64_t)blockIdx.x * 64 + lane_id();
  if ((r >= n) | (c->held != 0)) return;
  const int side = span_side(p.R);
  for (int i = part; i < side * side * side; i += kParts) {
    const int32_t id = fs.span[i * cap + r];
    if (id >= 0) fs.bin_list[m.tpos[id] + fs.rank[i * cap + r]] = (int32_t)r;
  }
  if (part == kParts - 1) point_view(r, fa->Q, fa->frame, p, pts, fs);
}

// A frame that ends after its blocks got their ids: the blocks stay in the map,
// unknown voxels that they are, and the frame's new point keys leave the hash
// again.  (They are the last ones that entered it, so every other key is found
// as before, and the slots they took are free as before.)
__global__ void __launch_bounds__(kThreads)
k_frame_stop(MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c) {
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < c->n_new_points; i += gridDim.x * kThreads)
    pts.h.keys[fs.new_kslot[i]] = kEmpty;
  if (blockIdx.x == 0 && threadIdx.x == 0) commit_blocks(m, c);
}

// A block's returns are dealt to its workgroup's eight waves; a wave takes up
// to 64 of them at once, a lane each (its box of voxels in the block, the
// return's place and direction), then goes through them one by one, a lane
// per voxel of the box.  A thread per voxel of the block that tests every
// return of the bin, as before, has half the waves skip and the others run a
// third full: a cube covers 4.5^3 of the block's 8^3 voxels on average.  The
// cone test is made in float first (a is exact, a.u within 2^-20.6 |a|, so q
// within 2^-19.6 |a|^2, compared with a margin of 2^-16) and in integers where
// that does not decide.  The vector ALU and, where a block has few returns,
// its chain of reads bound it: 64 registers a lane, so that four workgroups
// share a CU.  (Tree frame of 20,000 returns 149 -> 82 us, cluster frame
// of 40,000 202 -> 68, 2,000 returns on 200 blocks 47 -> 18; with 256 threads
// a block 73, 73 and 24.)
// A voxel's sum holds the distances above the lower clamp (less than 2^12
// each) in its low 22 bits and their count above: good for the 1,023 returns
// of a pass.
// LIST: also list every voxel that received a contribution (incremental
// mode); a separate instance, so the plain fold keeps its register budget.
constexpr int kFoldPass = 1023;

// behind the return within the cos > 0.95 cone: 400 (a.b)^2 > 361 |a|^2 |b|^2,
// the return at P, the voxel centre at P + a, b = P - Q.  Decided in double
// when the sides differ by more than 2^-40 relative (each side is within
// 2^-50 of its exact value: |a.b| < 2^53 converts exactly, |b|^2 rounds once,
// three roundings per product), otherwise in 128-bit integers.
__device__ inline bool behind_exact(int32_t a0, int32_t a1, int32_t a2, int32_t b0, int32_t b1,
                                          int32_t b2) {
  const int64_t ab = (int64_t)a0 * b0 + (int64_t)a1 * b1 + (int64_t)a2 * b2;
  if (ab <= 0) return false;
  const int64_t aa = (int64_t)a0 * a0 + (int64_t)a1 * a1 + (int64_t)a2 * a2;
  const int64_t bb = (int64_t)b0 * b0 + (int64_t)b1 * b1 + (int64_t)b2 * b2;
  const double x = 400.0 * (double)ab * (double)ab;
  const double y = 361.0 * (double)aa * (double)bb;
  if (x > y * (1.0 + 0x1p-40)) return true;
  if (x < y * (1.0 - 0x1p-40)) return false;
  return (__int128)400 * ab * ab > (__int128)361 * aa * bb;
}

__device__ inline int32_t lane_i(int32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline float lane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ inline int mul_hi24(int a, uint32_t b) {   // (a * b) >> 32, both below 2^24
  int d;
  asm("v_mul_hi_u32_u24 %0, %1, %2" : "=v"(d) : "v"(a), "s"(b));
  return d;
}
__device__ inline int mad_i24(int a, int b, int c) {
  int d;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "s"(b), "v"(c));
  return d;
}
__device__ inline int clamp0(int v, int hi) {   // to [0, hi]
  int d;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(d) : "v"(v), "s"(hi));
  return d;
}

template <int LIST>
__global__ void __launch_bounds__(kFoldThreads) __attribute__((amdgpu_waves_per_eu(8)))
k_integrate_fold(const FrameArgs *fa, Params p, MapDev m, FrameScratch fs, FrameCounters *c,
                 GridDev g) {
  const int3 Q = fa->Q;
  __shared__ uint32_t s_sum[kBlockVox];
  __shared__ int32_t s_dist[kBlockVox];      // isqrt |voxel centre - Q|
  __shared__ int s_list[kBlockVox / 64 + 1]; // LIST: per-slice offsets, then the block's base
  __shared__ uint32_t s_occ4;
  __shared__ unsigned long long s_stat[3];
  if (threadIdx.x < 3) s_stat[threadIdx.x] = 0ull;
  const int nt = c->n_touched;
  const int t = threadIdx.x, lane0 = lane_id();
  const int wave0 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lo_clamp = p.clamp_neg ? -(int)p.tau_u : 0, range = (int)p.tau_u - lo_clamp;
  unsigned long long excluded = 0;   // of the wave
  unsigned long long pairs = 0;      // of the lane's returns
  unsigned folded = 0;
  for (int i = blockIdx.x; i < nt; i += gridDim.x) {
    const int64_t id = fs.touched[i];
    // the block's own words first: their latency overlaps the gather below
    const int64_t v = id * kBlockVox + t;
    int32_t S[kFoldVox], W[kFoldVox];
    uint32_t clrw[kFoldVox];
    for (int h = 0; h < kFoldVox; ++h) {
      S[h] = m.S[v + kFoldThreads * h];
      W[h] = m.W[v + kFoldThreads * h];
      clrw[h] = m.clr[id * 16 + ((t + kFoldThreads * h) >> 5)];
    }
    const uint32_t surfw = (t >= 32 && t < 48) ? m.surf[id * 16 + (t - 32)] : 0u;
    const int64_t bkey = m.bkey[id];
    const int2 bin = fs.bin[i];
    int32_t b[3];
    unpack_key(bkey, b[0], b[1], b[2]);
    if (t == 0) {
      bool in = true;
      for (int a = 0; a < 3; ++a)
        in = in && b[a] - g.g0[a] >= g.margin && b[a] - g.g0[a] < g.gd[a] - g.margin;
      if (!in) atomicOr(&c->status, kStatusOutsideGrid);
      m.tpos[id] = 0;   // the next frame counts from 0
      s_occ4 = 0u;
    }
    int64_t dS[kFoldVox] = {};
    int dW[kFoldVox] = {};
    for (int h = 0; h < kFoldVox && bin.y > 0; ++h) {
      const int u = t + kFoldThreads * h;
      const int64_t cq0 = 256 * (int64_t)(8 * b[0] + (u & 7)) + 128 - Q.x;  // voxel centre - sensor
      const int64_t cq1 = 256 * (int64_t)(8 * b[1] + ((u >> 3) & 7)) + 128 - Q.y;
      const int64_t cq2 = 256 * (int64_t)(8 * b[2] + (u >> 6)) + 128 - Q.z;
      s_dist[u] = (int32_t)isqrt64(cq0 * cq0 + cq1 * cq1 + cq2 * cq2);
      s_sum[u] = 0u;
    }
    __syncthreads();
    for (int pass = 0; pass < bin.y; pass += kFoldPass) {
      const int count = bin.y - pass < kFoldPass ? bin.y - pass : kFoldPass;
      const int32_t *list = fs.bin_list + bin.x + pass;
      for (int e0 = wave0; e0 < count; e0 += 64 * kFoldWaves) {
        const int e = e0 + kFoldWaves * lane0;
        const int4 P = fs.P[list[e < count ? e : e0]];
        // the box, from its corner; the return's place from the centre of the
        // block's first voxel, 1/256 voxels
        int lo[3], len[3];
        const int pv[3] = {P.x, P.y, P.z};
        float at[3];
        for (int a = 0; a < 3; ++a) {
          const int q = (pv[a] >> 8) - 8 * b[a];
          lo[a] = q - p.R > 0 ? q - p.R : 0;
          len[a] = (q + p.R < 7 ? q + p.R : 7) - lo[a] + 1;
          at[a] = (float)(2048 * b[a] + 256 * lo[a] + 128 - pv[a]);
        }
        const int nxy = len[0] * len[1], vol = nxy * len[2];
        const int box = len[0] | (nxy << 4) | (vol << 11) | ((lo[0] | (lo[1] << 3) | (lo[2] << 6)) << 21);
        // idx / n as (idx * i) >> 18, right for idx < 512 where i is at least
        // 2^18 / n and less than 2^9 / n above it (n <= 64; the float is within
        // 1/16 of 2^18 / n)
        const uint32_t iy = (uint32_t)(262144.0f * __builtin_amdgcn_rcpf((float)len[0])) + 1u,
                       iz = (uint32_t)(262144.0f * __builtin_amdgcn_rcpf((float)nxy)) + 1u;
        const int32_t b0 = P.x - Q.x, b1 = P.y - Q.y, b2 = P.z - Q.z;
        const float g0 = (float)b0, g1 = (float)b1, g2 = (float)b2;
        const float inv = __builtin_amdgcn_rsqf(__builtin_fmaf(g0, g0, __builtin_fmaf(g1, g1, g2 * g2)));
        const float u0 = g0 * inv, u1 = g1 * inv, u2 = g2 * inv;
        pairs += e < count ? (unsigned)vol : 0u;
        const int here = (count - e0 + kFoldWaves - 1) / kFoldWaves;
        for (int j = 0; j < (here < 64 ? here : 64); ++j) {
          const uint32_t d = (uint32_t)lane_i(box, j);
          const uint32_t jy = (uint32_t)lane_i((int)iy, j), jz = (uint32_t)lane_i((int)iz, j);
          const int w = lane_i(P.w, j) - lo_clamp;
          const float f0 = lane_f(at[0], j), f1 = lane_f(at[1], j), f2 = lane_f(at[2], j);
          const float v0 = lane_f(u0, j), v1 = lane_f(u1, j), v2 = lane_f(u2, j);
          const int nx = (int)(d & 15u), nsl = (int)((d >> 4) & 127u), size = (int)((d >> 11) & 1023u);
          int idx = lane0, from = lane0 + (int)(d >> 21), idx14 = lane0 << 14;
          for (int done = 0; done < size; done += 64, idx += 64, from += 64, idx14 += 64 << 14) {
            // idx = x + nx y + nx ny z, kept times 2^14 so that a quotient is
            // the upper word of a 24-bit product
            const int z = mul_hi24(idx14, jz), rem14 = mad_i24(z, -(nsl << 14), idx14);
            const int y = mul_hi24(rem14, jy), x14 = mad_i24(y, -(nx << 14), rem14);
            // x + 8 y + 64 z from the box's corner (past the box's end the read wraps)
            const int cell = mad_i24(z, 64 - nsl, mad_i24(y, 8 - nx, from)) & 511;
            int dist = w - s_dist[cell];
            const float a0 = __builtin_fmaf(0x1p-6f, (float)x14, f0), a1 = __builtin_fmaf(256.0f, (float)y, f1),
                        a2 = __builtin_fmaf(256.0f, (float)z, f2);
            const float ab = __builtin_fmaf(a0, v0, __builtin_fmaf(a1, v1, a2 * v2));
            const float aa = __builtin_fmaf(a0, a0, __builtin_fmaf(a1, a1, a2 * a2));
            // (with the sign of a.b)
            const float q = __builtin_fmaf(ab, __builtin_fabsf(ab), -0.9025f * aa);
            const uint64_t act = __builtin_amdgcn_ballot_w64(idx < size);
            uint64_t behind = act & __builtin_amdgcn_ballot_w64(q > 0.0f);
            const uint64_t close =
                act & __builtin_amdgcn_ballot_w64(__builtin_fabsf(q) <= 0x1p-16f * aa);
            if (close != 0ull) {
              const int32_t c0 = lane_i(b0, j), c1 = lane_i(b1, j), c2 = lane_i(b2, j);
              const bool exact = behind_exact((int32_t)a0, (int32_t)a1, (int32_t)a2, c0, c1, c2);
              behind = (behind & ~close) | (close & __builtin_amdgcn_ballot_w64(exact));
            }
            excluded += (unsigned)__popcll(behind);
            dist = clamp0(dist, range);
            if (__builtin_amdgcn_inverse_ballot_w64(act & ~behind))
              atomicAdd(&s_sum[cell], (1u << 22) + (uint32_t)dist);
          }
        }
      }
      __syncthreads();
      for (int h = 0; h < kFoldVox; ++h) {
        const uint32_t sum = s_sum[t + kFoldThreads * h];
        s_sum[t + kFoldThreads * h] = 0u;
        const int n = (int)(sum >> 22);
        dS[h] += (int64_t)(sum & 0x3FFFFFu) + (int64_t)lo_clamp * n;
        dW[h] += n;
      }
      __syncthreads();
    }
    for (int h = 0; h < kFoldVox; ++h) {
      if (dW[h] <= 0) continue;
      int64_t S2 = (int64_t)S[h] + dS[h], W2 = (int64_t)W[h] + dW[h];
      if (W2 > p.cap) {
        S2 = div_floor(S2 * p.cap, W2);
        W2 = p.cap;
      }
      S[h] = (int32_t)S2;
      W[h] = (int32_t)W2;
      m.S[v + kFoldThreads * h] = S[h];
      m.W[v + kFoldThreads * h] = (uint16_t)W[h];
      ++folded;
    }
    if (LIST) {   // list each voxel that received a contribution (one atomic per block)
      for (int h = 0; h < kFoldVox; ++h) {
        const unsigned long long bal = __ballot(dW[h] > 0);
        if (lane0 == 0) s_list[wave0 + kFoldWaves * h] = __popcll(bal);
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        int tot = 0;
        for (int k = 0; k < kBlockVox / 64; ++k) {
          const int n = s_list[k];
          s_list[k] = tot;
          tot += n;
        }
        s_list[kBlockVox / 64] = tot ? atomicAdd(&c->n_changed, tot) : 0;
      }
      __syncthreads();
      for (int h = 0; h < kFoldVox; ++h) {
        const unsigned long long bal = __ballot(dW[h] > 0);
        if (dW[h] > 0)
          fs.changed[s_list[kBlockVox / 64] + s_list[wave0 + kFoldWaves * h] +
                     __popcll(bal & ((1ull << lane0) - 1ull))] = (int32_t)(v + kFoldThreads * h);
      }
    }
    write_brick(p, g, S, W, &s_occ4, clrw, surfw, bkey);
  }
  unsigned long long sa = pairs, sf = folded;
  const unsigned long long se = excluded;
  for (int off = 32; off >= 1; off >>= 1) {
    sa += __shfl_xor(sa, off);
    sf += __shfl_xor((unsigned)sf, off);
  }
  sa -= se;   // applied
  __syncthreads();
  if (lane_id() == 0) {
    if (sa) atomicAdd(&s_stat[0], sa);
    if (se) atomicAdd(&s_stat[1], se);
    if (sf) atomicAdd(&s_stat[2], sf);
  }
  __syncthreads();
  if (threadIdx.x < 3 && s_stat[threadIdx.x])
    atomicAdd(&c->fold[blockIdx.x % kStatSlots][threadIdx.x], s_stat[threadIdx.x]);
}

__global__ void __launch_bounds__(kFoldThreads)
k_grid_rebuild(Params p, MapDev m, GridDev g, int64_t n_blocks) {
  __shared__ uint32_t s_occ4;
  for (int64_t id = blockIdx.x; id < n_blocks; id += gridDim.x) {
    const int64_t bkey = m.bkey[id];
    if (bkey == kEmpty) continue;   // an evicted block's free id
    const int t = threadIdx.x;
    int32_t S[kFoldVox], W[kFoldVox];
    uint32_t clrw[kFoldVox];
    for (int h = 0; h < kFoldVox; ++h) {
      const int u = t + kFoldThreads * h;
      S[h] = m.S[id * kBlockVox + u];
      W[h] = m.W[id * kBlockVox + u];
      clrw[h] = m.clr[id * 16 + (u >> 5)];
    }
    if (t == 0) s_occ4 = 0u;
    __syncthreads();
    write_brick(p, g, S, W, &s_occ4, clrw, (t >= 32 && t < 48) ? m.surf[id * 16 + (t - 32)] : 0u, bkey);
  }
}

__global__ void k_grid_fill(GridDev g, int64_t nbricks) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = i; j < nbricks * 32; j += stride) g.pred[j] = kUnknownWord;
  for (int64_t j = i; j < nbricks * 16; j += stride) g.surf[j] = 0u;
  for (int64_t j = i; j < (nbricks + 31) / 32; j += stride) g.occ_any[j] = 0u;
  for (int64_t j = i; j < nbricks; j += stride) g.occ4[j] = 0u;
  for (int64_t j = i; j < nbricks * 16; j += stride) g.occ1[j] = 0u;
}

__global__ void k_stick_status(FrameCounters *c, const int32_t *n_blocks,
                               const int32_t *n_points) {
  c->sticky |= c->status;
  if (c->n_new_blocks > 0)
    for (int a = 0; a < 3; ++a) {
      c->sbmin[a] = c->bmin[a] < c->sbmin[a] ? c->bmin[a] : c->sbmin[a];
      c->sbmax[a] = c->bmax[a] > c->sbmax[a] ? c->bmax[a] : c->sbmax[a];
    }
  c->snap_blocks = *n_blocks;
  c->snap_points = *n_points;
}

__global__ void k_zero_words(uint32_t *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

__global__ void k_set_frame_args(FrameArgs *fa, int64_t n, int3 Q, int32_t frame, int3 wlo,
                                 int3 whi, FrameCounters *clear) {
  fa->n = n;
  fa->Q = Q;
  fa->frame = frame;
  fa->wlo = wlo;
  fa->whi = whi;
  if (clear) {
    clear->sticky = 0;
    for (int a = 0; a < 3; ++a) {
      clear->sbmin[a] = 0x7fffffff;
      clear->sbmax[a] = -0x7fffffff - 1;
    }
  }
}

// ------------------------------------------------------- sliding window
// One workgroup per block id: a live block outside [lo, hi] is cleared (its
// voxels read unknown again), its key removed and its id pushed on the free
// list.
__global__ void __launch_bounds__(kThreads)
k_window_evict(MapDev m, int64_t n_blocks, int3 lo, int3 hi) {
  for (int64_t id = blockIdx.x; id < n_blocks; id += gridDim.x) {
    const int64_t key = m.bkey[id];
    if (key == kEmpty) continue;
    int32_t b[3];
    unpack_key(key, b[0], b[1], b[2]);
    if (in_box(b[0], b[1], b[2], lo, hi)) continue;
    for (int t = threadIdx.x; t < kBlockVox; t += kThreads) {
      m.S[id * kBlockVox + t] = 0;
      m.W[id * kBlockVox + t] = 0;
    }
    if (threadIdx.x < 16) {
      m.clr[id * 16 + threadIdx.x] = 0;
      m.surf[id * 16 + threadIdx.x] = 0;
    }
    __syncthreads();   // every thread has read bkey[id] before it changes
    if (threadIdx.x == 0) {
      m.bkey[id] = kEmpty;
      m.touched[id] = -1;
      m.free_ids[atomicAdd(m.n_free, 1)] = (int32_t)id;
    }
  }
}

__global__ void k_hash_clear(HashTable h) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= (int64_t)h.mask;
       i += (int64_t)gridDim.x * blockDim.x) {
    h.keys[i] = kEmpty;
    h.vals[i] = -1;
  }
}

// Live blocks back into the cleared hash.
__global__ void __launch_bounds__(kThreads) k_window_rehash(MapDev m, int64_t n_blocks) {
  const int64_t id = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (id >= n_blocks) return;
  const int64_t key = m.bkey[id];
  if (key == kEmpty) return;
  bool fresh;
  const int32_t s = hash_insert(m.h, key, fresh);
  if (s >= 0) m.h.vals[s] = (int32_t)id;   // the hash holds 2 max_blocks slots: never full
}

__device__ inline void point_block(const PointsDev &pts, int64_t i, int32_t v[3]) {
  unpack_key(pts.key[i], v[0], v[1], v[2]);
}

// Points outside [lo, hi] lose their voxel address (their block is gone).
__global__ void __launch_bounds__(kThreads)
k_window_points(PointsDev pts, int64_t n_points, int3 lo, int3 hi) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n_points) return;
  int32_t v[3];
  point_block(pts, i, v);
  if (!in_box(v[0] >> 3, v[1] >> 3, v[2] >> 3, lo, hi)) pts.addr[i] = -1;
}

// Points inside [lo, hi] without a block: their block joins the frame's new
// blocks (assigned and cleared with them).
__global__ void __launch_bounds__(kThreads)
k_window_thaw(MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c, int64_t n_points,
              int3 lo, int3 hi) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n_points || pts.addr[i] >= 0) return;
  int32_t v[3];
  point_block(pts, i, v);
  if (!in_box(v[0] >> 3, v[1] >> 3, v[2] >> 3, lo, hi)) return;
  bool fresh;
  const int32_t s = hash_insert(m.h, pack_key(v[0] >> 3, v[1] >> 3, v[2] >> 3), fresh);
  if (s < 0) atomicOr(&c->status, kStatusHashFull);
  if (fresh) fs.new_blocks[atomicAdd(&c->n_new_blocks, 1)] = s;
}

// After assignment: those points get their voxel address and surface bit.
__global__ void __launch_bounds__(kThreads)
k_window_link(MapDev m, PointsDev pts, int64_t n_points, int3 lo, int3 hi) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n_points || pts.addr[i] >= 0) return;
  int32_t v[3];
  point_block(pts, i, v);
  if (!in_box(v[0] >> 3, v[1] >> 3, v[2] >> 3, lo, hi)) return;
  const int32_t bs = hash_find(m.h, pack_key(v[0] >> 3, v[1] >> 3, v[2] >> 3));
  const int32_t bid = bs >= 0 ? m.h.vals[bs] : -1;
  if (bid < 0) return;   // block capacity exhausted (the frame reports it)
  const int vi = (v[0] & 7) | ((v[1] & 7) << 3) | ((v[2] & 7) << 6);
  pts.addr[i] = bid * kBlockVox + vi;
  atomicOr(&m.surf[(int64_t)bid * 16 + (vi >> 5)], 1u << (vi & 31));
}

// Points inside [lo, hi] listed: the waves' counts are combined in LDS, so
// a workgroup of 1024 points takes one atomic on the list's counter (one per
// wave serialised some 30,000 atomics on that address per call).  A negative
// n_points reads the count on the device (a recorded frame).
constexpr int kListThreads = 1024;
__global__ void __launch_bounds__(kListThreads)
k_window_list(PointsDev pts, int64_t n_points, int3 lo, int3 hi, int32_t *sel, int32_t *n_sel) {
  __shared__ int part[kListThreads / 64 + 1];
  const int64_t i = (int64_t)blockIdx.x * kListThreads + threadIdx.x;
  const int64_t n = n_points < 0 ? (int64_t)*pts.n_points : n_points;
  bool take = false;
  if (i < n) {
    int32_t v[3];
    point_block(pts, i, v);
    take = in_box(v[0] >> 3, v[1] >> 3, v[2] >> 3, lo, hi);
  }
  const unsigned long long bal = __ballot(take);
  const int lane = lane_id(), wave = (int)(threadIdx.x >> 6);
  if (lane == 0) part[wave] = __popcll(bal);
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int k = 0; k < kListThreads / 64; ++k) {
      const int c = part[k];
      part[k] = tot;
      tot += c;
    }
    part[kListThreads / 64] = tot ? atomicAdd(n_sel, tot) : 0;
  }
  __syncthreads();
  if (take)
    sel[part[kListThreads / 64] + part[wave] + __popcll(bal & ((1ull << lane) - 1ull))] =
        (int32_t)i;
}

__global__ void k_label_fill(uint8_t *label, int16_t *ff, int64_t from, int64_t to) {
  for (int64_t i = from + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < to;
       i += (int64_t)gridDim.x * blockDim.x) {
    label[i] = 255;
    ff[i] = -1;
  }
}

inline unsigned grid_for(int64_t threads) {
  int64_t b = (threads + kThreads - 1) / kThreads;
  return (unsigned)(b > 0 ? b : 1);
}
inline unsigned part_grid(int64_t returns) { return (unsigned)((returns + 63) / 64); }

}  // namespace

void launch_zero_words(void *p, int64_t bytes, hipStream_t s) {
  const int64_t n = bytes / 4;
  hipLaunchKernelGGL(k_zero_words, dim3((unsigned)std::min<int64_t>(1024, (n + 255) / 256)),
                     dim3(256), 0, s, (uint32_t *)p, n);
}

void launch_stick_status(FrameCounters *c, const int32_t *n_blocks, const int32_t *n_points,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_stick_status, dim3(1), dim3(1), 0, s, c, n_blocks, n_points);
}

void launch_set_frame_args(FrameArgs *fa, int64_t n, int3 Q, int32_t frame, int3 wlo, int3 whi,
                           hipStream_t s, FrameCounters *clear) {
  hipLaunchKernelGGL(k_set_frame_args, dim3(1), dim3(1), 0, s, fa, n, Q, frame, wlo, whi, clear);
}

void launch_window_evict(MapDev m, PointsDev pts, int64_t n_blocks, int64_t n_points, int3 lo,
                         int3 hi, hipStream_t s) {
  if (n_blocks > 0)
    hipLaunchKernelGGL(k_window_evict, dim3((unsigned)std::min<int64_t>(n_blocks, 8192)),
                       dim3(kThreads), 0, s, m, n_blocks, lo, hi);
  const int64_t slots = (int64_t)m.h.mask + 1;
  hipLaunchKernelGGL(k_hash_clear, dim3((unsigned)std::min<int64_t>(4096, (slots + 255) / 256)),
                     dim3(256), 0, s, m.h);
  if (n_blocks > 0)
    hipLaunchKernelGGL(k_window_rehash, dim3(grid_for(n_blocks)), dim3(kThreads), 0, s, m,
                       n_blocks);
  if (n_points > 0)
    hipLaunchKernelGGL(k_window_points, dim3(grid_for(n_points)), dim3(kThreads), 0, s, pts,
                       n_points, lo, hi);
}

void launch_window_thaw(MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c,
                        int64_t n_points, int3 lo, int3 hi, hipStream_t s) {
  if (n_points > 0)
    hipLaunchKernelGGL(k_window_thaw, dim3(grid_for(n_points)), dim3(kThreads), 0, s, m, pts, fs,
                       c, n_points, lo, hi);
}

void launch_window_link(MapDev m, PointsDev pts, int64_t n_points, int3 lo, int3 hi,
                        hipStream_t s) {
  if (n_points > 0)
    hipLaunchKernelGGL(k_window_link, dim3(grid_for(n_points)), dim3(kThreads), 0, s, m, pts,
                       n_points, lo, hi);
}

void launch_window_list(PointsDev pts, int64_t n_points, int3 lo, int3 hi, int32_t *sel,
                        int32_t *n_sel, hipStream_t s, bool dev_n) {
  launch_zero_words(n_sel, sizeof(int32_t), s);
  if (n_points > 0)
    hipLaunchKernelGGL(k_window_list, dim3((unsigned)((n_points + kListThreads - 1) / kListThreads)),
                       dim3(kListThreads), 0, s, pts, dev_n ? (int64_t)-1 : n_points, lo, hi, sel,
                       n_sel);
}

void launch_label_fill(uint8_t *label, int16_t *first_free, int64_t from, int64_t to,
                       hipStream_t s) {
  if (to > from)
    hipLaunchKernelGGL(k_label_fill,
                       dim3((unsigned)std::min<int64_t>(1024, (to - from + 255) / 256)),
                       dim3(256), 0, s, label, first_free, from, to);
}

void launch_frame_prep(const float *xyz, FrameArgs *fa, const FrameArgs &fa_new, int64_t nb,
                       const Params &p, MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_reset_counters, dim3(1), dim3(128), 0, s, c, m, pts, fa, fa_new);
  if (nb > 0)
    hipLaunchKernelGGL(k_frame_prep, dim3(part_grid(nb)), dim3(kPartThreads), 0, s, xyz, fa, p, m,
                       pts, fs, c);
}

void launch_assign_blocks(MapDev m, FrameScratch fs, FrameCounters *c, const FrameArgs *fa, int3 glo,
                          int3 ghi, hipStream_t s) {
  hipLaunchKernelGGL(k_assign_blocks, dim3(4096), dim3(kThreads), 0, s, m, fs, c, fa, glo, ghi);
}

void launch_bins(const FrameArgs *fa, int64_t nb, const Params &p, MapDev m, PointsDev pts,
                 FrameScratch fs, FrameCounters *c, int64_t max_touched, hipStream_t s) {
  hipLaunchKernelGGL(k_bin_place, dim3((unsigned)std::min<int64_t>(256, grid_for(max_touched))),
                     dim3(kThreads), 0, s, m, pts, fs, c);
  if (nb > 0)
    hipLaunchKernelGGL(k_bin_fill, dim3(part_grid(nb)), dim3(kPartThreads), 0, s, fa, p, m, pts, fs, c);
}

void launch_frame_stop(MapDev m, PointsDev pts, FrameScratch fs, FrameCounters *c, hipStream_t s) {
  hipLaunchKernelGGL(k_frame_stop, dim3(256), dim3(kThreads), 0, s, m, pts, fs, c);
}

void launch_fold(const FrameArgs *fa, const Params &p, MapDev m, FrameScratch fs, FrameCounters *c,
                 GridDev g, int64_t max_touched, hipStream_t s) {
  int64_t wg = max_touched < 8192 ? max_touched : 8192;
  if (wg > 0) {
    if (fs.changed)
      hipLaunchKernelGGL(k_integrate_fold<1>, dim3((unsigned)wg), dim3(kFoldThreads), 0, s, fa, p,
                         m, fs, c, g);
    else
      hipLaunchKernelGGL(k_integrate_fold<0>, dim3((unsigned)wg), dim3(kFoldThreads), 0, s, fa, p,
                         m, fs, c, g);
  }
}

void launch_touch_band(const FrameArgs *fa, int64_t nb, const Params &p, MapDev m,
                       FrameScratch fs, FrameCounters *c, hipStream_t s) {
  if (nb > 0)
    hipLaunchKernelGGL(k_touch_band, dim3(part_grid(nb)), dim3(kPartThreads), 0, s, fa, p, m, fs,
                       c);
}

void launch_points_append(int64_t n_new, MapDev m, PointsDev pts, FrameScratch fs,
                          FrameCounters *c, const FrameArgs *fa, hipStream_t s) {
  if (n_new > 0) {
    hipLaunchKernelGGL(k_sort_new_tiles, dim3(grid_for(n_new)), dim3(kThreads), 0, s, fs, c);
    hipLaunchKernelGGL(k_points_append, dim3((unsigned)((n_new + 63) / 64)), dim3(64 * kAppendWaves),
                       0, s, m, pts, fs, c, fa);
  }
}

void launch_grid_fill(GridDev g, hipStream_t s) {
  int64_t nb = (int64_t)g.gd[0] * g.gd[1] * g.gd[2];
  int64_t blocks = (nb * 32 + kThreads - 1) / kThreads;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_grid_fill, dim3((unsigned)blocks), dim3(kThreads), 0, s, g, nb);
}

void launch_grid_rebuild(const Params &p, MapDev m, GridDev g, int64_t n_blocks,
                         hipStream_t s) {
  int64_t wg = n_blocks < 8192 ? n_blocks : 8192;
  if (wg > 0)
    hipLaunchKernelGGL(k_grid_rebuild, dim3((unsigned)wg), dim3(kFoldThreads), 0, s, p, m, g,
                       n_blocks);
}

}  // namespace af
