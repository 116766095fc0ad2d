// Smoothed clearance score and its adjoint.
//
// A differentiable companion of the collision-count score of Section 3.5:
// each sample o of the tool solid (local frame, approach axis +x, tip at the
// origin) placed at p + R(q) o contributes log sigma((T - c) / tau_s), where
// T is the TSDF (Section 3.2) interpolated trilinearly between voxel centres
// and a voxel without weight reads the truncation distance.  Gradients with
// respect to the quaternion q (through q / |q|) and the point p come from the
// same pass: d log sigma(z) / dz = sigma(-z).
//
// Layout: one tool sample per lane, so the 64 lanes read neighbouring voxels
// along the tool and the sums are a wave reduction.  What depends on the pair
// (point, orientation) alone, its rotation in double and the update of its
// quaternion, is more work than a sample when all 64 lanes repeat it, so a
// wave takes four pairs, pair lane & 3 in a lane, for that part, goes through
// them one by one for the samples and reduces their sums together.
// The TSDF is first expanded into "apron" bricks of 9^3 floats: brick b holds
// voxels 8b .. 8b + 8 on each axis, i.e. its own 8^3 voxels plus the first
// layer of its +x/+y/+z neighbours, so the 2^3 voxels of any interpolation
// cell whose lowest corner lies in b are all in b's apron brick.  Apron bricks
// exist for every mapped brick and every brick with a mapped +1 neighbour (the
// "halo"); a brick-to-apron table over the dense brick grid finds them, so a
// sample costs one table load and eight value loads, with no hashing.  Apron 0
// holds the truncation distance throughout: the table's 0 outside the aprons,
// and what a read outside the table gives.
//
// Precision: the placement of a sample in its voxel cell (p + R o, divided by
// v) is computed in double precision, because an fp32 position is only good
// to ~1e-5 voxel at metre scale and the gradient's relative error follows the
// cell fractions; interpolation, score and adjoint are fp32.  The quaternion
// derivative comes from the torque: a small rotation dtheta applied after R
// moves sample u = R o by dtheta x u, so s changes by dtheta . sum(u x g) with
// g the weighted TSDF gradient; with dq = (0, dtheta) q / 2 this gives
// ds/dq = 2 (-tau.v, w tau + tau x v) / |q| for q / |q| = (w, v) and
// tau = sum(u x g) -- three sums per pair instead of four, no projection.
// This file lets the compiler fuse multiply-adds (unlike the table builder,
// nothing here needs to round like the oracle).

#include "af_internal.h"

#pragma clang fp contract(fast)

namespace af {
namespace {

constexpr int kSmoothThreads = 256;

// An empty field: no aprons but apron 0, the truncation distance.
__global__ void __launch_bounds__(kSmoothThreads)
k_field_clear(int32_t *bid9, int64_t n, int32_t *count, float tau, float *T9) {
  const int64_t i0 = (int64_t)blockIdx.x * kSmoothThreads + threadIdx.x;
  for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * kSmoothThreads) bid9[i] = 0;
  if (blockIdx.x != 0) return;
  for (int v = threadIdx.x; v < 729; v += kSmoothThreads) T9[v] = tau;
  if (threadIdx.x == 0) *count = 1;
}

// Number every brick whose cell may reach a mapped brick (the mapped brick
// itself and its -1 neighbours along any set of axes), in any order, and
// record each apron's brick; a thread per block and neighbour.  (cap is at
// least the number of those bricks, 8 per mapped block at most; an index past
// it would be left unmapped rather than read out of bounds.)
__global__ void __launch_bounds__(kSmoothThreads)
k_apron_mark(MapDev m, int64_t n_blocks, GridDev g, int32_t *bid9, int32_t *count,
             int32_t *brick_of, int64_t cap) {
  const int64_t i = (int64_t)blockIdx.x * kSmoothThreads + threadIdx.x;
  if (i >= 8 * n_blocks) return;
  const int k = (int)(i & 7);
  int32_t b[3];
  unpack_key(m.bkey[i >> 3], b[0], b[1], b[2]);
  const int x = b[0] - g.g0[0] - (k & 1), y = b[1] - g.g0[1] - ((k >> 1) & 1),
            z = b[2] - g.g0[2] - (k >> 2);
  if ((unsigned)x >= (unsigned)g.gd[0] || (unsigned)y >= (unsigned)g.gd[1] ||
      (unsigned)z >= (unsigned)g.gd[2])
    return;
  const int64_t brick = ((int64_t)z * g.gd[1] + y) * g.gd[0] + x;
  if (atomicCAS(&bid9[brick], 0, -1) != 0) return;   // another thread's
  const int32_t e = atomicAdd(count, 1);
  if (e <= cap) brick_of[e - 1] = (int32_t)brick;
  bid9[brick] = e <= cap ? e : 0;
}

// Fill the aprons, a workgroup each, straight from the map's sums: what bounds
// it is the map's reading and the aprons' writing.  (29,000 aprons: 142 us from
// an expanded copy of the map that took another 18, with a thread per voxel of
// 8 aprons per block; 55 us now.)  Voxel (lx, ly, lz) in [0, 9)^3 of the
// apron's brick, from the eight blocks it reaches.
__global__ void __launch_bounds__(kSmoothThreads)
k_apron_fill(MapDev m, const int32_t *count, const int32_t *brick_of, GridDev g, double scale,
             float tau, int64_t cap, float *T9) {
  __shared__ int32_t s_id[2][8];
  const int t = threadIdx.x;
  const int64_t last = *count - 1 < cap ? *count - 1 : cap;
  int turn = 0;
  for (int64_t e = 1 + blockIdx.x; e <= last; e += gridDim.x, turn ^= 1) {
    if (t < 8) {
      const int32_t br = brick_of[e - 1];
      const int x = br % g.gd[0] + (t & 1), y = br / g.gd[0] % g.gd[1] + ((t >> 1) & 1),
                z = br / (g.gd[0] * g.gd[1]) + (t >> 2);
      const int32_t slot = hash_find(m.h, pack_key(x + g.g0[0], y + g.g0[1], z + g.g0[2]));
      s_id[turn][t] = slot >= 0 ? m.h.vals[slot] : -1;
    }
    __syncthreads();   // (the other half is free again: its readers are past it)
    for (int v = t; v < 729; v += kSmoothThreads) {
      const int lx = v % 9, ly = (v / 9) % 9, lz = v / 81;
      const int32_t id = s_id[turn][(lx >> 3) | ((ly >> 3) << 1) | ((lz >> 3) << 2)];
      float value = tau;
      if (id >= 0) {
        const int64_t at = (int64_t)id * kBlockVox + ((lx & 7) | ((ly & 7) << 3) | ((lz & 7) << 6));
        const int32_t W = m.W[at];
        if (W > 0) value = (float)(((double)m.S[at] / (double)W) / scale);
      }
      T9[e * 729 + v] = value;
    }
  }
}

// x + the value DPP control `ctrl` routes to this lane.
template <int ctrl>
__device__ inline float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, false);
  return x + __int_as_float(y);
}

// The sums over the wave of v[0..3], v[lane & 3]'s in each lane: swaps within
// quads, each followed by keeping the half that the lane is for, rotations
// within rows by whole quads, and swaps of rows.  (39 instructions for three
// times four sums; each by itself takes 24.)
__device__ inline float wave_sums(const float v[4]) {
  const int lane = threadIdx.x & 63;
  // (every lane adds before it chooses: a swap reads its neighbour's value)
  const float a0 = dpp_add<0xb1>(v[0]), a1 = dpp_add<0xb1>(v[1]);   // quad_perm [1, 0, 3, 2]
  const float a2 = dpp_add<0xb1>(v[2]), a3 = dpp_add<0xb1>(v[3]);
  float x = (lane & 1) ? a1 : a0, y = (lane & 1) ? a3 : a2;
  x = dpp_add<0x4e>(x);    // quad_perm [2, 3, 0, 1]
  y = dpp_add<0x4e>(y);
  x = (lane & 2) ? y : x;
  x = dpp_add<0x124>(x);   // row_ror:4
  x = dpp_add<0x128>(x);   // row_ror:8
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// The field as the samples read it.
struct FieldView {
  __amdgpu_buffer_rsrc_t bid9;
  const float *T9;
  int32_t g0[3], gd[3];
  float tau;
};

__device__ inline FieldView field_view(const SmoothField &f) {
  FieldView w;
  w.bid9 = __builtin_amdgcn_make_buffer_rsrc(
      (void *)f.bid9, (short)0, (int)(4u * (uint32_t)f.gd[0] * (uint32_t)f.gd[1] * (uint32_t)f.gd[2]),
      0x00020000);
  w.T9 = f.T9;
  w.tau = f.tau;
  for (int a = 0; a < 3; ++a) {
    w.g0[a] = f.g0[a];
    w.gd[a] = f.gd[a];
  }
  return w;
}

// The 2^3 voxel values of the cell whose lowest corner is voxel (X, Y, Z),
// t[a | b << 1 | c << 2] for corner (X + a, Y + b, Z + c).
__device__ inline void cell_values(const FieldView &f, int X, int Y, int Z, float t[8]) {
  const int bx = (X >> 3) - f.g0[0], by = (Y >> 3) - f.g0[1], bz = (Z >> 3) - f.g0[2];
  const bool in = ((unsigned)bx < (unsigned)f.gd[0]) & ((unsigned)by < (unsigned)f.gd[1]) &
                  ((unsigned)bz < (unsigned)f.gd[2]);
  // (a grid has less than 2^25 bricks and several per axis: 24-bit products)
  const uint32_t brick = __umul24(__umul24(bz, f.gd[1]) + by, f.gd[0]) + bx;
  const int32_t e =
      __builtin_amdgcn_raw_buffer_load_b32(f.bid9, in ? (int)(brick << 2) : -4, 0, 0);
  for (int k = 0; k < 8; ++k) t[k] = f.tau;
  if (e != 0) {
    const float *c = f.T9 + (int64_t)e * 729 + (int)(__umul24(Z & 7, 81) + __umul24(Y & 7, 9) + (X & 7));
#pragma unroll
    for (int k = 0; k < 8; ++k) t[k] = c[(k & 1) + ((k >> 1) & 1) * 9 + (k >> 2) * 81];
  }
}

// A pair's point as integer voxel coordinate + fraction of p / v - 1/2.
struct PairBase {
  int ip[3];
  double rp[3];
};

__device__ inline PairBase pair_base(const float *p, double v) {
  PairBase b;
  for (int a = 0; a < 3; ++a) {
    const double g = (double)p[a] / v - 0.5;
    const double fl = floor(g);
    b.ip[a] = (int)fl;
    b.rp[a] = g - fl;
  }
  return b;
}

// Normalised quaternion, its norm, and the rotation (row-major, double for
// the placement of samples).
struct Rot {
  float qn[4];
  float nq;
  double R[9];
};

__device__ inline Rot make_rot(const float q[4]) {
  Rot r;
  const double q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
  const double n = sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
  const double in = 1.0 / n;
  const double w = q0 * in, x = q1 * in, y = q2 * in, z = q3 * in;
  r.nq = (float)n;
  r.qn[0] = (float)w;
  r.qn[1] = (float)x;
  r.qn[2] = (float)y;
  r.qn[3] = (float)z;
  r.R[0] = 1.0 - 2.0 * (y * y + z * z);
  r.R[1] = 2.0 * (x * y - w * z);
  r.R[2] = 2.0 * (x * z + w * y);
  r.R[3] = 2.0 * (x * y + w * z);
  r.R[4] = 1.0 - 2.0 * (x * x + z * z);
  r.R[5] = 2.0 * (y * z - w * x);
  r.R[6] = 2.0 * (x * z - w * y);
  r.R[7] = 2.0 * (y * z + w * x);
  r.R[8] = 1.0 - 2.0 * (x * x + y * y);
  return r;
}

__device__ inline float log_sigmoid(float z) {
  return z >= 0.f ? -log1pf(expf(-z)) : z - log1pf(expf(z));
}

// sigma(-z) = 1 / (1 + e^z) with the hardware exponential and reciprocal
// (about 1 ulp each; e^z = inf gives 0).
__device__ inline float sigmoid_neg(float z) {
  return __builtin_amdgcn_rcpf(1.f + __expf(z));
}

// One pair as its samples read it, the same in every lane: the rotation
// divided by the voxel size, and the point.
struct PairView {
  double R[9], rp[3];
  int ip[3];
};

__device__ inline double lane_d(double v, int l) {
  const int64_t b = __double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((int64_t)hi << 32) | lo);
}

__device__ inline PairView pair_view(const PairBase &pb, const double Rv[9], int l) {
  PairView w;
  for (int a = 0; a < 9; ++a) w.R[a] = lane_d(Rv[a], l);
  for (int a = 0; a < 3; ++a) {
    w.rp[a] = lane_d(pb.rp[a], l);
    w.ip[a] = __builtin_amdgcn_readlane(pb.ip[a], l);
  }
  return w;
}

// No sample's cell: smooth_sample keeps x above it.  (A point or a sample beyond
// 2^31 voxels has a coordinate anywhere: the conversion to int stops at the
// ends, and their sum wraps.  With the values set instead, so that no cell
// would do, the refinement takes 2.2 ms, not 1.95.)
constexpr int kNoCell = -0x7fffffff - 1;

// A lane's cell of a pair and its values, kept while the samples stay in their
// cells: the refinement moves most by less than a voxel a step, and a wave's
// cells of one pair are 22 KB of lines, which would not last in the first-level
// cache until the next step.  (256,000 pairs of 64 samples, 20 steps: 3.34 ms
// with one pair a wave and a gather a step; 1.89 now, 2.9 where the steps are
// so large that most samples change their cells.  More waves a SIMD, for which
// registers spill: 2.3 at four, 3.6 at five.)
struct Cell {
  int x[3];
  float t[8];
};

// One sample: returns its log sigma term (not with G == 2); with G > 0 adds
// the torque u x dT/dx into tq and, with G == 1, dT/dx into dp, weighted with
// sigma(-z); distances in voxels.
template <int G>
__device__ inline float smooth_sample(const FieldView &f, const PairView &w, const float o[3],
                                      float c, float inv_ts, Cell &cell, float dp[3], float tq[3]) {
  int at[3];
  float fr[3], u[3];
  for (int a = 0; a < 3; ++a) {
    const double ud = w.R[3 * a] * (double)o[0] + w.R[3 * a + 1] * (double)o[1] +
                      w.R[3 * a + 2] * (double)o[2];
    const double gl = w.rp[a] + ud;
    const double fl = floor(gl);
    at[a] = w.ip[a] + (int)fl;
    fr[a] = (float)(gl - fl);
    u[a] = (float)ud;
  }
  at[0] = at[0] > kNoCell ? at[0] : kNoCell + 1;   // (both are outside every grid)
  if ((at[0] != cell.x[0]) | (at[1] != cell.x[1]) | (at[2] != cell.x[2])) {
    for (int a = 0; a < 3; ++a) cell.x[a] = at[a];
    cell_values(f, at[0], at[1], at[2], cell.t);
  }
  const float *t = cell.t;
  const float fx = fr[0], fy = fr[1], fz = fr[2];
  // trilinear interpolation as lerps along x, then y, then z
  const float e0 = t[1] - t[0], e1 = t[3] - t[2], e2 = t[5] - t[4], e3 = t[7] - t[6];
  const float a00 = t[0] + fx * e0, a10 = t[2] + fx * e1;
  const float a01 = t[4] + fx * e2, a11 = t[6] + fx * e3;
  const float y0 = a10 - a00, y1 = a11 - a01;
  const float b0 = a00 + fy * y0, b1 = a01 + fy * y1;
  const float z1 = b1 - b0;
  const float val = b0 + fz * z1;
  const float z = (val - c) * inv_ts;
  if (G > 0) {
    // derivatives of the interpolant in cell units
    const float dx0 = e0 + fy * (e1 - e0);
    const float dx1 = e2 + fy * (e3 - e2);
    const float gx = dx0 + fz * (dx1 - dx0);
    const float gy = y0 + fz * (y1 - y0);
    const float wgt = sigmoid_neg(z);
    const float g0 = wgt * gx, g1 = wgt * gy, g2 = wgt * z1;
    if (G == 1) {
      dp[0] += g0;
      dp[1] += g1;
      dp[2] += g2;
    }
    tq[0] += u[1] * g2 - u[2] * g1;
    tq[1] += u[2] * g0 - u[0] * g2;
    tq[2] += u[0] * g1 - u[1] * g0;
  }
  return G == 2 ? 0.f : log_sigmoid(z);
}

constexpr int kGroup = 4;   // pairs of a wave

// s and the gradients of up to kGroup pairs, pair lane & 3 in each lane (pb,
// r): the pairs one by one, a lane per sample, then their sums.  o0: the
// lane's sample of the first 64 (loaded once per kernel), cells: its cells.
// dp comes in 1 / metre, tq as ds/d(rotation).
template <int G>
__device__ inline float smooth_group(const FieldView &f, const PairBase &pb, const Rot &r, int count,
                                     double inv_v, const float *samples, int M, const float o0[3],
                                     float c, float inv_ts, Cell cells[kGroup], float dp[3],
                                     float tq[3]) {
  const int lane = threadIdx.x & 63;
  double Rv[9];
  for (int a = 0; a < 9; ++a) Rv[a] = r.R[a] * inv_v;
  float s[kGroup] = {}, d[3][kGroup] = {}, t[3][kGroup] = {};
#pragma unroll
  for (int j = 0; j < kGroup; ++j) {
    if (j >= count) break;
    const PairView w = pair_view(pb, Rv, j);
    float dj[3] = {0.f, 0.f, 0.f}, tj[3] = {0.f, 0.f, 0.f};
    if (lane < M) s[j] += smooth_sample<G>(f, w, o0, c, inv_ts, cells[j], dj, tj);
    for (int m0 = 64; m0 < M; m0 += 64) {
      const int m = m0 + lane;
      if (m < M) {
        const float o[3] = {samples[3 * m], samples[3 * m + 1], samples[3 * m + 2]};
        Cell any;
        any.x[0] = kNoCell;
        s[j] += smooth_sample<G>(f, w, o, c, inv_ts, any, dj, tj);
      }
    }
    for (int a = 0; a < 3; ++a) {
      d[a][j] = dj[a];
      t[a][j] = tj[a];
    }
  }
  for (int a = 0; a < 3; ++a) {
    dp[a] = G == 1 ? wave_sums(d[a]) * (inv_ts * (float)inv_v) : 0.f;
    tq[a] = G > 0 ? wave_sums(t[a]) * inv_ts : 0.f;
  }
  return G == 2 ? 0.f : wave_sums(s);
}

// ds/dq from the torque tau: 2 (-tau.v, w tau + tau x v) / |q|.
__device__ inline void unnormalise(const Rot &r, const float tq[3], float dq[4]) {
  const float w = r.qn[0], x = r.qn[1], y = r.qn[2], z = r.qn[3];
  const float k = 2.f / r.nq;
  dq[0] = -k * (tq[0] * x + tq[1] * y + tq[2] * z);
  dq[1] = k * (w * tq[0] + tq[1] * z - tq[2] * y);
  dq[2] = k * (w * tq[1] + tq[2] * x - tq[0] * z);
  dq[3] = k * (w * tq[2] + tq[0] * y - tq[1] * x);
}

// Work distribution: every pair takes the same work, so the groups go round
// the waves without a counter.  Workgroup i runs on XCD i mod 8, each with its
// own L2: a wave's place counts the workgroups XCD by XCD, so that in each round
// the waves sharing an L2 take neighbouring groups.  (Over the rounds every XCD
// reads the whole map: of 64 M pairs of ordered points 55 % of the reads hit L2.)
constexpr int kXcds = 8;

__device__ inline int64_t smooth_wave() {
  const int64_t per = gridDim.x / kXcds;   // a multiple of kXcds workgroups
  return ((blockIdx.x % kXcds) * per + blockIdx.x / kXcds) * (kSmoothThreads / 64) +
         __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

__device__ inline void lane_sample(const float *samples, int M, float o[3]) {
  const int lane = threadIdx.x & 63;
  const int m = lane < M ? lane : 0;
  o[0] = samples[3 * m];
  o[1] = samples[3 * m + 1];
  o[2] = samples[3 * m + 2];
}

template <int G>
__global__ void __launch_bounds__(kSmoothThreads)
k_smooth_eval(SmoothField field, double v, const float *p, const float *q, int64_t n, int group,
              const float *samples, int M, float c, float tau_s, const float *grad_s,
              float *s_out, float *dq_out, float *dp_out) {
  const int lane = threadIdx.x & 63;
  const FieldView f = field_view(field);
  const double inv_v = 1.0 / v;
  const float inv_ts = 1.f / tau_s;
  float o0[3];
  lane_sample(samples, M, o0);
  const int64_t waves = (int64_t)gridDim.x * (kSmoothThreads / 64);
  for (int64_t b0 = smooth_wave() * group; b0 < n; b0 += waves * group) {
    const int count = (int)(n - b0 < group ? n - b0 : group);
    const int own = lane & (kGroup - 1);
    const int64_t i = b0 + (own < count ? own : 0);
    Cell cells[kGroup];
    for (int j = 0; j < kGroup; ++j) cells[j].x[0] = kNoCell;
    const PairBase pb = pair_base(p + 3 * i, v);
    const float q4[4] = {q[4 * i], q[4 * i + 1], q[4 * i + 2], q[4 * i + 3]};
    const Rot r = make_rot(q4);
    const float gs = grad_s ? grad_s[i] : 1.f;
    float dp[3], tq[3];
    const float s = smooth_group<G>(f, pb, r, count, inv_v, samples, M, o0, c, inv_ts, cells, dp, tq);
    if (lane < count) {
      if (s_out) s_out[i] = s;
      if (G == 1) {
        float dq[4];
        for (int a = 0; a < 3; ++a) tq[a] *= gs;
        unnormalise(r, tq, dq);
        for (int a = 0; a < 4; ++a) dq_out[4 * i + a] = dq[a];
        for (int a = 0; a < 3; ++a) dp_out[3 * i + a] = gs * dp[a];
      }
    }
  }
}

// Orientation ascent: per (point, start) pair, `steps` updates
// q <- (q + D) / |q + D|, D = eta ds/dq clipped to length max_step, with q
// kept in registers; then s at the final q.
__global__ void __launch_bounds__(kSmoothThreads)
k_smooth_refine(SmoothField field, double v, const float *p, int64_t n_points, const float *q0,
                int n_starts, int group, const float *samples, int M, float c, float tau_s, int steps,
                float eta, float max_step, float *q_out, float *s_out) {
  const int lane = threadIdx.x & 63;
  const FieldView f = field_view(field);
  const int64_t n = n_points * n_starts;
  const double inv_v = 1.0 / v;
  const float inv_ts = 1.f / tau_s;
  float o0[3];
  lane_sample(samples, M, o0);
  const int64_t waves = (int64_t)gridDim.x * (kSmoothThreads / 64);
  for (int64_t b0 = smooth_wave() * group; b0 < n; b0 += waves * group) {
    const int count = (int)(n - b0 < group ? n - b0 : group);
    const int own = lane & (kGroup - 1);
    const int64_t i = b0 + (own < count ? own : 0);
    Cell cells[kGroup];
    for (int j = 0; j < kGroup; ++j) cells[j].x[0] = kNoCell;
    const PairBase pb = pair_base(p + 3 * (i / n_starts), v);
    float q[4] = {q0[4 * i], q0[4 * i + 1], q0[4 * i + 2], q0[4 * i + 3]};
    float dp[3], tq[3], dq[4];
    for (int t = 0; t < steps; ++t) {
      const Rot r = make_rot(q);
      smooth_group<2>(f, pb, r, count, inv_v, samples, M, o0, c, inv_ts, cells, dp, tq);
      unnormalise(r, tq, dq);
      float D[4], len = 0.f;
      for (int a = 0; a < 4; ++a) {
        D[a] = eta * dq[a];
        len += D[a] * D[a];
      }
      len = sqrtf(len);
      const float sc = len > max_step ? max_step / len : 1.f;
      float nn = 0.f;
      for (int a = 0; a < 4; ++a) {
        q[a] += D[a] * sc;
        nn += q[a] * q[a];
      }
      nn = sqrtf(nn);
      for (int a = 0; a < 4; ++a) q[a] /= nn;
    }
    const Rot r = make_rot(q);
    const float s = smooth_group<0>(f, pb, r, count, inv_v, samples, M, o0, c, inv_ts, cells, dp, tq);
    if (lane < count) {
      s_out[i] = s;
      for (int a = 0; a < 4; ++a) q_out[4 * i + a] = r.qn[a];
    }
  }
}

// Pairs a wave takes at once, and the grid: one each where there are fewer
// pairs than waves on the chip, else so many (at most kGroup) that those waves
// all go the same number of rounds.  (1,000 pairs: 19 us in batches of 16 a
// wave, 4.5 with one a wave.)
struct SmoothShape {
  int group;
  unsigned grid;
};

SmoothShape smooth_shape(const void *fn, int64_t pairs) {
  static int n_cu = 0;
  if (n_cu == 0) {
    int dev = 0;
    hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n_cu <= 0)
      n_cu = 1;
  }
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kSmoothThreads, 0) != hipSuccess ||
      per_cu <= 0)
    per_cu = 1;
  const int64_t per_wg = kSmoothThreads / 64, waves = (int64_t)per_cu * n_cu * per_wg;
  const int64_t rounds = (pairs + kGroup * waves - 1) / (kGroup * waves);
  SmoothShape sh;
  sh.group = (int)std::max<int64_t>(1, (pairs + rounds * waves - 1) / (rounds * waves));
  const int64_t wgs = (pairs + per_wg * sh.group - 1) / (per_wg * sh.group);
  const int64_t grid = std::min<int64_t>(wgs, (int64_t)per_cu * n_cu);
  sh.grid = (unsigned)((grid + kXcds - 1) / kXcds * kXcds);
  return sh;
}

}  // namespace

void launch_smooth_prepare(const Params &p, MapDev m, int64_t n_blocks, GridDev g,
                           int64_t grid_bricks, float tau, const SmoothBuffers &b,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_field_clear,
                     dim3((unsigned)std::max<int64_t>(
                         1, std::min<int64_t>(1024, grid_bricks / kSmoothThreads))),
                     dim3(kSmoothThreads), 0, s, b.bid9, grid_bricks, b.count, tau, b.T9);
  if (n_blocks <= 0 || grid_bricks <= 0) return;
  hipLaunchKernelGGL(k_apron_mark,
                     dim3((unsigned)((8 * n_blocks + kSmoothThreads - 1) / kSmoothThreads)),
                     dim3(kSmoothThreads), 0, s, m, n_blocks, g, b.bid9, b.count, b.brick_of, b.apron_cap);
  hipLaunchKernelGGL(k_apron_fill, dim3((unsigned)std::min<int64_t>(b.apron_cap, 2048)),
                     dim3(kSmoothThreads), 0, s, m, b.count, b.brick_of, g, p.scale, tau, b.apron_cap,
                     b.T9);
}

void launch_smooth_eval(const SmoothField &f, double v, const float *p, const float *q, int64_t n,
                        const float *samples, int32_t M, float c, float tau_s,
                        const float *grad_s, float *s_out, float *dq, float *dp, hipStream_t s) {
  if (n <= 0) return;
  const auto fn = dq ? k_smooth_eval<1> : k_smooth_eval<0>;
  const SmoothShape sh = smooth_shape((const void *)fn, n);
  hipLaunchKernelGGL(fn, dim3(sh.grid), dim3(kSmoothThreads), 0, s, f, v, p, q, n, sh.group, samples,
                     M, c, tau_s, grad_s, s_out, dq, dp);
}

void launch_smooth_refine(const SmoothField &f, double v, const float *p, int64_t n_points,
                          const float *q0, int32_t n_starts, const float *samples, int32_t M,
                          float c, float tau_s, int32_t steps, float eta, float max_step,
                          float *q_out, float *s_out, hipStream_t s) {
  const int64_t n = n_points * n_starts;
  if (n <= 0) return;
  const SmoothShape sh = smooth_shape((const void *)k_smooth_refine, n);
  hipLaunchKernelGGL(k_smooth_refine, dim3(sh.grid), dim3(kSmoothThreads), 0, s, f, v, p, n_points, q0,
                     n_starts, sh.group, samples, M, c, tau_s, steps, eta, max_step, q_out, s_out);
}

}  // namespace af
