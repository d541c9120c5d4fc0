// ProximityTaxel readout (App. A.6) behind include/tg_proximity.h.
//
// Per (env, taxel, step) the taxel sums, over the tracked object's surface points inside its
// sensing sphere, the penetration P_ij = R_j - |p_i - q_j| and its first moment P_ij (p_i - q_j).
// Every channel of the sensor follows from those two moments, because a point's velocity
// v_O + w_O x (p_i - p_O) is affine in its position:
//   sum P v_p  = S0 (v_O + w_O x (q_j - p_O)) + w_O x S1,      S0 = sum P,  S1 = sum P (p_i - q_j)
//   f   = k rho S0 a + k_s rho [V - a (V . a)],  V = sum P v_p - S0 v_tax
//   tau = k rho S1 x a
// The neighbour search runs in the object frame (distances are rotation invariant).  Where few points
// are in reach of a taxel, a thread takes a probe (tg_prox_cells_kernel; cells_are_faster draws the line).
// Otherwise create sorts each cloud by recursive median splits into chunks of 8 points, and keeps a
// bounding sphere per chunk, per 8 chunks and per 512 chunks.  Create also splits every link's taxels
// into tiles of at most 16 neighbouring probes.  A wave takes one tile of one env: its lanes test the
// spheres against the tile's box grown by the probes' radius, list the chunks that pass, and run
// through the list eight chunks at a time.  Every (point, probe) pair of a listed chunk is evaluated,
// without branches, as two contractions on the matrix cores in FP32 (v_mfma_f32_4x4x1: 16
// independent 4 x 4 blocks, the points broadcast to the blocks of the tile's probe quads):
//   p - q = p 1 + (-q), one axis at a time, and
//   (S1 + S0 q, S0) = sum over points of max(R - |p - q|, 0) (p, 1), p and q from the tile's centre.
// Each axis of a difference is rounded once, as a subtraction would be, so a pair's penetration has
// the error of its own distance however near the point and however wide the tile; the square as
// |q|^2 - 2 p . q + |p|^2, a quarter of the vector instructions, loses the digits of near points (a
// point at a probe of R = 1 cm: 5 um off) and of small probes in wide tiles.  Error of the channels
// against FP64 over 16 steps of the hand: 1.2e-7; 4.4e-7 with the sums in one chain per probe.
//
// Bound: vector issue: per 256 pairs 12 instructions for the squares, 4 square roots, 4 subtractions
// and the 7 MFMA, and about as much again of loads, sphere tests and set-up per tile.  Measured on the
// hand, 4096 envs x 200 taxels x 16 steps, 5000-point clouds: 4.7 ms (4.1 with the expanded square)
// against 21.4 ms for a thread a probe, where the lanes of a wave run the union of their rows of cells
// and a pair costs about 13 vector instructions.  About 766 pairs are evaluated
// per probe (372 lie inside the sphere).  Before the differences: chunks of 4 points and of 16 evaluate
// 704 and 856, but cost or save sphere tests: 4.5 ms with 4; a sphere instead of a box around the tile
// evaluates 986.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/tg_proximity.h"
#include "readout_device.h"

using namespace tg;

namespace {
thread_local std::string g_prox_create_error;
constexpr int PX_THREADS = 256;   // also the most taxels of a workgroup's span
constexpr int PX_WAVES = PX_THREADS / 64;
constexpr int PX_ENVS = 16;       // most envs of a workgroup
constexpr int PX_CHUNK = 8;       // points of a chunk
constexpr int PX_LIST = 256;      // a wave's list of chunks; run through when 64 more may not fit

struct CloudDesc {       // one object's chunks
  int32_t chunk0;        // first chunk
  int32_t n_chunks;
  int32_t group0;        // first sphere over 8 chunks
  int32_t super0;        // first sphere over 64 groups
  int32_t n_points;      // N_active of an env holding this object
  int32_t pad[3];
};

struct ProxTile {        // up to 16 neighbouring probes of one link
  float centre[3];       // link frame
  int32_t link;
  int32_t nq;            // probe quads, as a power of two: 0, 1, 2
  int32_t pad[3];
  int16_t probe[16];     // taxel within the span, -1: none
};

struct ProxSpan {        // taxels [j0, j0 + n) and tiles [t0, t0 + nt) of a workgroup
  int32_t j0, n, t0, nt;
};

struct CloudCells {      // one object's cell grid, where the taxels walk cells
  float origin[3];       // corner of cell (0, 0, 0), object frame
  float hinv;            // 1 / cell edge
  int32_t dims[3];       // cells per axis
  int32_t cell_off;      // first entry of this object's cell table (dims product + 1 entries)
  float h;               // cell edge
  int32_t pad[3];
};

struct ProxParams {
  int32_t E, L, T, n_obj;
  int32_t n_spans, envs;    // envs: envs per workgroup (1 with more than one span)
  int32_t dummy;            // a chunk of padding points
  float k, k_s, density, radius_rho, two_rho, neg_rho;
  uint32_t key0, key1;
  const float4* tax_a;      // [T] (x_j, R_j)
  const float4* tax_b;      // [T] (n_j, link id as float bits)
  const CloudDesc* clouds;  // [n_obj]  (with cells: n_points alone)
  const ProxSpan* spans;
  const ProxTile* tiles;
  const float4* sphere;     // [chunks] centre, radius (object frame)
  const float4* group;      // spheres over 8 chunks
  const float4* super;      // spheres over 64 groups
  const float4* pts;        // [chunks][8] points (x, y, z, 0), object frame
  const float4* mom;        // [chunks][2][4]: x, y, z of four of the chunk's points, then ones
  const CloudCells* grids;  // [n_obj], null: tiles
  const int32_t* cells;     // concatenated cell start tables (point index into pts, sorted by cell)
};

struct ProxLaunch {
  const float* link_state;  // [S][13][E*L]
  const float* obj_state;   // [S][13][E] or null
  const int32_t* obj_id;    // [S][E]
  float* ft;                // [S][6][E][T]
  float* mass;              // [S][E][T] or null
  const float* gain;        // [E][T] or null
  int64_t step0;
  int32_t n_steps;
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The clamp modifier of the instruction that gives x (0 for a NaN).
__device__ __forceinline__ float clamp01(float x) { return __builtin_amdgcn_fmed3f(x, 0.f, 1.f); }

// Eight listed chunks against the 4 << NQ probes of a tile.  Lane 4 i + k carries point k of quad i
// and row k of quad i's moment operand (x: one value per point).  Block b of the 16 serves probe
// quad b mod 2^NQ; the blocks that differ only in it form a broadcast group, which takes each of
// its own point quads in turn (the instruction's broadcast-block field).  qx, qy, qz: the lane's
// probe, negated, once for each of a quad's points, so that p u - q u comes out of the matrix core as
// one rounded difference.  The tile's unit u, a power of two, makes its radii at most 1 (u = 1 below a
// metre), so that max(R - d, 0) is the clamp modifier of the subtraction: 4.70 ms per 16 steps of the
// hand against 5.02 with an instruction for the maximum.
template <int NQ>
__device__ __forceinline__ void prox_group(const float4& pt, const f32x4& x, float u, const f32x4& qx, const f32x4& qy,
                                           const f32x4& qz, float R, f32x4& M0, f32x4& M1) {
  f32x4 w[4];
#define PX_TURNS(F) F(0) F(1) F(2) F(3)
#define PX_ON(A) if constexpr ((A) < (1 << NQ))
#define PX_W(A)                                                                                                 \
  PX_ON(A) {                                                                                                    \
    const f32x4 dx = __builtin_amdgcn_mfma_f32_4x4x1f32(pt.x, u, qx, NQ, A, 0);                                 \
    const f32x4 dy = __builtin_amdgcn_mfma_f32_4x4x1f32(pt.y, u, qy, NQ, A, 0);                                 \
    const f32x4 dz = __builtin_amdgcn_mfma_f32_4x4x1f32(pt.z, u, qz, NQ, A, 0);                                 \
    _Pragma("unroll") for (int r = 0; r < 4; ++r)                                                               \
        w[A][r] = clamp01(R - __builtin_amdgcn_sqrtf(fmaf(dz[r], dz[r], fmaf(dy[r], dy[r], dx[r] * dx[r]))));   \
  }
#define PX_M(A)                                                                                                 \
  PX_ON(A) {                                                                                                    \
    M0 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[0], w[A][0], M0, NQ, A, 0);                                       \
    M1 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[1], w[A][1], M1, NQ, A, 0);                                       \
    M0 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[2], w[A][2], M0, NQ, A, 0);                                       \
    M1 = __builtin_amdgcn_mfma_f32_4x4x1f32(x[3], w[A][3], M1, NQ, A, 0);                                       \
  }
  PX_TURNS(PX_W) PX_TURNS(PX_M)
#undef PX_TURNS
#undef PX_ON
#undef PX_W
#undef PX_M
}

// Maximum over each row of 16 lanes, in every lane.
__device__ __forceinline__ float row_max(float v) {
#define PX_ROR(n) v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + n, 0xF, 0xF, true)));
  PX_ROR(8) PX_ROR(4) PX_ROR(2) PX_ROR(1)
#undef PX_ROR
  return v;
}
// v plus the value of the lane n places on in its row of 16 (around it)
template <int n>
__device__ __forceinline__ float add_ror(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + n, 0xF, 0xF, true));
}
// Sum of the four rows of 16 lanes, in every lane: two exchanges of half rows of the wave.
__device__ __forceinline__ float rows_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Set bits of a wave's mask below this lane.
__device__ __forceinline__ int lane_rank(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// A pose's position and quaternion at one column of step s.
__device__ __forceinline__ void load_pose7(const float* state, int64_t cols, int64_t s, int64_t col, float* v) {
#pragma unroll
  for (int c = 0; c < 7; ++c) v[c] = state[(s * 13 + c) * cols + col];
}
// A taxel's link and its env's object at one step.
struct ProxFrame {
  float pL[3], RL[9];   // the link's pose
  float x[3];           // R_L x_j = q_j - p_L
  float pO[3], RO[9];   // the object's pose (the origin without object states)
};
__device__ __forceinline__ void load_frame(const ProxParams& p, const ProxLaunch& q, int s, int e, const float4& ta,
                                           int l, bool object, ProxFrame& f) {
  float v[7], o[7] = {0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f};
  load_pose7(q.link_state, (int64_t)p.E * p.L, s, (int64_t)e * p.L + l, v);
  if (object && q.obj_state) load_pose7(q.obj_state, p.E, s, e, o);
  quat_to_R(v[3], v[4], v[5], v[6], f.RL);
  quat_to_R(o[3], o[4], o[5], o[6], f.RO);
  mat_vec(f.RL, ta.x, ta.y, ta.z, f.x);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    f.pL[i] = v[i];
    f.pO[i] = o[i];
  }
}
// The six velocities at one column of step s.
__device__ __forceinline__ void load_velocity(const float* state, int64_t cols, int64_t s, int64_t col, float* v) {
#pragma unroll
  for (int c = 0; c < 6; ++c) v[c] = state[(s * 13 + 7 + c) * cols + col];
}
// One taxel's channels of step s from its moments (object frame).  npts: its env's points, 0 without
// an object.
__device__ __forceinline__ void put_channels(const ProxParams& p, const ProxLaunch& q, int s, int e, int j,
                                             const float4& tb, const ProxFrame& w, int npts, float S0, float S1x,
                                             float S1y, float S1z) {
  const int64_t ET = (int64_t)p.E * p.T, idx = (int64_t)e * p.T + j;
  const float g = q.gain ? q.gain[idx] : 1.0f;
  float f[3] = {0.f, 0.f, 0.f}, tau[3] = {0.f, 0.f, 0.f};
  if (npts > 0) {
    const float rho = p.density / (float)npts;
    float a[3], Sw[3], vL[6], vO[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    load_velocity(q.link_state, (int64_t)p.E * p.L, s, (int64_t)e * p.L + __float_as_int(tb.w), vL);
    if (q.obj_state) load_velocity(q.obj_state, p.E, s, e, vO);
    mat_vec(w.RL, tb.x, tb.y, tb.z, a);          // a_j
    mat_vec(w.RO, S1x, S1y, S1z, Sw);            // world-frame sum P (p_i - q_j)
    // relative velocity moment V = S0 (v_O + w_O x (q - p_O) - v_tax) + w_O x Sw
    float rq[3], c1[3], c2[3], c3[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) rq[i] = (w.pL[i] + w.x[i]) - w.pO[i];
    cross3(vO + 3, rq, c1);                      // w_O x (q - p_O)
    cross3(vL + 3, w.x, c2);                     // w_L x (q - p_L)
    cross3(vO + 3, Sw, c3);
    float V[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) V[i] = fmaf(S0, (vO[i] + c1[i]) - (vL[i] + c2[i]), c3[i]);
    const float vn = fmaf(V[2], a[2], fmaf(V[1], a[1], V[0] * a[0]));
    const float kr = p.k * rho, ksr = p.k_s * rho;
    float t3[3];
    cross3(Sw, a, t3);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      f[i] = fmaf(kr * S0, a[i], ksr * fmaf(-a[i], vn, V[i]));
      tau[i] = kr * t3[i];
    }
  }
  float fl[3], tl[3];
  mat_T_vec(w.RL, f[0], f[1], f[2], fl);
  mat_T_vec(w.RL, tau[0], tau[1], tau[2], tl);
  float* out = q.ft + (int64_t)s * 6 * ET + idx;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    __builtin_nontemporal_store(g * fl[i], out + i * ET);
    __builtin_nontemporal_store(g * tl[i], out + (3 + i) * ET);
  }
  if (q.mass) __builtin_nontemporal_store(S0, q.mass + (int64_t)s * ET + idx);
}
}  // namespace

// 4 waves a SIMD: 127 registers and no scratch, 4.69 ms; 5 waves spill 27 of 96 registers: 4.74.
__global__ __launch_bounds__(PX_THREADS, 4) void tg_prox_kernel(const ProxParams p, const ProxLaunch q) {
  __shared__ float4 s_q[2 * PX_THREADS];      // per env: the span's probe centres (and R), its tile centres
  __shared__ float4 s_rot[PX_THREADS];        // per (env, tile): rotation link frame -> object frame
  __shared__ float4 s_sum[PX_THREADS];        // per (env, probe): S0, S1 (object frame)
  __shared__ int32_t s_list[PX_WAVES][PX_LIST];
  __shared__ int32_t s_groups[PX_WAVES][64];
  __shared__ int32_t s_oid[PX_ENVS];
  __shared__ int32_t s_next;
  const int64_t EL = (int64_t)p.E * p.L;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e_blk = blockIdx.x / p.n_spans;
  const ProxSpan sp = p.spans[blockIdx.x - e_blk * p.n_spans];
  const int e0 = e_blk * p.envs;
  const int ne = min(p.envs, p.E - e0);
  const int per = sp.n + sp.nt;
  // one step per block row (the steps are independent)
  for (int s = blockIdx.y; s < q.n_steps; s += gridDim.y) {
    const int32_t* oid_s = q.obj_id + (int64_t)s * p.E + e0;
    // 1. probe and tile centres in the object frame, radii
    if (tid == 0) s_next = 0;
    if (tid < ne) {
      const int oid = oid_s[tid];
      s_oid[tid] = oid >= 0 && oid < p.n_obj ? oid : -1;
    }
    for (int i = tid; i < ne * per; i += PX_THREADS) {
      const int el = i / per, r = i - el * per, e = e0 + el;
      float c[3], R = 0.f;
      int l;
      if (r < sp.n) {
        const float4 ta = p.tax_a[sp.j0 + r];
        c[0] = ta.x; c[1] = ta.y; c[2] = ta.z;
        R = ta.w;
        l = __float_as_int(p.tax_b[sp.j0 + r].w);
      } else {
        const ProxTile& tl = p.tiles[sp.t0 + r - sp.n];
        c[0] = tl.centre[0]; c[1] = tl.centre[1]; c[2] = tl.centre[2];
        l = tl.link;
      }
      float v[7], RL[9], x[3], qo[3];
      load_pose7(q.link_state, EL, s, (int64_t)e * p.L + l, v);
      quat_to_R(v[3], v[4], v[5], v[6], RL);
      mat_vec(RL, c[0], c[1], c[2], x);
      float o[7] = {0.f, 0.f, 0.f, 1.f, 0.f, 0.f, 0.f}, RO[9];
      if (q.obj_state) load_pose7(q.obj_state, p.E, s, e, o);
      quat_to_R(o[3], o[4], o[5], o[6], RO);
      mat_T_vec(RO, (v[0] + x[0]) - o[0], (v[1] + x[1]) - o[1], (v[2] + x[2]) - o[2], qo);
      if (r < sp.n && p.radius_rho > 0.f) {
        uint32_t x0 = (uint32_t)e, x1 = (uint32_t)(sp.j0 + r), x2 = (uint32_t)(q.step0 + s), x3 = 9u;
        philox4x32_10(x0, x1, x2, x3, p.key0, p.key1);
        R = R + fmaf(u01(x0), p.two_rho, p.neg_rho);
        R = R > 0.f ? R : 0.f;
      }
      if (!(R < INFINITY)) R = 0.f;   // an infinite sphere senses nothing
      s_q[i] = make_float4(qo[0], qo[1], qo[2], R);
      if (r >= sp.n) {   // conj(q_O) q_L
        const float w = o[3], a = o[4], b = o[5], c = o[6];
        s_rot[el * sp.nt + r - sp.n] = make_float4(w * v[3] + a * v[4] + b * v[5] + c * v[6], w * v[4] - a * v[3] - b * v[6] + c * v[5],
                                                   w * v[5] + a * v[6] - b * v[3] - c * v[4], w * v[6] - a * v[5] + b * v[4] - c * v[3]);
      }
    }
    __syncthreads();
    // 2. tiles, taken in turn by the waves (the largest first)
    int32_t *list = s_list[wave], *groups = s_groups[wave];
    for (;;) {
      int task = 0;
      if (lane == 0) task = atomicAdd(&s_next, 1);
      task = __builtin_amdgcn_readfirstlane(task);
      if (task >= ne * sp.nt) break;
      const int tile = ne == 1 ? task : task / ne, el = task - tile * ne;
      const ProxTile& tl = p.tiles[sp.t0 + tile];
      const int nq = tl.nq;
      const int col = lane & 3;
      const int pi = tl.probe[(((lane >> 2) & ((1 << nq) - 1)) << 2) + col];
      const int oid = __builtin_amdgcn_readfirstlane(s_oid[el]);
      const float4 ctr = s_q[el * per + sp.n + tile];
      const float4 pr = pi >= 0 ? s_q[el * per + pi] : make_float4(ctr.x, ctr.y, ctr.z, 0.f);
      const float R = pr.w;
      const float ax = pr.x - ctr.x, ay = pr.y - ctr.y, az = pr.z - ctr.z;
      f32x4 M = {0.f, 0.f, 0.f, 0.f};
      if (oid >= 0) {
        // The tile's box in its link's frame, and how far its probes sense: grown by a relative 1e-5
        // (and 0.1 um), so rounding never drops a quad that holds a point inside a sphere.  The
        // axes come from the normalised quaternion, so they are orthonormal for any input.
        const float4 rq = s_rot[el * sp.nt + tile];
        const float rn = __builtin_amdgcn_rsqf(fmaf(rq.w, rq.w, fmaf(rq.z, rq.z, fmaf(rq.y, rq.y, rq.x * rq.x))));
        float B[9];
        quat_to_R(rq.x * rn, rq.y * rn, rq.z * rn, rq.w * rn, B);
        float hb[3];
        mat_T_vec(B, ax, ay, az, hb);
#pragma unroll
        for (int k = 0; k < 3; ++k) hb[k] = pi >= 0 ? fabsf(hb[k]) * 1.00001f : 0.f;
        const float rmax = row_max(R), far = rmax > 0.f ? fmaf(rmax, 1.00001f, 1e-7f) : 0.f;
        const int ue = max(0, __builtin_amdgcn_frexp_expf(rmax));
        const float u = __builtin_amdgcn_ldexpf(1.f, -ue);
#pragma unroll
        for (int k = 0; k < 3; ++k) hb[k] = row_max(hb[k]);
        auto near = [&](const float4& c) {   // (kept when NaN)
          float z[3];
          mat_T_vec(B, c.x - ctr.x, c.y - ctr.y, c.z - ctr.z, z);
#pragma unroll
          for (int k = 0; k < 3; ++k) z[k] = fmaxf(fabsf(z[k]) - hb[k], 0.f);
          const float r = c.w + far;
          return !(fmaf(z[2], z[2], fmaf(z[1], z[1], z[0] * z[0])) >= r * r);
        };
        const float nx = -pr.x * u, ny = -pr.y * u, nz = -pr.z * u;
        const f32x4 qx = {nx, nx, nx, nx}, qy = {ny, ny, ny, ny}, qz = {nz, nz, nz, nz};
        const float cc = col == 0 ? ctr.x : (col == 1 ? ctr.y : (col == 2 ? ctr.z : 0.f));
        const CloudDesc cd = p.clouds[oid];
        f32x4 M1 = {0.f, 0.f, 0.f, 0.f};
        auto run = [&](int n, auto nqc) {   // the first n of the list, eight chunks at a time
          n = __builtin_amdgcn_readfirstlane(n);
          for (int it = 0; it < n; it += 8) {
            const int i = it + (lane >> 3);
            const int64_t at = (int64_t)(i < n ? list[i] : p.dummy) * PX_CHUNK + (lane & 7);
            const float4 pt = p.pts[at];
            const float4 m = p.mom[at];
            const f32x4 x = {m.x - cc, m.y - cc, m.z - cc, m.w - cc};
            prox_group<decltype(nqc)::value>(pt, x, u, qx, qy, qz, R * u, M, M1);
          }
        };
        int cnt = 0;
        auto run_list = [&](int n) {
          __builtin_amdgcn_wave_barrier();
          if (nq == 2) run(n, std::integral_constant<int, 2>{});
          else if (nq == 1) run(n, std::integral_constant<int, 1>{});
          else run(n, std::integral_constant<int, 0>{});
          __builtin_amdgcn_wave_barrier();
        };
        // Above 8192 points (128 groups) a sphere over 64 groups is tested first.
        const int n_groups = far > 0.f ? (cd.n_chunks + 7) >> 3 : 0;
        for (int g0 = 0; g0 < n_groups; g0 += 64) {
          if (n_groups > 128 && __builtin_amdgcn_readfirstlane(!near(p.super[cd.super0 + (g0 >> 6)]))) continue;
          const bool ing = g0 + lane < n_groups && near(p.group[cd.group0 + min(g0 + lane, n_groups - 1)]);
          const uint64_t gmask = __ballot(ing);
          if (ing) groups[lane_rank(gmask)] = g0 + lane;
          const int ng = __popcll(gmask);
          __builtin_amdgcn_wave_barrier();
          for (int g = 0; g < ng; g += 8) {
            if (cnt > PX_LIST - 64) {
              run_list(cnt & ~7);
              const int done = cnt & ~7;   // (the list may be full: nothing is left past its end then)
              cnt -= done;
              const int left = lane < cnt ? list[done + lane] : 0;
              __builtin_amdgcn_wave_barrier();
              if (lane < cnt) list[lane] = left;
            }
            const int gi = g + (lane >> 3);
            const int ci = gi < ng ? groups[gi] * 8 + (lane & 7) : cd.n_chunks;
            const int ch = cd.chunk0 + min(ci, cd.n_chunks - 1);
            const bool in = ci < cd.n_chunks && near(p.sphere[ch]);
            const uint64_t mask = __ballot(in);
            if (in) list[cnt + lane_rank(mask)] = ch;
            cnt += __popcll(mask);
          }
          __builtin_amdgcn_wave_barrier();
        }
        run_list(cnt);
        // add the blocks that share a probe quad (they differ in the lane bits above the quad's)
        M += M1;
        if (nq == 0) {
#pragma unroll
          for (int r = 0; r < 4; ++r) M[r] = add_ror<4>(M[r]);
        }
        if (nq < 2) {
#pragma unroll
          for (int r = 0; r < 4; ++r) M[r] = add_ror<8>(M[r]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) M[r] = __builtin_amdgcn_ldexpf(rows_sum(M[r]), ue);
      }
      if (lane < (4 << nq) && pi >= 0) {
        // moments (x, y, z, 1) about the tile's centre -> S0 and sum P (p - q)
        const float S0 = M[3];
        s_sum[el * sp.n + pi] = S0 > 0.f ? make_float4(S0, fmaf(-S0, ax, M[0]), fmaf(-S0, ay, M[1]), fmaf(-S0, az, M[2]))
                                         : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    __syncthreads();
    // 3. the channels from the moments, one taxel per thread
    if (tid < ne * sp.n) {
      const int el = tid / sp.n, j = sp.j0 + tid - el * sp.n, e = e0 + el, oid = s_oid[el];
      const float4 tb = p.tax_b[j], sum = s_sum[tid];
      ProxFrame w;
      load_frame(p, q, s, e, p.tax_a[j], __float_as_int(tb.w), oid >= 0, w);
      put_channels(p, q, s, e, j, tb, w, oid >= 0 ? p.clouds[oid].n_points : 0, sum.x, sum.y, sum.z, sum.w);
    }
    __syncthreads();   // the shared arrays belong to the next step
  }
}

// Few points in reach of a taxel: a thread a probe.  Each cloud lies in a uniform cell grid, cell edge
// half the largest sensing radius, points sorted by cell, x fastest.  A probe visits the rows of cells
// (fixed y and z) that its sphere reaches; in each the sphere's chord fixes the cells, one contiguous
// run of points.  Neighbouring lanes hold neighbouring taxels of one link and walk nearly the same
// cells; the steps are independent, a block row each.  The poses are
// read again, from cache, after the walk: 74 registers, 6 waves a SIMD and no scratch.  Held over it, 8
// spilled: 4096 envs x 200 taxels x 16 steps, 5000 points, R = 1 mm 1.22 ms, 1.29 held; 2 mm 1.52, 1.67; 20
// points at 10 mm 0.53, 0.57; 8 waves, which spill, 1.20, 1.50 and 0.55.
__global__ __launch_bounds__(PX_THREADS, 6) void tg_prox_cells_kernel(const ProxParams p, const ProxLaunch q) {
  const int64_t idx = (int64_t)blockIdx.x * PX_THREADS + threadIdx.x;
  if (idx >= (int64_t)p.E * p.T) return;
  const int e = (int)(idx / p.T), j = (int)(idx - (int64_t)e * p.T);
  const float4 ta = p.tax_a[j];
  const int l = __float_as_int(p.tax_b[j].w);
  for (int s = blockIdx.y; s < q.n_steps; s += gridDim.y) {
    int oid = q.obj_id[(int64_t)s * p.E + e];
    oid = oid >= 0 && oid < p.n_obj ? oid : -1;
    ProxFrame w;
    load_frame(p, q, s, e, ta, l, oid >= 0, w);
    float S0 = 0.f, S1[3] = {0.f, 0.f, 0.f};
    if (oid >= 0) {
      float qo[3], R = ta.w;
      mat_T_vec(w.RO, (w.pL[0] + w.x[0]) - w.pO[0], (w.pL[1] + w.x[1]) - w.pO[1], (w.pL[2] + w.x[2]) - w.pO[2], qo);
      if (p.radius_rho > 0.f) {
        uint32_t x0 = (uint32_t)e, x1 = (uint32_t)j, x2 = (uint32_t)(q.step0 + s), x3 = 9u;
        philox4x32_10(x0, x1, x2, x3, p.key0, p.key1);
        R = R + fmaf(u01(x0), p.two_rho, p.neg_rho);
        R = R > 0.f ? R : 0.f;
      }
      const CloudCells cd = p.grids[oid];
      const float R2 = R * R;
      // the culling uses a radius grown by a relative 1e-5 (and 0.1 um), so rounding never drops a row
      // or cell that holds a point inside the sphere; the point test is exact
      const float Rc = fmaf(R, 1.00001f, 1e-7f), Rc2 = Rc * Rc;
      int lo[3], hi[3];
      bool empty = !(R > 0.f);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const float u0 = (qo[i] - Rc - cd.origin[i]) * cd.hinv, u1 = (qo[i] + Rc - cd.origin[i]) * cd.hinv;
        // NaN or entirely outside the grid: no points in range
        if (!(u1 >= 0.f) || !(u0 < (float)cd.dims[i])) empty = true;
        lo[i] = u0 > 0.f ? (int)u0 : 0;
        hi[i] = u1 < (float)(cd.dims[i] - 1) ? (int)u1 : cd.dims[i] - 1;
      }
      if (!empty) {
        const int32_t* cs = p.cells + cd.cell_off;
        for (int cz = lo[2]; cz <= hi[2]; ++cz) {
          const float zl = fmaf((float)cz, cd.h, cd.origin[2]);
          const float ez = fmaxf(fmaxf(zl - qo[2], qo[2] - (zl + cd.h)), 0.f);
          for (int cy = lo[1]; cy <= hi[1]; ++cy) {
            const float yl = fmaf((float)cy, cd.h, cd.origin[1]);
            const float ey = fmaxf(fmaxf(yl - qo[1], qo[1] - (yl + cd.h)), 0.f);
            const float c2 = Rc2 - fmaf(ey, ey, ez * ez);
            if (!(c2 > 0.f)) continue;
            const float half = __builtin_amdgcn_sqrtf(c2);
            const float x0 = (qo[0] - half - cd.origin[0]) * cd.hinv, x1 = (qo[0] + half - cd.origin[0]) * cd.hinv;
            const int ax = x0 > (float)lo[0] ? (int)x0 : lo[0];
            const int bx = x1 < (float)hi[0] ? (int)x1 : hi[0];
            if (ax > bx) continue;
            const int row = (cz * cd.dims[1] + cy) * cd.dims[0];
            const int b = cs[row + ax], t = cs[row + bx + 1];
            for (int i = b; i < t; ++i) {
              const float4 pt = p.pts[i];
              const float dx = pt.x - qo[0], dy = pt.y - qo[1], dz = pt.z - qo[2];
              const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
              if (d2 < R2) {
                const float P = R - __builtin_amdgcn_sqrtf(d2);
                S0 += P;
                S1[0] = fmaf(P, dx, S1[0]);
                S1[1] = fmaf(P, dy, S1[1]);
                S1[2] = fmaf(P, dz, S1[2]);
              }
            }
          }
        }
      }
    }
    // the poses are read again (from cache) rather than held over the walk
    int s_ = s, j_ = j;
    asm volatile("" : "+s"(s_), "+v"(j_));
    const float4 tb = p.tax_b[j_];
    load_frame(p, q, s_, e, p.tax_a[j_], __float_as_int(tb.w), oid >= 0, w);
    put_channels(p, q, s_, e, j_, tb, w, oid >= 0 ? p.clouds[oid].n_points : 0, S0, S1[0], S1[1], S1[2]);
  }
}

struct tg_prox {
  ProxParams p{};
  std::vector<void*> allocs;
  std::string err;
};

namespace {
tg_status pfail(tg_prox* h, tg_status s, const std::string& msg) {
  if (h) h->err = msg; else g_prox_create_error = msg;
  return s;
}
template <class T>
hipError_t palloc(tg_prox* h, T** p, size_t n) {
  void* q = nullptr;
  const hipError_t e = hipMalloc(&q, std::max<size_t>(n, 1) * sizeof(T));
  if (e == hipSuccess) h->allocs.push_back(q);
  *p = (T*)q;
  return e;
}
template <class T>
hipError_t pupload(tg_prox* h, const T** p, const std::vector<T>& v) {
  T* d = nullptr;
  hipError_t e = palloc(h, &d, v.size());
  if (e == hipSuccess && !v.empty()) e = hipMemcpy(d, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
  *p = d;
  return e;
}
bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

struct CloudPoint { float x[3]; };

// Reorder p[0, n) by recursive median splits along the longest axis, so that every aligned run of
// `unit` points is compact, and so is every aligned run of unit * 2^k.
void split_sort(CloudPoint* p, int64_t n, int64_t unit) {
  while (n > unit) {
    CloudPoint lo = p[0], hi = p[0];
    for (int64_t i = 1; i < n; ++i)
      for (int k = 0; k < 3; ++k) {
        lo.x[k] = std::min(lo.x[k], p[i].x[k]);
        hi.x[k] = std::max(hi.x[k], p[i].x[k]);
      }
    int ax = 0;
    for (int k = 1; k < 3; ++k)
      if (hi.x[k] - lo.x[k] > hi.x[ax] - lo.x[ax]) ax = k;
    int64_t half = unit;   // the largest unit * 2^k that leaves something to the right
    while (2 * half < n) half *= 2;
    std::nth_element(p, p + half, p + n, [ax](const CloudPoint& u, const CloudPoint& w) { return u.x[ax] < w.x[ax]; });
    split_sort(p, half, unit);
    p += half;
    n -= half;
  }
}

// A sphere around the box of n points: centre, and a radius grown by the rounding of the centre
// and of the kernel's differences (a relative 1e-6 of the coordinates).
float4 bounding_sphere(const CloudPoint* p, int64_t n) {
  CloudPoint lo = p[0], hi = p[0];
  for (int64_t i = 1; i < n; ++i)
    for (int k = 0; k < 3; ++k) {
      lo.x[k] = std::min(lo.x[k], p[i].x[k]);
      hi.x[k] = std::max(hi.x[k], p[i].x[k]);
    }
  float c[3];
  double size = 0, r2 = 0;
  for (int k = 0; k < 3; ++k) {
    c[k] = (float)(0.5 * ((double)lo.x[k] + (double)hi.x[k]));
    size = std::max(size, (double)std::max(std::fabs(lo.x[k]), std::fabs(hi.x[k])));
  }
  for (int64_t i = 0; i < n; ++i) {
    double d2 = 0;
    for (int k = 0; k < 3; ++k) {
      const double d = (double)p[i].x[k] - (double)c[k];
      d2 += d * d;
    }
    r2 = std::max(r2, d2);
  }
  return make_float4(c[0], c[1], c[2], (float)(std::sqrt(r2) * (1.0 + 1e-6) + 1e-6 * size));
}

// Split taxels idx[b, e) of one link into tiles of at most 16 probes, their sensing radii within a
// factor of two and none further from the tile's centre than the smallest of them: the moments are
// taken from the centre, so a wider tile would cost its small probes digits of their torque.
void split_tiles(const float* pos, const float* radius, int32_t* idx, int b, int e, int link, int j0,
                 std::vector<ProxTile>& out) {
  float lo[3], hi[3], rlo = INFINITY, rhi = 0.f;   // (a radius of 0 senses nothing, wherever it lies)
  for (int k = 0; k < 3; ++k) lo[k] = hi[k] = pos[3 * idx[b] + k];
  for (int i = b; i < e; ++i) {
    for (int k = 0; k < 3; ++k) {
      lo[k] = std::min(lo[k], pos[3 * idx[i] + k]);
      hi[k] = std::max(hi[k], pos[3 * idx[i] + k]);
    }
    rhi = std::max(rhi, radius[idx[i]]);
    if (radius[idx[i]] > 0.f) rlo = std::min(rlo, radius[idx[i]]);
  }
  if (rhi > 2.0 * rlo) {
    const double at = std::sqrt((double)rlo * rhi);
    const int left = (int)(std::stable_partition(idx + b, idx + e, [&](int32_t j) { return radius[j] < at; }) - idx);
    split_tiles(pos, radius, idx, b, left, link, j0, out);
    split_tiles(pos, radius, idx, left, e, link, j0, out);
    return;
  }
  ProxTile t{};
  float r2 = 0.f;
  int ax = 0;
  for (int k = 0; k < 3; ++k) {
    t.centre[k] = 0.5f * lo[k] + 0.5f * hi[k];
    if (hi[k] - lo[k] > hi[ax] - lo[ax]) ax = k;
  }
  for (int i = b; i < e; ++i) {
    float d2 = 0.f;
    for (int k = 0; k < 3; ++k) d2 += (pos[3 * idx[i] + k] - t.centre[k]) * (pos[3 * idx[i] + k] - t.centre[k]);
    r2 = std::max(r2, d2);
  }
  const int n = e - b;
  if (n == 1 || (n <= 16 && r2 <= (double)rlo * rlo)) {
    t.link = link;
    t.nq = n > 8 ? 2 : (n > 4 ? 1 : 0);
    for (int i = 0; i < 16; ++i) t.probe[i] = (int16_t)(i < n ? idx[b + i] - j0 : -1);
    out.push_back(t);
    return;
  }
  const int left = n > 16 ? 16 * std::max(1, (n + 15) / 32) : (n + 1) / 2;
  std::nth_element(idx + b, idx + b + left, idx + e, [&](int32_t u, int32_t w) {
    return pos[3 * u + ax] < pos[3 * w + ax] || (pos[3 * u + ax] == pos[3 * w + ax] && u < w);
  });
  split_tiles(pos, radius, idx, b, b + left, link, j0, out);
  split_tiles(pos, radius, idx, b + left, e, link, j0, out);
}

// Which kernel a handle takes: a tile costs a wave its set-up and the sphere tests however few points are in
// reach, and small radii make small tiles.  The two sides are nanoseconds per env and step of a full chip,
// fitted to 20 runs with n, the points that a sphere of the taxels' root mean square radius holds around a
// point of the clouds (32 of them are tried).  200-taxel hand, 4096 envs x 16 steps, tiles / cells in ms:
// 5000-point clouds R = 1 mm 7.39 / 1.29, 2 mm 3.32 / 1.65, 2.5 mm 2.45 / 2.14, 3 mm 2.17 / 2.74, 5 mm
// 2.24 / 6.28, 10 mm 4.69 / 18.5; 300 points, 3 mm 1.68 / 0.76, 10 mm 1.28 / 1.64 (the cells while the
// poses were held over the walk, 5 to 9% slower than now).
bool cells_are_faster(const tg_prox_config& cfg, const std::vector<ProxTile>& tiles) {
  double r2 = 0;
  const double rho = cfg.radius_rho;
  int sensing = 0;
  for (int j = 0; j < cfg.num_taxels; ++j) {
    const double r = cfg.sensing_radius[j];
    if (r + rho > 0 && r + rho < INFINITY) {
      r2 += r * r + rho * rho / 3;
      ++sensing;
    }
  }
  if (!sensing) return true;
  r2 /= sensing;
  int64_t inside = 0, tried = 0;
  const int per = std::max(1, 32 / cfg.num_objects);
  for (int o = 0; o < cfg.num_objects && tried < 32; ++o) {
    const tg_point_cloud& c = cfg.clouds[o];
    const int n = std::min(per, c.num_points);
    for (int t = 0; t < n; ++t, ++tried) {
      const float* a = c.points + 3 * ((int64_t)c.num_points * t / n);
      const int64_t step = std::max<int64_t>(1, c.num_points / 2048);
      for (int64_t i = 0; i < c.num_points; i += step) {
        const float* x = c.points + 3 * i;
        const float dx = x[0] - a[0], dy = x[1] - a[1], dz = x[2] - a[2];
        if (dx * dx + dy * dy + dz * dz < (float)r2) inside += step;
      }
    }
  }
  const double n = tried ? (double)inside / (double)tried : 0.0;
  double by_tile = 0;
  for (const ProxTile& t : tiles) by_tile += t.nq == 0 ? 0.45 + 0.05 * std::sqrt(n) : 0.85 + 0.0055 * n;
  return cfg.num_taxels * (0.04 + 0.0032 * n) < by_tile;
}
}  // namespace

extern "C" {

tg_status tg_prox_create(const tg_prox_config* cfg, tg_prox** out) {
  if (!out) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "out is NULL");
  *out = nullptr;
  if (!cfg) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "cfg is NULL");
  if (cfg->abi_version != TG_ABI_VERSION) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "abi_version mismatch");
  const int E = cfg->num_envs, L = cfg->num_links, T = cfg->num_taxels, NO = cfg->num_objects;
  if (E < 1 || L < 1 || T < 1 || NO < 1) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "sizes must be positive");
  if (!cfg->link_taxel_offset || !cfg->taxel_pos || !cfg->taxel_normal || !cfg->sensing_radius || !cfg->clouds)
    return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "NULL array");
  if ((int64_t)E * T * 6 >= (int64_t(1) << 31)) return pfail(nullptr, TG_ERR_UNSUPPORTED, "E * T * 6 exceeds 2^31");
  const int32_t* off = cfg->link_taxel_offset;
  if (off[0] != 0 || off[L] != T) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "link offsets must run 0..T");
  for (int l = 0; l < L; ++l)
    if (off[l + 1] < off[l]) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "link offsets decrease");
  if (!(cfg->radius_rho >= 0.f) || !(cfg->k >= 0.f) || !(cfg->k_s >= 0.f) || !(cfg->density >= 0.f))
    return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "negative constant");
  float rmax = 0.f;
  std::vector<float4> ta(T), tb(T);
  for (int l = 0; l < L; ++l)
    for (int j = off[l]; j < off[l + 1]; ++j) {
      const float r = cfg->sensing_radius[j];
      if (!(r >= 0.f)) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "negative sensing radius");
      rmax = std::max(rmax, r);
      ta[j] = make_float4(cfg->taxel_pos[3 * j], cfg->taxel_pos[3 * j + 1], cfg->taxel_pos[3 * j + 2], r);
      int li = l;
      float lf;
      std::memcpy(&lf, &li, 4);
      tb[j] = make_float4(cfg->taxel_normal[3 * j], cfg->taxel_normal[3 * j + 1], cfg->taxel_normal[3 * j + 2], lf);
    }
  // Spans of at most PX_THREADS taxels and their tiles, the largest first.
  std::vector<ProxSpan> spans;
  std::vector<ProxTile> tiles;
  std::vector<int32_t> order(T);
  std::iota(order.begin(), order.end(), 0);
  for (int j0 = 0; j0 < T; j0 += PX_THREADS) {
    const int j1 = std::min(T, j0 + PX_THREADS), t0 = (int)tiles.size();
    for (int l = 0; l < L; ++l) {
      const int b = std::max(off[l], j0), e = std::min(off[l + 1], j1);
      // a taxel without a finite position senses nothing; in a tile of its own it spoils no other's centre
      const auto placed = [&](int32_t j) {
        return std::isfinite(ta[j].x) && std::isfinite(ta[j].y) && std::isfinite(ta[j].z);
      };
      int f = b;
      if (b < e) f = (int)(std::stable_partition(order.begin() + b, order.begin() + e, placed) - order.begin());
      if (b < f) split_tiles(cfg->taxel_pos, cfg->sensing_radius, order.data(), b, f, l, j0, tiles);
      for (; f < e; ++f) split_tiles(cfg->taxel_pos, cfg->sensing_radius, order.data(), f, f + 1, l, j0, tiles);
    }
    std::stable_sort(tiles.begin() + t0, tiles.end(), [](const ProxTile& u, const ProxTile& w) { return u.nq > w.nq; });
    spans.push_back({j0, j1 - j0, t0, (int)tiles.size() - t0});
  }
  // A cloud may span at most 2^24 cells of half the largest radius a query can take (at least 0.1 mm).
  const float h = std::max(0.5f * (rmax + cfg->radius_rho), 1e-4f);
  std::vector<CloudDesc> cds(NO);
  std::vector<CloudCells> grids(NO);
  std::vector<int32_t> cells;
  std::vector<float4> sphere, group, super, pts, mom;
  auto pad_chunk = [&] {   // points at infinity, out of every reach; their moments 0 times 0
    for (int i = 0; i < PX_CHUNK; ++i) {
      pts.push_back(make_float4(INFINITY, INFINITY, INFINITY, 0.f));
      mom.push_back(i % 4 == 3 ? make_float4(1.f, 1.f, 1.f, 1.f) : make_float4(0.f, 0.f, 0.f, 0.f));
    }
  };
  for (int o = 0; o < NO; ++o) {
    const tg_point_cloud& c = cfg->clouds[o];
    if (c.num_points < 0 || (c.num_points > 0 && !c.points))
      return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "cloud " + std::to_string(o) + " invalid");
    float lo[3] = {0.f, 0.f, 0.f}, hi[3] = {0.f, 0.f, 0.f};
    for (int64_t i = 0; i < c.num_points; ++i)
      for (int k = 0; k < 3; ++k) {
        const float x = c.points[3 * i + k];
        if (!std::isfinite(x)) return pfail(nullptr, TG_ERR_INVALID_ARGUMENT, "non-finite cloud point");
        lo[k] = i ? std::min(lo[k], x) : x;
        hi[k] = i ? std::max(hi[k], x) : x;
      }
    double ncell = 1;   // (also of clouds whose counts no integer holds)
    CloudCells& g = grids[o];
    for (int k = 0; k < 3; ++k) {
      g.origin[k] = lo[k];
      const double n = std::floor((hi[k] - lo[k]) / h) + 1.0;
      g.dims[k] = (int)std::min(16777216.0, n);
      ncell *= n;
    }
    if (!(ncell <= 16777216.0)) return pfail(nullptr, TG_ERR_UNSUPPORTED, "cloud cell grid too large");
    g.hinv = 1.0f / h;
    g.h = h;
  }
  const bool use_cells = cells_are_faster(*cfg, tiles);
  for (int o = 0; o < NO && use_cells; ++o) {   // counting sort of the points by cell (x fastest)
    const tg_point_cloud& c = cfg->clouds[o];
    CloudCells& g = grids[o];
    cds[o] = CloudDesc{};
    cds[o].n_points = c.num_points;
    g.cell_off = (int32_t)cells.size();
    const int64_t ncell = (int64_t)g.dims[0] * g.dims[1] * g.dims[2];
    std::vector<int32_t> cid(c.num_points), cnt(ncell + 1, 0);
    for (int i = 0; i < c.num_points; ++i) {
      int ci[3];
      for (int k = 0; k < 3; ++k)
        ci[k] = std::min(std::max((int)((c.points[3 * (int64_t)i + k] - g.origin[k]) * g.hinv), 0), g.dims[k] - 1);
      cid[i] = (ci[2] * g.dims[1] + ci[1]) * g.dims[0] + ci[0];
      ++cnt[cid[i] + 1];
    }
    for (int64_t k = 0; k < ncell; ++k) cnt[k + 1] += cnt[k];
    const int32_t base = (int32_t)pts.size();
    for (int64_t k = 0; k <= ncell; ++k) cells.push_back(base + cnt[k]);
    pts.resize(pts.size() + c.num_points);
    for (int i = 0; i < c.num_points; ++i) {
      const float* x = c.points + 3 * (int64_t)i;
      pts[base + cnt[cid[i]]++] = make_float4(x[0], x[1], x[2], 0.f);
    }
  }
  for (int o = 0; o < NO && !use_cells; ++o) {
    const tg_point_cloud& c = cfg->clouds[o];
    std::vector<CloudPoint> cp(c.num_points);
    if (c.num_points) std::memcpy(cp.data(), c.points, c.num_points * sizeof(CloudPoint));
    split_sort(cp.data(), c.num_points, PX_CHUNK);
    CloudDesc& d = cds[o];
    d.chunk0 = (int32_t)sphere.size();
    d.group0 = (int32_t)group.size();
    d.super0 = (int32_t)super.size();
    d.n_points = c.num_points;
    d.n_chunks = (int32_t)(((int64_t)c.num_points + PX_CHUNK - 1) / PX_CHUNK);
    for (int ch = 0; ch < d.n_chunks; ++ch) {
      const int64_t b = (int64_t)ch * PX_CHUNK, e = std::min<int64_t>(b + PX_CHUNK, c.num_points);
      const size_t at = pts.size();
      pad_chunk();
      for (int64_t i = b; i < e; ++i) {
        const float* x = cp[i].x;
        pts[at + (i - b)] = make_float4(x[0], x[1], x[2], 0.f);
        for (int k = 0; k < 3; ++k) (&mom[at + 4 * ((i - b) / 4) + k].x)[(i - b) & 3] = x[k];
      }
      auto over = [&](int64_t chunks) {
        return bounding_sphere(&cp[b], std::min<int64_t>(chunks * PX_CHUNK, c.num_points - b));
      };
      sphere.push_back(over(1));
      if (ch % 8 == 0) group.push_back(over(8));
      if (ch % 512 == 0) super.push_back(over(512));
    }
  }
  const int32_t dummy = (int32_t)sphere.size();
  if (!use_cells) pad_chunk();
  tg_prox* hd = new (std::nothrow) tg_prox();
  if (!hd) return pfail(nullptr, TG_ERR_OUT_OF_MEMORY, "host allocation failed");
  ProxParams& p = hd->p;
  p.E = E; p.L = L; p.T = T; p.n_obj = NO;
  p.n_spans = (int32_t)spans.size();
  // a small hand shares its workgroup with other envs
  p.envs = p.n_spans > 1 ? 1 : std::max(1, std::min(PX_ENVS, PX_THREADS / T));
  p.dummy = dummy;
  p.k = cfg->k; p.k_s = cfg->k_s; p.density = cfg->density;
  p.radius_rho = cfg->radius_rho;
  p.two_rho = 2.0f * cfg->radius_rho;
  p.neg_rho = -cfg->radius_rho;
  p.key0 = (uint32_t)cfg->seed;
  p.key1 = (uint32_t)(cfg->seed >> 32);
  hipError_t e = pupload(hd, &p.tax_a, ta);
  if (e == hipSuccess) e = pupload(hd, &p.tax_b, tb);
  if (e == hipSuccess) e = pupload(hd, &p.clouds, cds);
  if (e == hipSuccess) e = pupload(hd, &p.spans, spans);
  if (e == hipSuccess) e = pupload(hd, &p.tiles, tiles);
  if (e == hipSuccess) e = pupload(hd, &p.sphere, sphere);
  if (e == hipSuccess) e = pupload(hd, &p.group, group);
  if (e == hipSuccess) e = pupload(hd, &p.super, super);
  if (e == hipSuccess) e = pupload(hd, &p.pts, pts);
  if (e == hipSuccess) e = pupload(hd, &p.mom, mom);
  if (e == hipSuccess && use_cells) e = pupload(hd, &p.grids, grids);
  if (e == hipSuccess && use_cells) e = pupload(hd, &p.cells, cells);
  if (e != hipSuccess) {
    tg_prox_destroy(hd);
    return pfail(nullptr, TG_ERR_OUT_OF_MEMORY, std::string("device setup: ") + hipGetErrorString(e));
  }
  *out = hd;
  return TG_OK;
}

tg_status tg_prox_rollout(tg_prox* h, const tg_step_inputs* in, float* ft, float* mass, const float* gain,
                          int32_t n_steps, void* hip_stream) {
  if (!h) return TG_ERR_INVALID_ARGUMENT;
  h->err.clear();
  if (!in || !ft) return pfail(h, TG_ERR_INVALID_ARGUMENT, "inputs or ft is NULL");
  if (n_steps < 0) return pfail(h, TG_ERR_INVALID_ARGUMENT, "n_steps < 0");
  if (n_steps == 0) return TG_OK;
  if (in->step < 0 || in->step + n_steps > (int64_t(1) << 32))
    return pfail(h, TG_ERR_INVALID_ARGUMENT, "steps must lie in [0, 2^32)");
  if (!in->link_state || !in->obj_id) return pfail(h, TG_ERR_INVALID_ARGUMENT, "link_state and obj_id are required");
  if (!aligned16(in->link_state) || !aligned16(in->obj_id) || (in->obj_state && !aligned16(in->obj_state)) ||
      !aligned16(ft) || (mass && !aligned16(mass)) || (gain && !aligned16(gain)))
    return pfail(h, TG_ERR_INVALID_ARGUMENT, "pointers must be 16-byte aligned");
  ProxLaunch q{};
  q.link_state = in->link_state;
  q.obj_state = in->obj_state;
  q.obj_id = in->obj_id;
  q.ft = ft;
  q.mass = mass;
  q.gain = gain;
  q.step0 = in->step;
  q.n_steps = n_steps;
  const int64_t blocks = h->p.grids ? ((int64_t)h->p.E * h->p.T + PX_THREADS - 1) / PX_THREADS
                                    : (int64_t)((h->p.E + h->p.envs - 1) / h->p.envs) * h->p.n_spans;
  const dim3 grid((unsigned)blocks, (unsigned)std::min(n_steps, 65535));
  if (h->p.grids)
    hipLaunchKernelGGL(tg_prox_cells_kernel, grid, dim3(PX_THREADS), 0, (hipStream_t)hip_stream, h->p, q);
  else
    hipLaunchKernelGGL(tg_prox_kernel, grid, dim3(PX_THREADS), 0, (hipStream_t)hip_stream, h->p, q);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? TG_OK : pfail(h, TG_ERR_HIP, hipGetErrorString(e));
}

tg_status tg_prox_destroy(tg_prox* h) {
  if (!h) return TG_OK;
  for (void* p : h->allocs) (void)hipFree(p);
  delete h;
  return TG_OK;
}

const char* tg_prox_last_error(const tg_prox* h) { return h ? h->err.c_str() : g_prox_create_error.c_str(); }

}  // extern "C"
