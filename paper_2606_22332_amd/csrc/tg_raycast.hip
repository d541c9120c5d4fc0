// Raycast contact-depth backend (App. A.1) behind include/tg_raycast.h.
//
// Data: per object a BVH over its triangles, built on the host by median splits along the
// longest axis of the triangle centroids (at most 4 triangles per leaf), boxes grown by a
// relative 1e-6 so FP32 rounding never culls a triangle the exact test would keep.  An interior
// node is one 64-byte record holding its two children's entries (box, and either the child's
// record or its leaf's first triangle and count), so one load gives both boxes and a child that
// fails its test is never loaded; each object's root entry is kept apart.  Triangles are stored
// in leaf order as (a, b, c, outward unit normal), 64 B each, with the mesh's own index.
//
// One wave per (step, span of up to 3 x 64 probes), in four passes with the probes that go on packed
// to the front of an LDS queue in between:
//   1. a lane a probe: its centre in the object frame; a probe that its object's box does not reach
//      (half of them in a grasp) writes its zeros and is done;
//   2. the sphere query: children within R - best of the centre, nearer box first; at a leaf the
//      closest point of each triangle (Voronoi regions of the triangle, with the hardware
//      reciprocal: 1 ulp); best penetration R - dist, the square root taken only for a triangle
//      closer than the bound;
//   3. a lane a probe again: whether it needs the ray query, which it does not where its centre is
//      known to be outside (outside the object's box, or on the outer side of the face holding the
//      closest point), for then its first crossing could only enter the mesh;
//   4. the ray query along -a: children the ray enters before the nearest hit so far, nearer
//      entry first; at a leaf the ray-triangle test (Moller-Trumbore, barycentric slack 1e-6);
//      if the nearest hit leaves the mesh, R + t competes with the sphere's best.
// The traversals park far children on a stack in LDS (one column per lane, so equal stack depths
// fall in different banks).  They are of very unequal length (none to some dozens of nodes), so a lane
// that ends one takes the next of the queue (walk below).
// Bound: vector issue (all of the SIMDs' cycles at 100 steps) with 24 of 64 lanes at work, and behind it
// the L1's data rate: the nodes and triangles come from L1 / L2, the meshes are a few hundred KB.
// 4096 envs x 200 probes x 16 steps, a third of them in contact: 3.26 ms with a thread a probe, whose
// instructions had 10 of 64 lanes at work; 2.42 ms with the reached probes packed and lanes refilled
// for the sphere query, 1.84 ms with the ray query likewise and stacks of 4 bytes an entry (a key
// beside it, tested again before a record is opened, cost 0.3 ms: its LDS holds fewer waves), 1.36 ms
// with each kind of step taken until no lane waits for it (until fewer than 24 do: 1.76 ms) and spans
// of 3 chunks.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/tg_raycast.h"
#include "readout_device.h"

using namespace tg;

namespace {
thread_local std::string g_ray_create_error;
constexpr int RC_STACK = 32;      // deepest tree
constexpr int RC_CHUNKS = 3;      // most chunks of 64 probes in a wave's span
constexpr int RC_QUEUE = 64 * RC_CHUNKS;
constexpr int RC_REFILL = 8;      // free lanes that take new queries
// A span of more than one chunk only from here on, about the waves the chip holds: longer spans keep
// the lanes busy, shorter ones spread a small launch.  200-taxel hands, spans of 1 / 2 / 3 / 4 chunks:
// 3200 chunks 82 / 99 / 111 / 135 us, 6400 117 / 113 / 136 / 135 us, 12800 192 / 160 / 153 / 146 us,
// 204800 2012 / 1459 / 1359 / 1508 us (at 4 the queue's LDS costs waves).
constexpr int RC_WAVES = 4096;


struct RayNode {   // a child entry: an interior record's two children are entries 2 r and 2 r + 1
  float4 lo;   // box min; w: the child's record (interior) or its first triangle (leaf), as int bits
  float4 hi;   // box max; w: 0 (interior) or the leaf's triangle count, as int bits
};
struct RayTri {
  float4 a;    // w: the triangle's index in its mesh, as int bits
  float4 b;
  float4 c;
  float4 n;    // outward unit normal
};

struct RayParams {
  int32_t E, L, T, n_obj;
  const float4* tax_a;      // [T] (x_j, R_j)
  const float4* tax_b;      // [T] (n_j, link id as int bits)
  const RayNode* root;      // [n_obj] root entry of each object
  const RayNode* nodes;     // [2 * records] child entries
  const RayTri* tris;
};

struct RayLaunch {
  const float* link_state;  // [S][13][E*L]
  const float* obj_state;   // [S][13][E] or null
  const int32_t* obj_id;    // [S][E]
  float* depth;             // [S][E][T]
  float* normal;            // [S][3][E][T] or null
  int32_t* tri;             // [S][E][T] or null
  int32_t n_steps, chunks;  // chunks of 64 probes per wave
};

__device__ __forceinline__ float dot3f(float ax, float ay, float az, float bx, float by, float bz) {
  return fmaf(az, bz, fmaf(ay, by, ax * bx));
}
// squared distance from p to the closest point of triangle (a, b, c); face: whether that point
// lies inside the face (not on an edge or vertex).  The Voronoi region of the point (Ericson's
// tests, in his order of precedence) picks the closest point as a + v (b - a) + w (c - a) with
// v = nv / den and w = nw / den; the regions are selected without branches, so the lanes of a
// wave, whose probes fall in different regions, do not diverge, and one reciprocal serves them all.
__device__ float tri_dist2(float px, float py, float pz, const float4& a, const float4& b, const float4& c, bool& face) {
  const float abx = b.x - a.x, aby = b.y - a.y, abz = b.z - a.z;
  const float acx = c.x - a.x, acy = c.y - a.y, acz = c.z - a.z;
  const float apx = px - a.x, apy = py - a.y, apz = pz - a.z;
  const float d1 = dot3f(abx, aby, abz, apx, apy, apz), d2 = dot3f(acx, acy, acz, apx, apy, apz);
  const float bpx = px - b.x, bpy = py - b.y, bpz = pz - b.z;
  const float d3 = dot3f(abx, aby, abz, bpx, bpy, bpz), d4 = dot3f(acx, acy, acz, bpx, bpy, bpz);
  const float cpx = px - c.x, cpy = py - c.y, cpz = pz - c.z;
  const float d5 = dot3f(abx, aby, abz, cpx, cpy, cpz), d6 = dot3f(acx, acy, acz, cpx, cpy, cpz);
  const float vc = d1 * d4 - d3 * d2, vb = d5 * d2 - d1 * d6, va = d3 * d6 - d5 * d4;
  const float e43 = d4 - d3, e56 = d5 - d6;
  // lowest precedence first: the face, then edge bc, edge ac, vertex c, edge ab, vertex b, vertex a
  float nv = vb, nw = vc, den = va + vb + vc;
  bool f = true;
  if (va <= 0.f && e43 >= 0.f && e56 >= 0.f) { nv = e56; nw = e43; den = e43 + e56; f = false; }   // edge bc
  if (vb <= 0.f && d2 >= 0.f && d6 <= 0.f) { nv = 0.f; nw = d2; den = d2 - d6; f = false; }        // edge ac
  if (d6 >= 0.f && d5 <= d6) { nv = 0.f; nw = 1.f; den = 1.f; f = false; }                        // vertex c
  if (vc <= 0.f && d1 >= 0.f && d3 <= 0.f) { nv = d1; nw = 0.f; den = d1 - d3; f = false; }        // edge ab
  if (d3 >= 0.f && d4 <= d3) { nv = 1.f; nw = 0.f; den = 1.f; f = false; }                        // vertex b
  if (d1 <= 0.f && d2 <= 0.f) { nv = 0.f; nw = 0.f; den = 1.f; f = false; }                       // vertex a
  face = f;
  const float inv = __builtin_amdgcn_rcpf(den), v = nv * inv, w = nw * inv;
  const float qx = fmaf(w, acx, fmaf(v, abx, a.x));
  const float qy = fmaf(w, acy, fmaf(v, aby, a.y));
  const float qz = fmaf(w, acz, fmaf(v, abz, a.z));
  const float dx = px - qx, dy = py - qy, dz = pz - qz;
  return dot3f(dx, dy, dz, dx, dy, dz);
}
// ray o + t d against triangle (a, b, c): t > 0 with barycentric slack 1e-6; returns t or +inf
__device__ float tri_ray(float ox, float oy, float oz, float dx, float dy, float dz, const float4& a, const float4& b,
                         const float4& c) {
  const float e1x = b.x - a.x, e1y = b.y - a.y, e1z = b.z - a.z;
  const float e2x = c.x - a.x, e2y = c.y - a.y, e2z = c.z - a.z;
  const float px = fmaf(dy, e2z, -(dz * e2y)), py = fmaf(dz, e2x, -(dx * e2z)), pz = fmaf(dx, e2y, -(dy * e2x));
  const float det = dot3f(e1x, e1y, e1z, px, py, pz);
  if (det == 0.f) return INFINITY;
  const float inv = __builtin_amdgcn_rcpf(det);
  const float tx = ox - a.x, ty = oy - a.y, tz = oz - a.z;
  const float u = dot3f(tx, ty, tz, px, py, pz) * inv;
  if (u < -1e-6f || u > 1.0f + 1e-6f) return INFINITY;
  const float qx = fmaf(ty, e1z, -(tz * e1y)), qy = fmaf(tz, e1x, -(tx * e1z)), qz = fmaf(tx, e1y, -(ty * e1x));
  const float v = dot3f(dx, dy, dz, qx, qy, qz) * inv;
  if (v < -1e-6f || u + v > 1.0f + 1e-6f) return INFINITY;
  const float t = dot3f(e2x, e2y, e2z, qx, qy, qz) * inv;
  return t > 0.f ? t : INFINITY;
}
// a probe's poses and object of one step
struct RayPose {
  float pL[3], RL[9], pO[3], RO[9];
  int oid;
};
__device__ __forceinline__ void load_pose(const RayParams& p, const RayLaunch& q, int s, int e, int l, RayPose& w) {
  const int64_t EL = (int64_t)p.E * p.L;
  const float* ls = q.link_state + (int64_t)s * 13 * EL + (int64_t)e * p.L + l;
  float v[7];
#pragma unroll
  for (int c = 0; c < 7; ++c) v[c] = ls[c * EL];
#pragma unroll
  for (int c = 0; c < 3; ++c) w.pL[c] = v[c];
  quat_to_R(v[3], v[4], v[5], v[6], w.RL);
  const int oid = q.obj_id[(int64_t)s * p.E + e];
  w.oid = oid >= 0 && oid < p.n_obj ? oid : -1;
#pragma unroll
  for (int c = 0; c < 9; ++c) w.RO[c] = c % 4 == 0 ? 1.f : 0.f;
  w.pO[0] = w.pO[1] = w.pO[2] = 0.f;
  if (w.oid >= 0 && q.obj_state) {
    const float* os = q.obj_state + (int64_t)s * 13 * p.E + e;
    w.pO[0] = os[0]; w.pO[1] = os[p.E]; w.pO[2] = os[2 * p.E];
    quat_to_R(os[3 * p.E], os[4 * p.E], os[5 * p.E], os[6 * p.E], w.RO);
  }
}
// squared distance from a point to a child's box
__device__ __forceinline__ float box_d2(const RayNode& c, const float4& x) {
  const float ex = fmaxf(fmaxf(c.lo.x - x.x, x.x - c.hi.x), 0.f);
  const float ey = fmaxf(fmaxf(c.lo.y - x.y, x.y - c.hi.y), 0.f);
  const float ez = fmaxf(fmaxf(c.lo.z - x.z, x.z - c.hi.z), 0.f);
  return dot3f(ex, ey, ez, ex, ey, ez);
}
__device__ __forceinline__ int rank_of(uint64_t bal) {   // the number of lanes below this one in a ballot
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
}

// Walks the trees of `count` queries, a lane a query, each as a state machine: an interior record to
// open (cur), triangles of a leaf to test (tri, ntri), a far child that waits for the near one's
// leaf (far, nfar, kfar), the stack of parked records.  The wave takes the kind of step that more
// lanes wait for, and takes it until no lane does; lanes that are done take the next queries.  Each
// query visits its nodes and triangles in the order in which it would alone: the nearer child (by
// key) first, a far leaf before a near subtree.  take(i) starts query i and returns its root entry's
// tags, keys(c0, c1, k0, k1) are the children's keys, pass(k) whether a child of key k can still
// improve the query, test(t) tests a triangle, done() ends the query.
template <class Take, class Keys, class Pass, class Test, class Done>
__device__ __forceinline__ void walk(const RayParams& p, int* st, int count, Take&& take, Keys&& keys, Pass&& pass,
                                     Test&& test, Done&& done) {
  float kfar = 0.f;
  int cur = -1, tri = 0, ntri = 0, far = 0, nfar = -1, sp = 0, next = 0;
  bool busy = false;
  for (;;) {
    if (ntri == 0 && cur < 0) {
      if (nfar >= 0) {   // (the bound may have shrunk at the near child's leaf)
        if (pass(kfar)) {
          if (nfar > 0) { tri = far; ntri = nfar; }
          else cur = far;
        }
        nfar = -1;
      }
      if (ntri == 0 && cur < 0 && sp > 0) cur = st[--sp * 64];
    }
    const bool idle = ntri == 0 && cur < 0 && sp == 0;
    if (idle && busy) {
      done();
      busy = false;
    }
    const uint64_t free = __ballot(idle);
    if (next < count && (__popcll(free) >= RC_REFILL || free == ~0ull)) {
      const int i = next + rank_of(free);
      if (idle && i < count) {
        const int2 root = take(i);
        busy = true;
        if (root.y > 0) { tri = root.x; ntri = root.y; }
        else cur = root.x;
      }
      next += __popcll(free);
    } else if (free == ~0ull) {
      break;
    }
    const int nleaf = __popcll(__ballot(ntri > 0)), nopen = __popcll(__ballot(ntri == 0 && cur >= 0));
    if (nleaf >= nopen) {
      while (ntri > 0) {
        test(tri);
        ++tri;
        --ntri;
      }
    } else {
      while (ntri == 0 && cur >= 0) {
        const RayNode c0 = p.nodes[2 * cur], c1 = p.nodes[2 * cur + 1];
        float k0, k1;
        keys(c0, c1, k0, k1);
        const bool sw = k1 < k0;
        const float ka = sw ? k1 : k0, kb = sw ? k0 : k1;
        const int wa = __float_as_int(sw ? c1.lo.w : c0.lo.w), na = __float_as_int(sw ? c1.hi.w : c0.hi.w);
        const int wb = __float_as_int(sw ? c0.lo.w : c1.lo.w), nb = __float_as_int(sw ? c0.hi.w : c1.hi.w);
        cur = -1;
        if (pass(ka)) {
          const bool both = pass(kb);
          if (na > 0) {
            tri = wa;
            ntri = na;
            if (both) { far = wb; nfar = nb; kfar = kb; }
          } else {
            cur = wa;
            if (both) {
              if (nb > 0) { tri = wb; ntri = nb; }
              else st[sp++ * 64] = wb;   // the host bounds the depth
            }
          }
        }
      }
    }
  }
}
// writes one probe's outputs
__device__ __forceinline__ void put(const RayParams& p, const RayLaunch& q, int s, int idx, const RayPose& w,
                                    float best, int bt) {
  const int64_t ET = (int64_t)p.E * p.T, o = (int64_t)s * ET + idx;
  q.depth[o] = best;
  float4 n = make_float4(0.f, 0.f, 0.f, 0.f);
  if (bt >= 0) n = p.tris[bt].n;
  if (q.tri) q.tri[o] = bt >= 0 ? __float_as_int(p.tris[bt].a.w) : -1;
  if (q.normal) {
    float nl[3] = {0.f, 0.f, 0.f};
    if (bt >= 0) {
      float nw[3];
      mat_vec(w.RO, n.x, n.y, n.z, nw);
      mat_T_vec(w.RL, nw[0], nw[1], nw[2], nl);
    }
    float* nm = q.normal + (int64_t)s * 3 * ET + idx;
    nm[0] = nl[0];
    nm[ET] = nl[1];
    nm[2 * ET] = nl[2];
  }
}
}  // namespace

__global__ __launch_bounds__(64, 6) void tg_ray_kernel(const RayParams p, const RayLaunch q) {
  __shared__ float4 qa[RC_QUEUE];         // the probe's centre in the object frame; R, then the sphere's penetration
  __shared__ float4 qb[RC_QUEUE];         // its root's tags; the sphere's result; the ray's direction and triangle
  __shared__ uint8_t item[RC_QUEUE];      // its place in the wave's span
  extern __shared__ int stk[];            // [depth][64] parked records
  const int lane = threadIdx.x;
  const int ET = p.E * p.T;
  const int span0 = (int)blockIdx.x * q.chunks * 64;
  int* const st = stk + lane;
  for (int s = blockIdx.y; s < q.n_steps; s += gridDim.y) {
    int count = 0;
    for (int k = 0; k < q.chunks; ++k) {
      if (span0 + 64 * k >= ET) break;   // uniform
      const int idx = span0 + 64 * k + lane;
      // 1. the probe's centre; a probe that its object's box does not reach is done
      float4 x4 = make_float4(0.f, 0.f, 0.f, 0.f);
      int2 root = make_int2(0, 0);
      bool in = false;
      if (idx < ET) {
        const int e = idx / p.T, j = idx - e * p.T;
        const float4 ta = p.tax_a[j];
        RayPose w;
        load_pose(p, q, s, e, __float_as_int(p.tax_b[j].w), w);
        if (w.oid >= 0 && ta.w > 0.f) {
          float x[3], qo[3];
          mat_vec(w.RL, ta.x, ta.y, ta.z, x);
          mat_T_vec(w.RO, (w.pL[0] + x[0]) - w.pO[0], (w.pL[1] + x[1]) - w.pO[1], (w.pL[2] + x[2]) - w.pO[2], qo);
          x4 = make_float4(qo[0], qo[1], qo[2], ta.w);
          const RayNode rt = p.root[w.oid];
          root = make_int2(__float_as_int(rt.lo.w), __float_as_int(rt.hi.w));
          // (a centre in the box may need the ray, also where the square of its radius is 0 in FP32)
          const float d2 = box_d2(rt, x4);
          in = d2 < ta.w * ta.w || d2 == 0.f;
        }
        if (!in) put(p, q, s, idx, w, 0.f, -1);
      }
      const uint64_t bal = __ballot(in);
      if (in) {
        const int slot = count + rank_of(bal);
        qa[slot] = x4;
        qb[slot].x = __int_as_float(root.x);
        qb[slot].y = __int_as_float(root.y);
        item[slot] = (uint8_t)(64 * k + lane);
      }
      count += __popcll(bal);
    }
    __syncthreads();

    // 2. sphere queries: children closer than R - best, nearer box first
    {
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      float best = 0.f, lim = 0.f;
      int bt = -1, slot = 0;
      bool bface = false;
      walk(p, st, count,
           [&](int i) {
             slot = i;
             x = qa[i];
             best = 0.f;
             lim = x.w;
             bt = -1;
             bface = false;
             return make_int2(__float_as_int(qb[i].x), __float_as_int(qb[i].y));
           },
           [&](const RayNode& c0, const RayNode& c1, float& k0, float& k1) {
             k0 = box_d2(c0, x);
             k1 = box_d2(c1, x);
           },
           [&](float k) { return k < lim * lim; },
           [&](int t) {
             const RayTri tr = p.tris[t];
             bool face;
             const float d2 = tri_dist2(x.x, x.y, x.z, tr.a, tr.b, tr.c, face);
             if (d2 < lim * lim) {   // (the square root only for a deeper triangle)
               const float pen = x.w - sqrtf(d2);
               if (pen > best) {
                 best = pen;
                 bt = t;
                 bface = face;
                 lim = x.w - best;
               }
             }
           },
           [&]() {
             qb[slot].x = bface ? -best : best;   // (a penetration on a face is positive)
             qb[slot].y = __int_as_float(bt);
           });
    }
    __syncthreads();

    // 3. the ray query along -a can only count when the centre is inside the mesh, so it is
    //    skipped when the centre is outside the object's box, or when its closest point lies
    //    inside a face and the centre is on that face's outer side (then the ray's first crossing
    //    enters the mesh).  Near the surface, where rounding could flip that side, the two tests
    //    agree to twice the centre's distance from the face.  The probes that need one move to the
    //    front of the queue.
    int rays = 0;
    for (int i0 = 0; i0 < count; i0 += 64) {
      const int i = i0 + lane;
      bool need = false;
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f), d = x;
      int it = 0;
      if (i < count) {
        it = item[i];
        const int idx = span0 + it, e = idx / p.T;
        const float4 tb = p.tax_b[idx - e * p.T];
        RayPose w;
        load_pose(p, q, s, e, __float_as_int(tb.w), w);
        x = qa[i];
        const float res = qb[i].x;
        const int bt = __float_as_int(qb[i].y);
        const RayNode rt = p.root[w.oid];
        need = x.x >= rt.lo.x && x.x <= rt.hi.x && x.y >= rt.lo.y && x.y <= rt.hi.y && x.z >= rt.lo.z && x.z <= rt.hi.z;
        if (need && bt >= 0 && res < 0.f) {
          const RayTri tr = p.tris[bt];
          need = !(dot3f(x.x - tr.a.x, x.y - tr.a.y, x.z - tr.a.z, tr.n.x, tr.n.y, tr.n.z) > 0.f);
        }
        if (need) {
          float a[3], ao[3];
          mat_vec(w.RL, tb.x, tb.y, tb.z, a);
          mat_T_vec(w.RO, a[0], a[1], a[2], ao);
          x.w = fabsf(res);
          d = make_float4(-ao[0], -ao[1], -ao[2], __int_as_float(bt));
        } else {
          put(p, q, s, idx, w, fabsf(res), bt);
        }
      }
      __syncthreads();
      const uint64_t bal = __ballot(need);
      if (need) {
        const int slot = rays + rank_of(bal);   // (at most i: every lane has read its own)
        qa[slot] = x;
        qb[slot] = d;
        item[slot] = (uint8_t)it;
      }
      rays += __popcll(bal);
    }
    __syncthreads();
    //    children the ray enters before the nearest hit so far, nearer entry first
    {
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      float dx = 0.f, dy = 0.f, dz = 0.f, ix = 0.f, iy = 0.f, iz = 0.f, tmin = INFINITY;
      int th = -1, slot = 0;
      // entry parameter of the ray into a box, or +inf when it misses it
      auto box_t = [&](const RayNode& c) {
        const float t1x = (c.lo.x - x.x) * ix, t2x = (c.hi.x - x.x) * ix;
        const float t1y = (c.lo.y - x.y) * iy, t2y = (c.hi.y - x.y) * iy;
        const float t1z = (c.lo.z - x.z) * iz, t2z = (c.hi.z - x.z) * iz;
        const float tn = fmaxf(fmaxf(fminf(t1x, t2x), fminf(t1y, t2y)), fmaxf(fminf(t1z, t2z), 0.f));
        const float tf = fminf(fminf(fmaxf(t1x, t2x), fmaxf(t1y, t2y)), fminf(fmaxf(t1z, t2z), tmin));
        return tn <= tf ? tn : INFINITY;
      };
      walk(p, st, rays,
           [&](int i) {
             slot = i;
             x = qa[i];
             dx = qb[i].x;
             dy = qb[i].y;
             dz = qb[i].z;
             ix = 1.0f / dx;
             iy = 1.0f / dy;
             iz = 1.0f / dz;
             tmin = INFINITY;
             th = -1;
             const int e = (span0 + item[i]) / p.T;
             const RayNode rt = p.root[q.obj_id[(int64_t)s * p.E + e]];
             int2 root = make_int2(__float_as_int(rt.lo.w), __float_as_int(rt.hi.w));
             if (!(box_t(rt) < INFINITY)) root = make_int2(-1, 0);
             return root;
           },
           [&](const RayNode& c0, const RayNode& c1, float& k0, float& k1) {
             k0 = box_t(c0);
             k1 = box_t(c1);
           },
           [&](float k) { return k <= tmin && k < INFINITY; },
           [&](int t) {
             const RayTri tr = p.tris[t];
             const float tt = tri_ray(x.x, x.y, x.z, dx, dy, dz, tr.a, tr.b, tr.c);
             if (tt < tmin) {
               tmin = tt;
               th = t;
             }
           },
           [&]() {   // a hit that leaves the mesh
             bool out = false;
             if (th >= 0) {
               const float4 n = p.tris[th].n;
               out = dot3f(dx, dy, dz, n.x, n.y, n.z) > 0.f;
             }
             qb[slot].x = out ? tmin : -1.f;
             qb[slot].y = __int_as_float(th);
           });
    }
    __syncthreads();
    for (int i = lane; i < rays; i += 64) {
      const int idx = span0 + item[i], e = idx / p.T, j = idx - e * p.T;
      RayPose w;
      load_pose(p, q, s, e, __float_as_int(p.tax_b[j].w), w);
      const float4 b = qb[i];
      const float R = p.tax_a[j].w;
      float best = qa[i].w;
      int bt = __float_as_int(b.w);
      if (b.x >= 0.f && R + b.x > best) {
        best = R + b.x;
        bt = __float_as_int(b.y);
      }
      put(p, q, s, idx, w, best, bt);
    }
    __syncthreads();
  }
}

struct tg_ray {
  RayParams p{};
  int depth = 1;   // of the deepest tree: a walk parks at most one record a level
  std::vector<void*> allocs;
  std::string err;
};

namespace {
tg_status rfail(tg_ray* h, tg_status s, const std::string& msg) {
  if (h) h->err = msg; else g_ray_create_error = msg;
  return s;
}
template <class T>
hipError_t ralloc(tg_ray* h, T** ptr, size_t n) {
  void* q = nullptr;
  const hipError_t e = hipMalloc(&q, std::max<size_t>(n, 1) * sizeof(T));
  if (e == hipSuccess) h->allocs.push_back(q);
  *ptr = (T*)q;
  return e;
}
bool aligned16(const void* ptr) { return ((uintptr_t)ptr & 15u) == 0; }
float ibits(int v) {   // an int's bits as a float (the node and triangle tags)
  float f;
  std::memcpy(&f, &v, 4);
  return f;
}

// Median-split BVH over one mesh's triangles, appended to nodes / tris (depth first).
struct Builder {
  const float* V;
  const int32_t* F;
  std::vector<int> idx;
  std::vector<double> cen;   // [m][3]
  std::vector<RayNode>* nodes;
  std::vector<RayTri>* tris;
  int max_depth = 0;
  void box(int b, int e, double lo[3], double hi[3]) const {
    for (int k = 0; k < 3; ++k) { lo[k] = INFINITY; hi[k] = -INFINITY; }
    for (int i = b; i < e; ++i)
      for (int c = 0; c < 3; ++c)
        for (int k = 0; k < 3; ++k) {
          const double x = V[3 * F[3 * idx[i] + c] + k];
          lo[k] = std::min(lo[k], x);
          hi[k] = std::max(hi[k], x);
        }
  }
  // Returns the entry of the subtree over idx[b, e): its box and either its record (appended to
  // nodes as two child entries) or its leaf's triangles (appended to tris).
  RayNode build(int b, int e, int depth) {
    max_depth = std::max(max_depth, depth);
    RayNode me;
    double lo[3], hi[3];
    box(b, e, lo, hi);
    float flo[3], fhi[3];
    for (int k = 0; k < 3; ++k) {   // grown so FP32 rounding never culls a triangle
      const double g = 1e-6 * std::max(1.0, std::fabs(lo[k]) + std::fabs(hi[k])) + 1e-6 * (hi[k] - lo[k]);
      flo[k] = (float)(lo[k] - g);
      fhi[k] = (float)(hi[k] + g);
    }
    if (e - b <= 4) {
      const int first = (int)tris->size();
      for (int i = b; i < e; ++i) {
        const int t = idx[i];
        double P[3][3];
        for (int c = 0; c < 3; ++c)
          for (int k = 0; k < 3; ++k) P[c][k] = V[3 * F[3 * t + c] + k];
        double e1[3], e2[3], n[3];
        for (int k = 0; k < 3; ++k) { e1[k] = P[1][k] - P[0][k]; e2[k] = P[2][k] - P[0][k]; }
        n[0] = e1[1] * e2[2] - e1[2] * e2[1];
        n[1] = e1[2] * e2[0] - e1[0] * e2[2];
        n[2] = e1[0] * e2[1] - e1[1] * e2[0];
        const double ln = std::sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
        RayTri tr;
        tr.a = make_float4((float)P[0][0], (float)P[0][1], (float)P[0][2], ibits(t));
        tr.b = make_float4((float)P[1][0], (float)P[1][1], (float)P[1][2], 0.f);
        tr.c = make_float4((float)P[2][0], (float)P[2][1], (float)P[2][2], 0.f);
        tr.n = make_float4((float)(n[0] / ln), (float)(n[1] / ln), (float)(n[2] / ln), 0.f);
        tris->push_back(tr);
      }
      me.lo = make_float4(flo[0], flo[1], flo[2], ibits(first));
      me.hi = make_float4(fhi[0], fhi[1], fhi[2], ibits(e - b));
      return me;
    }
    double clo[3] = {INFINITY, INFINITY, INFINITY}, chi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int i = b; i < e; ++i)
      for (int k = 0; k < 3; ++k) {
        clo[k] = std::min(clo[k], cen[3 * idx[i] + k]);
        chi[k] = std::max(chi[k], cen[3 * idx[i] + k]);
      }
    int ax = 0;
    for (int k = 1; k < 3; ++k)
      if (chi[k] - clo[k] > chi[ax] - clo[ax]) ax = k;
    const int mid = (b + e) / 2;
    std::nth_element(idx.begin() + b, idx.begin() + mid, idx.begin() + e, [&](int u, int w) {
      return cen[3 * u + ax] < cen[3 * w + ax] || (cen[3 * u + ax] == cen[3 * w + ax] && u < w);
    });
    const int rec = (int)(nodes->size() / 2);
    nodes->push_back(RayNode{});
    nodes->push_back(RayNode{});
    const RayNode left = build(b, mid, depth + 1);
    const RayNode right = build(mid, e, depth + 1);
    (*nodes)[2 * (size_t)rec] = left;
    (*nodes)[2 * (size_t)rec + 1] = right;
    me.lo = make_float4(flo[0], flo[1], flo[2], ibits(rec));
    me.hi = make_float4(fhi[0], fhi[1], fhi[2], ibits(0));
    return me;
  }
};
}  // namespace

extern "C" {

tg_status tg_ray_create(const tg_ray_config* cfg, tg_ray** out) {
  if (!out) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "out is NULL");
  *out = nullptr;
  if (!cfg) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "cfg is NULL");
  if (cfg->abi_version != TG_ABI_VERSION) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "abi_version mismatch");
  const int E = cfg->num_envs, L = cfg->num_links, T = cfg->num_taxels, NO = cfg->num_objects;
  if (E < 1 || L < 1 || T < 1 || NO < 1) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "sizes must be positive");
  if (!cfg->link_taxel_offset || !cfg->taxel_pos || !cfg->taxel_normal || !cfg->taxel_radius || !cfg->meshes)
    return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "NULL array");
  if ((int64_t)E * T * 3 >= (int64_t(1) << 31)) return rfail(nullptr, TG_ERR_UNSUPPORTED, "E * T * 3 exceeds 2^31");
  const int32_t* off = cfg->link_taxel_offset;
  if (off[0] != 0 || off[L] != T) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "link offsets must run 0..T");
  std::vector<float4> ta(T), tb(T);
  for (int l = 0; l < L; ++l) {
    if (off[l + 1] < off[l]) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "link offsets decrease");
    for (int j = off[l]; j < off[l + 1]; ++j) {
      const float r = cfg->taxel_radius[j];
      if (!(r >= 0.f) || !std::isfinite(r)) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "invalid probe radius");
      ta[j] = make_float4(cfg->taxel_pos[3 * j], cfg->taxel_pos[3 * j + 1], cfg->taxel_pos[3 * j + 2], r);
      tb[j] = make_float4(cfg->taxel_normal[3 * j], cfg->taxel_normal[3 * j + 1], cfg->taxel_normal[3 * j + 2],
                          ibits(l));
    }
  }
  std::vector<RayNode> nodes;
  std::vector<RayTri> tris;
  std::vector<RayNode> roots(NO);
  int depth = 1;
  for (int o = 0; o < NO; ++o) {
    const tg_mesh& m = cfg->meshes[o];
    if (m.num_verts < 3 || m.num_tris < 1 || !m.verts || !m.tris)
      return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "mesh " + std::to_string(o) + " invalid");
    if (m.num_tris > (1 << 20)) return rfail(nullptr, TG_ERR_UNSUPPORTED, "mesh of more than 2^20 triangles");
    for (int i = 0; i < 3 * m.num_verts; ++i)
      if (!std::isfinite(m.verts[i])) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "non-finite vertex");
    Builder bd;
    bd.V = m.verts;
    bd.F = m.tris;
    bd.nodes = &nodes;
    bd.tris = &tris;
    bd.idx.resize(m.num_tris);
    std::iota(bd.idx.begin(), bd.idx.end(), 0);
    bd.cen.resize(3 * (size_t)m.num_tris);
    for (int t = 0; t < m.num_tris; ++t) {
      double P[3][3];
      for (int c = 0; c < 3; ++c) {
        const int vi = m.tris[3 * t + c];
        if (vi < 0 || vi >= m.num_verts) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "vertex index out of range");
        for (int k = 0; k < 3; ++k) P[c][k] = m.verts[3 * vi + k];
      }
      double e1[3], e2[3];
      for (int k = 0; k < 3; ++k) { e1[k] = P[1][k] - P[0][k]; e2[k] = P[2][k] - P[0][k]; }
      const double nx = e1[1] * e2[2] - e1[2] * e2[1], ny = e1[2] * e2[0] - e1[0] * e2[2], nz = e1[0] * e2[1] - e1[1] * e2[0];
      if (!(nx * nx + ny * ny + nz * nz > 0.0)) return rfail(nullptr, TG_ERR_INVALID_ARGUMENT, "degenerate triangle");
      for (int k = 0; k < 3; ++k) bd.cen[3 * t + k] = (P[0][k] + P[1][k] + P[2][k]) / 3.0;
    }
    roots[o] = bd.build(0, m.num_tris, 0);
    if (bd.max_depth + 2 > RC_STACK) return rfail(nullptr, TG_ERR_UNSUPPORTED, "BVH deeper than the traversal stack");
    depth = std::max(depth, bd.max_depth);
  }
  tg_ray* h = new (std::nothrow) tg_ray();
  if (!h) return rfail(nullptr, TG_ERR_OUT_OF_MEMORY, "host allocation failed");
  h->depth = depth;
  RayParams& p = h->p;
  p.E = E; p.L = L; p.T = T; p.n_obj = NO;
  float4 *dta = nullptr, *dtb = nullptr;
  RayNode* droot = nullptr;
  RayNode* dn = nullptr;
  RayTri* dt = nullptr;
  hipError_t e = ralloc(h, &dta, T);
  if (e == hipSuccess) e = ralloc(h, &dtb, T);
  if (e == hipSuccess) e = ralloc(h, &droot, NO);
  if (e == hipSuccess) e = ralloc(h, &dn, nodes.size());
  if (e == hipSuccess) e = ralloc(h, &dt, tris.size());
  if (e == hipSuccess) e = hipMemcpy(dta, ta.data(), T * sizeof(float4), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(dtb, tb.data(), T * sizeof(float4), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(droot, roots.data(), NO * sizeof(RayNode), hipMemcpyHostToDevice);
  if (e == hipSuccess && !nodes.empty())
    e = hipMemcpy(dn, nodes.data(), nodes.size() * sizeof(RayNode), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(dt, tris.data(), tris.size() * sizeof(RayTri), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    tg_ray_destroy(h);
    return rfail(nullptr, TG_ERR_OUT_OF_MEMORY, std::string("device setup: ") + hipGetErrorString(e));
  }
  p.tax_a = dta; p.tax_b = dtb; p.root = droot; p.nodes = dn; p.tris = dt;
  *out = h;
  return TG_OK;
}

tg_status tg_ray_rollout(tg_ray* h, const tg_step_inputs* in, float* depth, float* normal, int32_t* tri,
                         int32_t n_steps, void* hip_stream) {
  if (!h) return TG_ERR_INVALID_ARGUMENT;
  h->err.clear();
  if (!in || !depth) return rfail(h, TG_ERR_INVALID_ARGUMENT, "inputs or depth is NULL");
  if (n_steps < 0) return rfail(h, TG_ERR_INVALID_ARGUMENT, "n_steps < 0");
  if (n_steps == 0) return TG_OK;
  if (!in->link_state || !in->obj_id) return rfail(h, TG_ERR_INVALID_ARGUMENT, "link_state and obj_id are required");
  if (!aligned16(in->link_state) || !aligned16(in->obj_id) || (in->obj_state && !aligned16(in->obj_state)) ||
      !aligned16(depth) || (normal && !aligned16(normal)) || (tri && !aligned16(tri)))
    return rfail(h, TG_ERR_INVALID_ARGUMENT, "pointers must be 16-byte aligned");
  RayLaunch q{};
  q.link_state = in->link_state;
  q.obj_state = in->obj_state;
  q.obj_id = in->obj_id;
  q.depth = depth;
  q.normal = normal;
  q.tri = tri;
  q.n_steps = n_steps;
  const int64_t chunks = ((int64_t)h->p.E * h->p.T + 63) / 64, rows = std::min(n_steps, 65535);
  q.chunks = (int)std::min<int64_t>(RC_CHUNKS, std::max<int64_t>(1, chunks * rows / RC_WAVES));
  const dim3 grid((unsigned)((chunks + q.chunks - 1) / q.chunks), (unsigned)rows);
  hipLaunchKernelGGL(tg_ray_kernel, grid, dim3(64), h->depth * 64 * sizeof(int), (hipStream_t)hip_stream, h->p, q);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? TG_OK : rfail(h, TG_ERR_HIP, hipGetErrorString(e));
}

tg_status tg_ray_destroy(tg_ray* h) {
  if (!h) return TG_OK;
  for (void* ptr : h->allocs) (void)hipFree(ptr);
  delete h;
  return TG_OK;
}

const char* tg_ray_last_error(const tg_ray* h) { return h ? h->err.c_str() : g_ray_create_error.c_str(); }

}  // extern "C"
