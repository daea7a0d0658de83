// pmbs_kernels.hip -- CDNA4 (gfx950) kernels of the batched push transition.
//
// One 64-lane wavefront (or two) advances one environment (cuboids on a plane
// plus a kinematic box pusher) through a push: the batch expansion /
// simulation of PMBS (Sec. IV-C), with the transition of Sec. III-A made
// explicit.
//
// Lane roles inside the lead wave: four lanes per body in the 16-box layout,
// two in the 31-box layout, all holding the body's whole state and together
// its first four table contacts; every other contact is a row contact, one
// per four lanes or, of more than 16, one per lane and slot.  Shared state goes
// through LDS: body frames, AABBs, the pair list, the row contacts' staging
// array (reused for the impulse exchange of the solver), per-body incidence
// lists, warm-start keys and impulses, and the clip polygons of face clipping.
//
// Per substep (all in one launch, the state in registers and LDS, read from HBM
// once and written once per call; the kernel at three waves per SIMD spills
// registers, which leave the L2: see step_kernel):
//   velocity stage -> frames -> AABB broadphase -> box-plane and
//   box-box/pusher-box contacts (15-axis SAT, Sutherland-Hodgman face
//   clipping or edge-edge closest points) -> contact prep (mass splitting,
//   Tonge et al. 2012) -> I projected-Jacobi iterations (normal clamp, then
//   circular friction cone; per-body sums in contact-index order) ->
//   symplectic position stage.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "pmbs_kernels.h"

namespace pmbs {

constexpr int MAXB = 32;             // boxes (<= 31) + the pusher
constexpr int POLY = 8;              // clip polygon capacity
// Growth of the AABBs of the broadphase's near list (m).  More lengthens the
// list, less has it listed anew more often: 700 x 27 1.39 to 1.40 ms with 3 mm,
// 1.38 with 6 and with 12, where more environments have more than one pass.
constexpr float SKIN = 0.006f;

// ------------------------------------------------------------------ vectors
struct f3 { float x, y, z; };
__device__ __forceinline__ f3 mk(float x, float y, float z) { return {x, y, z}; }
__device__ __forceinline__ f3 operator+(f3 a, f3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ f3 operator-(f3 a, f3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ f3 operator*(f3 a, float s) { return {a.x * s, a.y * s, a.z * s}; }
__device__ __forceinline__ f3 neg(f3 a) { return {-a.x, -a.y, -a.z}; }
__device__ __forceinline__ f3 sel(bool c, f3 a, f3 b) { return {c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z}; }
__device__ __forceinline__ float dot(f3 a, f3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ f3 cross(f3 a, f3 b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
// Fused forms.  The library is built with contraction limited to single
// source expressions, so every multiply-add that should be fused across a
// helper call is written here; the rounding of each result is then fixed by
// the source alone (the same in every kernel instantiation).
// a * s + c per component
__device__ __forceinline__ f3 fma3(f3 a, float s, f3 c) { return {fmaf(a.x, s, c.x), fmaf(a.y, s, c.y), fmaf(a.z, s, c.z)}; }
// c + a x b
__device__ __forceinline__ f3 cross_add(f3 a, f3 b, f3 c) {
  return {fmaf(a.y, b.z, fmaf(-a.z, b.y, c.x)), fmaf(a.z, b.x, fmaf(-a.x, b.z, c.y)),
          fmaf(a.x, b.y, fmaf(-a.y, b.x, c.z))};
}
// xyz of a float4 slot (the w lane is never read)
__device__ __forceinline__ void st3(float4* d, f3 v) {
  d->x = v.x;
  d->y = v.y;
  d->z = v.z;
}
__device__ __forceinline__ float sel(bool c, float a, float b) { return c ? a : b; }
__device__ __forceinline__ f3 xyz(float4 v) { return {v.x, v.y, v.z}; }
__device__ __forceinline__ float4 f4(f3 v, float w) { return make_float4(v.x, v.y, v.z, w); }

// ------------------------------------------------------------------ wave helpers
// Exclusive prefix sum across the wave, and its total: an inclusive scan by
// DPP row shifts (by 1, 2 and 3, then by 4 and 8 into the upper banks of
// each 16-lane row) and broadcasts of lanes 15 and 31 into the following
// rows; no LDS and no ballots.
__device__ __forceinline__ int wave_excl_scan(int x, int* total) {
  int v = x;
  v += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, x, 0x113, 0xf, 0xf, true);   // row_shr:3
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xe, true);   // row_shr:4, lanes 4-15
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xc, true);   // row_shr:8, lanes 8-15
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15, rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31, rows 2 and 3
  *total = __builtin_amdgcn_readlane(v, 63);
  return v - x;
}

// An opaque copy of a value: address arithmetic built from it stays where it
// is used (otherwise one 64-bit row offset per state row is computed at the
// start, shared by every later load and store of the rows, and held in
// registers, or scratch, for the whole kernel).
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The compiler has a value here, before and after other side effects as written.
__device__ __forceinline__ void hold(f3& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z)); }

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ f3 uniform(f3 v) { return mk(uniform(v.x), uniform(v.y), uniform(v.z)); }

// Orders the LDS accesses of one wave's lanes around this point (of two waves:
// sync_all).  A wave's LDS operations are performed in issue order, so a
// wavefront-scope fence (no wait instruction) plus a code-motion barrier
// suffices; no wait for outstanding LDS operations.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------ LDS layout
// Hardware reciprocal and reciprocal square root (about 1 ulp), used where
// a correctly rounded divide or square root would cost ten instructions.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

// NB: box capacity of the layout, 16 or 31 (NB 32 leaves one object for the
// pusher).
template <int K, int W, int NB>
struct Smem {
  static constexpr int C = 64 * K;
  static constexpr int MB = NB == 16 ? 17 : 32;   // boxes + the pusher
  static constexpr int PLANE = MB;                // LDS index of the table
  static constexpr int NOBJ = MB + 1;
  static constexpr int MAX_PAIRS = MB * (MB - 1) / 2;
  float4 pos[NOBJ];                  // centre, how far the body has moved in the push
  float4 col[3][NOBJ];               // rotation columns (body axes in world)
  float4 half[NOBJ];                 // hx, hy, hz, inverse mass
  float4 quat[MB];                   // orientation (the lanes' copy between the stages that use it)
  float4 iwa[NOBJ];                  // world inverse inertia xx, yy, zz, xy
  float4 iwb[NOBJ];                  // xz, yz, mu, -
  float4 vel[NOBJ];                  // solver snapshot: linear
  float4 ang[NOBJ];                  // solver snapshot: angular
  int cnt[NOBJ];                     // contacts touching each body (mass splitting)
  // Per-body incidence lists of the row contacts: contact index * 16 | side
  // (1 = b), in contact-index order.
  unsigned short inc[2 * C];
  int lstart[MB];                    // incidence list starts
  unsigned short pairs[MAX_PAIRS];   // candidate pairs
  float apart[(MAX_PAIRS + 63) / 64 * 64];   // pair number p's boxes stay apart while they have moved less than this
  // 31-box layout: the pairs whose AABBs, grown by SKIN, overlapped when they
  // were last listed, and those grown AABBs
  static constexpr bool KEEP = NB != 16;
  unsigned short near[KEEP ? MAX_PAIRS : 1];
  float4 glo[KEEP ? MB : 1], ghi[KEEP ? MB : 1];
  int cab[C];                        // packed a | b << 8 | feature << 16 of each row contact
  int wkey[C];                       // previous substep's row-contact keys (sorted)
  float wl[3][C];                    // and their accumulated impulses (n, t1, t2)
  union {
    struct {
      float4 stage[C][2];            // narrowphase output: (p, sep), (n, -)
      union alignas(16) {
        struct {
          float4 lo[MB], hi[MB];     // AABBs: min corner and pos's fourth, max corner
        } box;
        float clip[W][2][POLY][3][8];   // each wave's clip polygons, of up to eight pairs
        unsigned incm[NOBJ][2 * K];  // incidence build: contact bit masks per body
        float4 lam[MB * 4];          // table impulses (n, t1, t2) and corner mask of a changed corner set
      } x;
    } n;
    float4 imp[3][C];                // solver exchange: P, ra x P, rb x P
  } u;
  float4 zero;                       // a row of zeros after the impulse rows (never written)
  // counts the waves of an environment exchange: candidate pairs, table
  // contacts (all, those held by the body lanes, those staged as rows), and
  // each wave's kept contacts of a narrowphase round (by the round's parity)
  int sh_pairs, sh_table, sh_held, sh_extra;
  int sh_near;                       // (two waves) list the near pairs again
  int rcount[2][W];
};

// Contact key (a+1, b, feature) with the table as a = -1: strictly
// increasing along the contact list, so the previous list is searchable.
template <class S>
__device__ __forceinline__ int contact_key(int ab) {
  const int a = ab & 255, b = (ab >> 8) & 255, f = ab >> 16;
  return ((a == S::PLANE ? 0 : a + 1) << 16) | (b << 8) | f;
}

// ------------------------------------------------------------------ geometry
struct Box {
  f3 c, a0, a1, a2, h;
};

// per-component selects (no indexing into a struct copy) keep the boxes in
// registers when k varies across lanes
__device__ __forceinline__ f3 axis(const Box& b, int k) { return sel(k == 0, b.a0, sel(k == 1, b.a1, b.a2)); }
__device__ __forceinline__ float hcomp(const Box& b, int k) { return sel(k == 0, b.h.x, sel(k == 1, b.h.y, b.h.z)); }

template <class S>
__device__ __forceinline__ Box load_box(const S& s, int i) {
  Box b;
  b.c = xyz(s.pos[i]);
  b.a0 = xyz(s.col[0][i]);
  b.a1 = xyz(s.col[1][i]);
  b.a2 = xyz(s.col[2][i]);
  b.h = xyz(s.half[i]);
  return b;
}

__device__ __forceinline__ float radius_along(const Box& b, f3 L) {
  return b.h.x * fabsf(dot(b.a0, L)) + b.h.y * fabsf(dot(b.a1, L)) + b.h.z * fabsf(dot(b.a2, L));
}

// s(L) = |d.L| - r_A(L) - r_B(L) for a candidate axis L, d = B.c - A.c: the
// boxes' gap along L.
__device__ __forceinline__ float gap_along(const Box& A, const Box& B, f3 d, f3 L) {
  return fabsf(dot(d, L)) - radius_along(A, L) - radius_along(B, L);
}

// Whether an edge axis (a x b with |a x b| >= eps) has s > 0.
__device__ __forceinline__ bool edges_clear(const Box& A, const Box& B, float eps) {
  const f3 d = B.c - A.c;
  float best = -INFINITY;
#pragma unroll 1
  for (int idx = 0; idx < 9; ++idx) {
    const f3 v = cross(axis(A, idx / 3), axis(B, idx % 3));
    const float len = sqrtf(dot(v, v));
    if (len < eps) continue;
    best = fmaxf(best, gap_along(A, B, d, v * (1.0f / len)));
  }
  return best > 0.0f;
}

// Whether the separating-axis test keeps boxes A and B apart: the maximum
// of s(L) over the candidate axes (faces of A, faces of B, edge crosses with
// |a x b| >= eps) is > 0, that is, any of them is.  The face axes come first
// and the edge axes are skipped once a face axis has s > 0.  Every start-pose
// test makes this decision from gap_along and edges_clear.
__device__ __forceinline__ bool sat_clear(const Box& A, const Box& B, float eps) {
  const f3 d = B.c - A.c;
  float best = -INFINITY;
#pragma unroll
  for (int idx = 0; idx < 6; ++idx) best = fmaxf(best, gap_along(A, B, d, idx < 3 ? axis(A, idx) : axis(B, idx - 3)));
  return best > 0.0f || edges_clear(A, B, eps);
}

// The contour push a = obj * n_dirs + dir (Sec. IV-B): direction dir of
// n_dirs around object obj in its yaw frame, starting beyond the
// footprint's ray-to-boundary distance by the pusher half width plus the
// standoff, moving push_length toward the object centre; (x_s, y_s, x_e, y_e).
template <class S>
__device__ __forceinline__ float4 contour_start(const S& s, int obj, int dir, const Params& p) {
  const f3 oc = xyz(s.pos[obj]), oa0 = xyz(s.col[0][obj]), oh = xyz(s.half[obj]);
  const float th = 6.283185307179586f * (float)dir / (float)p.n_dirs;
  const float cth = cosf(th), sth = sinf(th);
  const float rx = fabsf(cth) > 0.0f ? oh.x / fabsf(cth) : INFINITY;
  const float ry = fabsf(sth) > 0.0f ? oh.y / fabsf(sth) : INFINITY;
  const float ray = fminf(rx, ry);
  const float yaw = atan2f(oa0.y, oa0.x);
  const float cy = cosf(yaw), sy = sinf(yaw);
  const float ddx = cy * cth - sy * sth, ddy = sy * cth + cy * sth;
  const float off = ray + p.phx + p.push_standoff;
  const float sxp = oc.x + off * ddx, syp = oc.y + off * ddy;
  return make_float4(sxp, syp, sxp - p.push_length * ddx, syp - p.push_length * ddy);
}

// The pusher of a push: unit direction, moving substeps, start centre and
// its first two rotation columns (yaw along the push).
struct PusherPose {
  f3 dir, x, c0, c1;
  int n_move;
};
__device__ __forceinline__ PusherPose pusher_pose(float4 push, const Params& p) {
  PusherPose r;
  r.dir = mk(1, 0, 0);
  const float dx = push.z - push.x, dy = push.w - push.y;
  const float len = sqrtf(dx * dx + dy * dy);
  if (len > 0.0f) r.dir = mk(dx / len, dy / len, 0.0f);
  r.n_move = (int)roundf(len / (p.push_speed * p.dt));
  r.x = mk(push.x, push.y, p.pusher_z);
  const float yaw = atan2f(r.dir.y, r.dir.x);
  const float cy = cosf(0.5f * yaw), sy = sinf(0.5f * yaw);
  // rotation about z from the half-angle quaternion (cy, 0, 0, sy)
  r.c0 = mk(1.0f - 2.0f * sy * sy, 2.0f * cy * sy, 0.0f);
  r.c1 = mk(-2.0f * cy * sy, 1.0f - 2.0f * sy * sy, 0.0f);
  return r;
}

__device__ __forceinline__ Box pusher_box(const PusherPose& q, const Params& p) {
  Box b;
  b.c = q.x;
  b.a0 = q.c0;
  b.a1 = q.c1;
  b.a2 = mk(0, 0, 1);
  b.h = mk(p.phx, p.phy, p.phz);
  return b;
}

// A DPP move of a value; of a quad permutation, lane i of each four takes lane
// (CTRL >> 2 i) & 3 of them.
template <int CTRL>
__device__ __forceinline__ float quad(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ f3 quad(f3 v) {
  return mk(quad<CTRL>(v.x), quad<CTRL>(v.y), quad<CTRL>(v.z));
}
constexpr int Q_XOR1 = 0xb1, Q_XOR2 = 0x4e;   // lane ^ 1, lane ^ 2
constexpr int ROW_HALF_MIRROR = 0x141, ROW_MIRROR = 0x140;   // lane 7 - i of each 8, 15 - i of each 16
constexpr int Q_LOW = 0x44, Q_HIGH = 0xee;    // lanes 0, 1, 0, 1 and 2, 3, 2, 3
// The greatest value of lanes 0 to 31, in every lane.
__device__ __forceinline__ float most32(float v) {
  v = fmaxf(v, quad<Q_XOR1>(v));
  v = fmaxf(v, quad<Q_XOR2>(v));
  v = fmaxf(v, quad<ROW_HALF_MIRROR>(v));
  v = fmaxf(v, quad<ROW_MIRROR>(v));
  const int i = __float_as_int(v);
  return fmaxf(__int_as_float(__builtin_amdgcn_readlane(i, 0)), __int_as_float(__builtin_amdgcn_readlane(i, 16)));
}

// ------------------------------------------------------------------ clipping
// the clip buffers of wave wid
template <class S>
__device__ __forceinline__ f3 cl_get(const S& s, int wid, int buf, int i, int grp) {
  const auto& c = s.u.n.x.clip[wid][buf][i];
  return mk(c[0][grp], c[1][grp], c[2][grp]);
}
template <class S>
__device__ __forceinline__ void cl_put(S& s, int wid, int buf, int i, int grp, f3 v) {
  auto& c = s.u.n.x.clip[wid][buf][i];
  c[0][grp] = v.x;
  c[1][grp] = v.y;
  c[2][grp] = v.z;
}

// Value of lane K of each group of LP = 16 or 8 lanes (DPP row broadcast; of
// eight lanes, each half of a row takes its own lane K).
template <int LP, int K>
__device__ __forceinline__ float group_value(float v) {
  const int i = __float_as_int(v);
  if constexpr (LP == 16) return __int_as_float(__builtin_amdgcn_mov_dpp(i, 0x150 + K, 0xf, 0xf, true));
  const int lower = __builtin_amdgcn_update_dpp(i, i, 0x150 + K, 0xf, 0x3, true);
  return __int_as_float(__builtin_amdgcn_update_dpp(lower, i, 0x150 + (K + 8) % 16, 0xf, 0xc, true));
}

// The lane before in each group, lane 0 taking the last: DPP row_ror:1, and
// row_ror:9 for the first lanes of eight.
template <int LP>
__device__ __forceinline__ float group_prev(float v, bool first) {
  const int i = __float_as_int(v);
  const int prev = __builtin_amdgcn_mov_dpp(i, 0x121, 0xf, 0xf, true);
  if constexpr (LP == 16) return __int_as_float(prev);
  const int wrap = __builtin_amdgcn_mov_dpp(i, 0x129, 0xf, 0xf, true);
  return __int_as_float(first ? wrap : prev);
}

// One Sutherland-Hodgman stage against sign * ((x - f).dir) - h <= 0 for
// the polygons of all groups of LP lanes at once, point i of a group's polygon
// in lane i of the group (lanes past the last point, lanes 8-15 too, hold copies
// of it).
// Lane i handles the edge from point i-1 (the last point for i = 0) to
// point i: it emits the crossing point if the edge crosses the plane, then
// point i if inside, at its rank among the group's emissions; at most POLY
// points are kept.  Called by the whole wave.  Copies in all sixteen lanes make
// the point before one DPP move, also for lane 0 (1024 x 15: 1.12 -> 1.11 ms
// against the two moves and the select of eight lanes).
template <int LP, class S>
__device__ __forceinline__ int clip_group(S& s, f3* P, int n, f3 f, f3 dir, float sign, float h, int buf,
                                          int grp, int gl, int lane, int wid) {
  const float dc = sign * dot(*P - f, dir) - h;
  // no point of any group outside this plane: nothing crosses it and every
  // point is kept in place, so the stage changes nothing
  if (__ballot(gl < n && !(dc <= 0.0f)) == 0ull) return n;
  // the previous point, for lane 0 the last lane's copy of the last
  const bool first = gl == 0;
  const f3 Pp = mk(group_prev<LP>(P->x, first), group_prev<LP>(P->y, first), group_prev<LP>(P->z, first));
  const float dp = group_prev<LP>(dc, first);
  const bool live = gl < n;
  const bool in_c = dc <= 0.0f, in_p = dp <= 0.0f;
  const bool emit_x = live && (in_c != in_p), emit_c = live && in_c;
  const unsigned long long mx = __ballot(emit_x), mc = __ballot(emit_c);
  const unsigned long long gm = ((1ull << LP) - 1ull) << (LP * grp), below = ((1ull << lane) - 1ull) & gm;
  const int q = __popcll(mx & below) + __popcll(mc & below);
  const int m = __popcll(mx & gm) + __popcll(mc & gm);
  if (emit_x && q < POLY) cl_put(s, wid, buf, q, grp, fma3(*P - Pp, dp * rcp(dp - dc), Pp));
  if (emit_c && q + (emit_x ? 1 : 0) < POLY) cl_put(s, wid, buf, q + (emit_x ? 1 : 0), grp, *P);
  wave_sync();
  const int nn = m < POLY ? m : POLY;
  if (nn > 0) *P = cl_get(s, wid, buf, gl < nn ? gl : nn - 1, grp);
  return nn;
}

// Axis k and half extent k of LDS body i (dynamic k reads LDS, so no
// register array is indexed at run time).
template <class S>
__device__ __forceinline__ f3 lds_axis(const S& s, int i, int k) {
  return xyz(s.col[k][i]);
}
template <class S>
__device__ __forceinline__ float lds_half(const S& s, int i, int k) {
  return reinterpret_cast<const float*>(&s.half[i])[k];
}

// Edge-axis contact: closest points of the two extreme edges parallel to the
// axis's edge directions (A extreme along +n, B along -n; sign 0 -> +).
template <class S>
__device__ __forceinline__ f3 edge_point(const S& s, int ia, int ib, int idx, f3 n) {
  const int i = (idx - 6) / 3, j = (idx - 6) % 3;
  f3 pa = xyz(s.pos[ia]), pb = xyz(s.pos[ib]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k != i) {
      f3 ak = xyz(s.col[k][ia]);
      pa = pa + ak * ((dot(n, ak) >= 0.0f ? 1.0f : -1.0f) * lds_half(s, ia, k));
    }
    if (k != j) {
      f3 bk = xyz(s.col[k][ib]);
      pb = pb + bk * ((dot(neg(n), bk) >= 0.0f ? 1.0f : -1.0f) * lds_half(s, ib, k));
    }
  }
  f3 ai = lds_axis(s, ia, i), bj = lds_axis(s, ib, j);
  float ha = lds_half(s, ia, i), hb = lds_half(s, ib, j);
  f3 r = pa - pb;
  float c = dot(ai, bj), ar = dot(ai, r), br = dot(bj, r);
  float denom = 1.0f - c * c;
  float ss = fminf(fmaxf((c * br - ar) / denom, -ha), ha);
  float tt = br + ss * c;
  if (tt < -hb || tt > hb) {
    tt = fminf(fmaxf(tt, -hb), hb);
    ss = fminf(fmaxf(tt * c - ar, -ha), ha);
  }
  f3 qa = pa + ai * ss, qb = pb + bj * tt;
  return (qa + qb) * 0.5f;
}

// ------------------------------------------------------------------ contact record in VGPRs
struct Contact {
  int ab;
  f3 n, t1, t2, ra, rb;
  float kn, kt1, kt2, vstar, mu;
  float ln, lt1, lt2;
};

// Index of a key in the previous substep's row contacts, -1 when absent.
template <class S>
__device__ __forceinline__ int warm_index(const S& s, int key, int nwarm) {
  int lo = 0, hi = nwarm - 1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1, km = s.wkey[mid];
    if (km == key) return mid;
    if (km < key) lo = mid + 1;
    else hi = mid - 1;
  }
  return -1;
}

template <class S>
__device__ __forceinline__ float eff_mass_side(const S& s, int i, f3 r, f3 d) {
  f3 cr = cross(r, d);
  float4 ia = s.iwa[i], ib = s.iwb[i];
  // symmetric Iw^-1 times cr
  f3 m = mk(ia.x * cr.x + ia.w * cr.y + ib.x * cr.z,
            ia.w * cr.x + ia.y * cr.y + ib.y * cr.z,
            ib.x * cr.x + ib.y * cr.y + ia.z * cr.z);
  return s.half[i].w + dot(cr, m);
}

// Tangent basis from the world axis least aligned with the normal.
__device__ __forceinline__ void tangents(f3 n, f3* t1, f3* t2) {
  float ax = fabsf(n.x), ay = fabsf(n.y), az = fabsf(n.z);
  const int ei = (ax <= ay && ax <= az) ? 0 : (ay <= az ? 1 : 2);
  f3 e = mk(ei == 0 ? 1.0f : 0.0f, ei == 1 ? 1.0f : 0.0f, ei == 2 ? 1.0f : 0.0f);
  *t1 = cross(e, n);
  *t1 = *t1 * rsq(dot(*t1, *t1));
  *t2 = cross(n, *t1);
}

// Row contact c of the staging array into registers.
template <class S>
__device__ __forceinline__ void prep_contact(const S& s, int c, const Params& p, Contact* ct) {
  const float4 s0 = s.u.n.stage[c][0], s1 = s.u.n.stage[c][1];
  f3 pt = xyz(s0);
  float sep = s0.w;
  int ab = s.cab[c];
  int a = ab & 255, b = (ab >> 8) & 255;
  ct->ab = ab;
  f3 n = xyz(s1);
  ct->n = n;
  ct->ra = pt - xyz(s.pos[a]);
  ct->rb = pt - xyz(s.pos[b]);
  f3 t1, t2;
  tangents(n, &t1, &t2);
  ct->t1 = t1;
  ct->t2 = t2;
  float ca = (float)s.cnt[a], cb = (float)s.cnt[b];
  ct->kn = rcp(ca * eff_mass_side(s, a, ct->ra, n) + cb * eff_mass_side(s, b, ct->rb, n));
  ct->kt1 = rcp(ca * eff_mass_side(s, a, ct->ra, t1) + cb * eff_mass_side(s, b, ct->rb, t1));
  ct->kt2 = rcp(ca * eff_mass_side(s, a, ct->ra, t2) + cb * eff_mass_side(s, b, ct->rb, t2));
  ct->mu = 0.5f * (s.iwb[a].z + s.iwb[b].z);
  ct->vstar = sep > 0.0f ? -sep * p.inv_dt : p.beta * fmaxf(-sep - p.slop, 0.0f) * p.inv_dt;
}

// The impulse (n, t1, t2) that row contact c starts from: the previous
// substep's of the same key, among its nwarm rows or, for one of the n_extra
// table corners among the rows, in the impulses that the lanes left in LDS.
template <class S>
__device__ __forceinline__ f3 warm_impulse(const S& s, int c, int nwarm, int n_extra) {
  const int ab = s.cab[c], key = contact_key<S>(ab);
  // an unchanged list prefix has it at the same index
  const int i = c < nwarm && s.wkey[c] == key ? c : warm_index(s, key, nwarm);
  f3 l = i >= 0 ? mk(s.wl[0][i], s.wl[1][i], s.wl[2][i]) : mk(0, 0, 0);
  if (c < n_extra) {
    const int b = (ab >> 8) & 255, kc = ab >> 16;
    const unsigned old = (unsigned)__float_as_int(s.u.n.x.lam[4 * b].w);
    const int o = __popc(old & ((1u << kc) - 1u));
    if ((old >> kc & 1u) && o < 4) l = xyz(s.u.n.x.lam[4 * b + o]);
  }
  return l;
}

// Row contact c in registers, with its impulse of the previous substep; past
// the last an absent contact of the table with itself: zero impulses.
template <class S>
__device__ __forceinline__ Contact begin_row(const S& s, int c, int n_rows, int nwarm, int n_extra, const Params& p) {
  Contact q;
  if (c < n_rows) {
    prep_contact(s, c, p, &q);
    const f3 l = warm_impulse(s, c, nwarm, n_extra);
    q.ln = l.x;
    q.lt1 = l.y;
    q.lt2 = l.z;
  } else {
    const f3 z = mk(0, 0, 0);
    q = Contact{S::PLANE | (S::PLANE << 8), z, z, z, z, z, 0, 0, 0, 0, 0, 0, 0, 0};
  }
  return q;
}

// The impulse rows (P, ra x P, rb x P) of the impulse R.
template <class S>
__device__ __forceinline__ void put_row(S& s, int c, const Contact& q, f3 R) {
  st3(&s.u.imp[0][c], R);
  st3(&s.u.imp[1][c], cross(q.ra, R));
  st3(&s.u.imp[2][c], cross(q.rb, R));
}

// One iteration's update from the published velocities.
template <class S>
__device__ __forceinline__ void update_row(S& s, int c, Contact& q) {
  const int a = q.ab & 255, bb = (q.ab >> 8) & 255;
  const f3 va = xyz(s.vel[a]), ta = xyz(s.ang[a]), vb = xyz(s.vel[bb]), tb = xyz(s.ang[bb]);
  const f3 wa = mk(ta.z, ta.x, ta.y), wb = mk(tb.z, tb.x, tb.y);
  const f3 u = cross_add(wb, q.rb, vb) - cross_add(wa, q.ra, va);
  const float ln = fmaxf(q.ln + q.kn * (q.vstar - dot(u, q.n)), 0.0f);
  const float dln = ln - q.ln;
  q.ln = ln;
  float lt1 = q.lt1 - q.kt1 * dot(u, q.t1);
  float lt2 = q.lt2 - q.kt2 * dot(u, q.t2);
  const float lim = q.mu * ln, mag2 = lt1 * lt1 + lt2 * lt2;
  const float sc = fminf(lim * rsq(mag2), 1.0f);
  lt1 *= sc;
  lt2 *= sc;
  const float dl1 = lt1 - q.lt1, dl2 = lt2 - q.lt2;
  q.lt1 = lt1;
  q.lt2 = lt2;
  put_row(s, c, q, fma3(q.n, dln, fma3(q.t1, dl1, q.t2 * dl2)));
}

// The substep's accumulated impulses by key, for the next one.
template <class S>
__device__ __forceinline__ void keep_row(S& s, int c, int n_rows, const Contact& q) {
  if (c < n_rows) {
    s.wkey[c] = contact_key<S>(q.ab);
    s.wl[0][c] = q.ln;
    s.wl[1][c] = q.lt1;
    s.wl[2][c] = q.lt2;
  }
}

// A wave's row contacts, a lane each: slots FIRST, FIRST + STEP, ... of 64
// contacts, all in registers.  exchange() orders the rows and velocities
// against the other lanes' (of every wave that has part in them); sums(),
// publish() and table() are the body lanes' part of an iteration.  Bound by the
// chain of an iteration: velocities gathered, about 90 instructions a slot, rows
// left in LDS and added by the bodies' lanes.  60 substeps of 1024 x 10 cubes in
// two touching towers (73 rows), 128-contact class: two waves 1.69 -> 1.16 ms
// against all rows on the lead wave, one wave 1.78 -> 1.49 with the sums below;
// 1024 x 30 touching cubes (244 rows, 512-contact class) 10.3 -> 8.6 ms.  Slots
// past the second in a lane's private memory instead, the next one's read ahead:
// 1024 x 15 touching cubes (134 rows, 256-contact class) 1.96 -> 2.13 ms.
template <int FIRST, int STEP, class S, class X, class Q, class V, class T>
__device__ __forceinline__ void solve_rows(S& s, int lane, int n_rows, int nwarm, int n_extra, const Params& p, X exchange,
                                           Q sums, V publish, T table) {
  constexpr int N = S::C / 64 / STEP;   // the wave's slots
  Contact ct[N];
  auto each_slot = [&](auto f) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = 64 * (FIRST + STEP * i);
      if (c == 0 || c < n_rows) f(c + lane, ct[i]);
    }
  };
  each_slot([&](int c, Contact& q) { q = begin_row(s, c, n_rows, nwarm, n_extra, p); });
  exchange();   // the rows take the staging array's place
  each_slot([&](int c, Contact& q) { put_row(s, c, q, fma3(q.n, q.ln, fma3(q.t1, q.lt1, q.t2 * q.lt2))); });
  exchange();
  sums();
  for (int it = 0; it < p.iters; ++it) {
    publish();
    table();
    each_slot([&](int c, Contact& q) { update_row(s, c, q); });
    exchange();   // the impulse rows
    sums();
  }
  each_slot([&](int c, Contact& q) { keep_row(s, c, n_rows, q); });
}

// A row contact spread over four lanes: lane q of the quad has row q of its
// frame (q = 0 normal, 1 and 2 tangents; impulse lam, effective mass k) and
// component q of its vectors (lane 3 repeats lane 0 and is not read).
struct QuadContact {
  int at_a, at_b;             // bodies a and b: offset of their velocity's component q
  f3 dir, comp;               // frame row q; component q of the three rows
  float ra1, ra2, rb1, rb2;   // components q + 1 and q + 2 of the lever arms
  float k, vs, mu, lam;
  int lo;                     // least impulse as an integer (negative floats are negative integers)
};

// Components q, q + 1 and q + 2 (cyclic) of a vector.
__device__ __forceinline__ f3 turn(f3 v, int q) {
  return sel(q == 1, mk(v.y, v.z, v.x), sel(q == 2, mk(v.z, v.x, v.y), v));
}

// Row contact c of the staging array into the lanes of a quad: the terms of
// prep_contact, each lane with its own row's effective mass.
template <class S>
__device__ __forceinline__ void prep_quad(const S& s, int c, int q, const Params& p, QuadContact* ct) {
  const float4 s0 = s.u.n.stage[c][0];
  const f3 pt = xyz(s0), n = xyz(s.u.n.stage[c][1]);
  const float sep = s0.w;
  const int ab = s.cab[c], a = ab & 255, b = (ab >> 8) & 255;
  const f3 ra = pt - xyz(s.pos[a]), rb = pt - xyz(s.pos[b]);
  f3 t1, t2;
  tangents(n, &t1, &t2);
  const f3 d = sel(q == 1, t1, sel(q == 2, t2, n));
  const float ca = (float)s.cnt[a], cb = (float)s.cnt[b];
  ct->k = rcp(ca * eff_mass_side(s, a, ra, d) + cb * eff_mass_side(s, b, rb, d));
  const bool normal = q != 1 && q != 2;
  const float vstar = sep > 0.0f ? -sep * p.inv_dt : p.beta * fmaxf(-sep - p.slop, 0.0f) * p.inv_dt;
  ct->mu = normal ? INFINITY : 0.5f * (s.iwb[a].z + s.iwb[b].z);
  ct->vs = normal ? vstar : 0.0f;
  // the normal impulse is clamped from below and not scaled by the friction
  // disc: an infinite limit scales by 1, also where it gives a nan
  ct->lo = normal ? 0 : INT32_MIN;
  ct->dir = d;
  ct->comp = mk(turn(n, q).x, turn(t1, q).x, turn(t2, q).x);
  const f3 ta = turn(ra, q), tb = turn(rb, q);
  ct->ra1 = ta.y;
  ct->ra2 = ta.z;
  ct->rb1 = tb.y;
  ct->rb2 = tb.z;
  const int qc = q < 3 ? q : 0;
  ct->at_a = 4 * a + qc;
  ct->at_b = 4 * b + qc;
}

// Row contact lane / 4 of n_rows in the lane's quad, with its impulse of the
// previous substep; past the last an absent contact of the table with itself:
// zero impulses.
template <class S>
__device__ __forceinline__ QuadContact begin_quad(const S& s, int lane, int n_rows, int nwarm, int n_extra, const Params& p) {
  const int c = lane >> 2, q = lane & 3;
  const f3 z = mk(0, 0, 0);
  QuadContact qc;
  if (c < n_rows) {
    prep_quad(s, c, q, p, &qc);
    qc.lam = turn(warm_impulse(s, c, nwarm, n_extra), q).x;
  } else {
    qc = QuadContact{4 * S::PLANE, 4 * S::PLANE, z, z, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  }
  return qc;
}

// The impulse rows (P, ra x P, rb x P) of a change dl of the quad's impulses.
template <class S>
__device__ __forceinline__ void put_quad(S& s, int lane, const QuadContact& qc, float dl) {
  float* const rows = reinterpret_cast<float*>(&s.u.imp[0][0]) + lane;
  const float R = fmaf(qc.comp.x, quad<0x00>(dl), fmaf(qc.comp.y, quad<0x55>(dl), qc.comp.z * quad<0xaa>(dl)));
  const float R1 = quad<0xc9>(R), R2 = quad<0xd2>(R);   // components q + 1, q + 2
  rows[0] = R;
  rows[4 * S::C] = qc.ra1 * R2 - qc.ra2 * R1;
  rows[8 * S::C] = qc.rb1 * R2 - qc.rb2 * R1;
}

// One iteration's update of the quad's impulses from the published velocities;
// meanwhile() runs while these load.  Returns the change.
template <class S, class F>
__device__ __forceinline__ float update_quad(const S& s, QuadContact& qc, F meanwhile) {
  const float* const vel = reinterpret_cast<const float*>(&s.vel[0]);
  const float* const ang = reinterpret_cast<const float*>(&s.ang[0]);
  const float va = vel[qc.at_a], wa1 = ang[qc.at_a], wa2 = ang[qc.at_a + 1];
  const float vb = vel[qc.at_b], wb1 = ang[qc.at_b], wb2 = ang[qc.at_b + 1];
  meanwhile();
  const float u = fmaf(wb1, qc.rb2, fmaf(-wb2, qc.rb1, vb)) - fmaf(wa1, qc.ra2, fmaf(-wa2, qc.ra1, va));
  const f3 U = mk(quad<0x00>(u), quad<0x55>(u), quad<0xaa>(u));
  float l = __int_as_float(max(__float_as_int(qc.lam + qc.k * (qc.vs - dot(U, qc.dir))), qc.lo));
  const float ln = quad<0x00>(l), lt1 = quad<0x55>(l), lt2 = quad<0xaa>(l);
  const float lim = qc.mu * ln, mag2 = lt1 * lt1 + lt2 * lt2;
  l *= fminf(lim * rsq(mag2), 1.0f);
  const float dl = l - qc.lam;
  qc.lam = l;
  return dl;
}

// The substep's accumulated impulses by key, for the next one.
template <class S>
__device__ __forceinline__ void keep_quad(S& s, int lane, int n_rows, const QuadContact& qc) {
  const int c = lane >> 2, q = lane & 3;
  if (c < n_rows && q < 3) {
    if (q == 0) s.wkey[c] = contact_key<S>(s.cab[c]);
    s.wl[q][c] = qc.lam;
  }
}

// A table contact: normal z, tangents -y and x, nothing on side a.  The
// impulse of changes (dn, d1, d2) is (d2, -d1, dn) exactly.
struct TableContact {
  f3 rb;
  float kn, kt1, kt2, vstar;
  float ln, lt1, lt2;
};

// r x z, r x -y and r x x against a symmetric matrix a (xx, yy, zz), o (xy,
// xz, yz): the effective-mass products of the general contact with the terms
// that are exactly zero left out, in the same order.
__device__ __forceinline__ f3 table_masses(f3 r, f3 a, f3 o) {
  const float n_x = r.y, n_y = -r.x;
  const float n_mx = fmaf(a.x, n_x, o.x * n_y), n_my = fmaf(o.x, n_x, a.y * n_y);
  const float u_x = r.z, u_z = -r.x;
  const float u_mx = fmaf(o.y, u_z, a.x * u_x), u_mz = fmaf(a.z, u_z, o.y * u_x);
  const float v_y = r.z, v_z = -r.y;
  const float v_my = fmaf(o.z, v_z, a.y * v_y), v_mz = fmaf(a.z, v_z, o.z * v_y);
  return mk(fmaf(n_x, n_mx, n_y * n_my), fmaf(u_z, u_mz, u_x * u_mx), fmaf(v_z, v_mz, v_y * v_my));
}

// Half extents along x, y, z of the margin-inflated AABB of a box.
__device__ __forceinline__ f3 aabb_ext(f3 a0, f3 a1, f3 a2, f3 hh, float margin) {
  return mk(fabsf(a0.x) * hh.x + fabsf(a1.x) * hh.y + fabsf(a2.x) * hh.z + margin,
            fabsf(a0.y) * hh.x + fabsf(a1.y) * hh.y + fabsf(a2.y) * hh.z + margin,
            fabsf(a0.z) * hh.x + fabsf(a1.z) * hh.y + fabsf(a2.z) * hh.z + margin);
}

// Pair number p of the pairs (i, j), i < j < n <= 32, in lexicographic order, as
// i | j << 5; (0, 0) past the last pair.  Row i begins at pair i (2 n - 1 - i) / 2;
// the root's inverse of that is off by less than one row, since the roots of a
// row's last pair and the next row's first are 0.03 apart or more.  (Eight a
// lane at an env's start in the 31-box layout: one substep of 30 boxes on two
// waves 25.8 -> 23.0 us against a rounded root and loops.)
__device__ __forceinline__ unsigned pair_of(int p, int n) {
  const int m = 2 * n - 1;
  int i = (int)(0.5f * ((float)m - __builtin_amdgcn_sqrtf((float)max(m * m - 8 * p, 0))));
  i += i * (m - i) / 2 > p ? -1 : (i + 1) * (m - i - 1) / 2 <= p ? 1 : 0;
  return p < n * (n - 1) / 2 ? (unsigned)(i | (p - i * (m - i) / 2 + i + 1) << 5) : 0u;
}

// The number of pair (i, j), i < j < n, in that order.
__device__ __forceinline__ int number_of(int i, int j, int n) { return i * (2 * n - i - 1) / 2 + j - i - 1; }

// |x| + |y| + |z|
__device__ __forceinline__ float sum_abs(f3 a) { return fabsf(a.x) + fabsf(a.y) + fabsf(a.z); }

// ------------------------------------------------------------------ footprint distance (reward)
// Footprint of a box = its projection on the table (a zonotope with
// generators h_k a_k projected).  Overlap: a separating axis among the
// generators' normals.  Distance when disjoint: minimum over projected
// vertices of one against the projected box edges of the other (the
// silhouette edges are among them).
struct Foot {
  float cx, cy;
  float gx[3], gy[3];
};

// squared distance of a point from a segment
__device__ __forceinline__ float seg_dist2(float px, float py, float ax, float ay, float bx, float by) {
  float dx = bx - ax, dy = by - ay;
  float l2 = dx * dx + dy * dy;
  float t = l2 > 0.0f ? ((px - ax) * dx + (py - ay) * dy) / l2 : 0.0f;
  t = fminf(fmaxf(t, 0.0f), 1.0f);
  float ex = ax + t * dx - px, ey = ay + t * dy - py;
  return ex * ex + ey * ey;
}

__device__ __forceinline__ void foot_vertex(const Foot& f, int k, float* x, float* y) {
  float sx = (k & 1) ? 1.0f : -1.0f, sy = (k & 2) ? 1.0f : -1.0f, sz = (k & 4) ? 1.0f : -1.0f;
  *x = f.cx + (f.gx[0] * sx + f.gx[1] * sy + f.gx[2] * sz);
  *y = f.cy + (f.gy[0] * sx + f.gy[1] * sy + f.gy[2] * sz);
}

// min over P's vertices j, j + L, ... to the 12 projected edges of Q
template <int L>
__device__ __forceinline__ float foot_point_dist2(const Foot& P, const Foot& Q, int j) {
  float best = INFINITY;
#pragma unroll 1
  for (int i = j; i < 8; i += L) {
    float px, py;
    foot_vertex(P, i, &px, &py);
#pragma unroll
    for (int a = 0; a < 8; ++a) {
#pragma unroll
      for (int bit = 1; bit < 8; bit <<= 1) {
        if (a & bit) continue;
        float ax, ay, bx, by;
        foot_vertex(Q, a, &ax, &ay);
        foot_vertex(Q, a | bit, &bx, &by);
        best = fminf(best, seg_dist2(px, py, ax, ay, bx, by));
      }
    }
  }
  return best;
}

__device__ __forceinline__ bool foot_separated_by(const Foot& F, const Foot& P, const Foot& Q, float dx, float dy) {
  bool sep = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    float lx = -F.gy[k], ly = F.gx[k];
    float rp = fabsf(P.gx[0] * lx + P.gy[0] * ly) + fabsf(P.gx[1] * lx + P.gy[1] * ly) + fabsf(P.gx[2] * lx + P.gy[2] * ly);
    float rq = fabsf(Q.gx[0] * lx + Q.gy[0] * ly) + fabsf(Q.gx[1] * lx + Q.gy[1] * ly) + fabsf(Q.gx[2] * lx + Q.gy[2] * ly);
    if (fabsf(dx * lx + dy * ly) > rp + rq) sep = true;
  }
  return sep;
}

// Squared distance of two footprints over lane j's share of their vertices
// (of L lanes whose least value is the distance); 0 when they overlap.  A
// correctly rounded square root is monotone, so the root of the least square
// is the least distance, bit for bit.
template <int L>
__device__ __forceinline__ float foot_distance2(const Foot& P, const Foot& Q, int j) {
  const float dx = Q.cx - P.cx, dy = Q.cy - P.cy;
  if (!(foot_separated_by(P, P, Q, dx, dy) || foot_separated_by(Q, P, Q, dx, dy))) return 0.0f;
  return fminf(foot_point_dist2<L>(P, Q, j), foot_point_dist2<L>(Q, P, j));
}

// footprint from the body frame: centre, rotation columns, half extents
__device__ __forceinline__ Foot foot_of(f3 c, f3 a0, f3 a1, f3 a2, f3 h) {
  Foot f;
  f.cx = c.x;
  f.cy = c.y;
  f.gx[0] = a0.x * h.x; f.gx[1] = a1.x * h.y; f.gx[2] = a2.x * h.z;
  f.gy[0] = a0.y * h.x; f.gy[1] = a1.y * h.y; f.gy[2] = a2.y * h.z;
  return f;
}

// rotation columns of a unit quaternion (body to world)
__device__ __forceinline__ void quat_cols(float q0, float q1, float q2, float q3, f3* c0, f3* c1, f3* c2) {
  *c0 = mk(1 - 2 * (q2 * q2 + q3 * q3), 2 * (q1 * q2 + q0 * q3), 2 * (q1 * q3 - q0 * q2));
  *c1 = mk(2 * (q1 * q2 - q0 * q3), 1 - 2 * (q1 * q1 + q3 * q3), 2 * (q2 * q3 + q0 * q1));
  *c2 = mk(2 * (q1 * q3 + q0 * q2), 2 * (q2 * q3 - q0 * q1), 1 - 2 * (q1 * q1 + q2 * q2));
}

// ------------------------------------------------------------------ random pushes
// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC 2011) keyed by a 64-bit
// seed; the random push of a simulation is the first output word modulo the
// number of actions, counter (node id, first action, replica << 8 | push
// index, 2).
__device__ __forceinline__ int philox_action(uint2 key, unsigned c0, unsigned c1, unsigned c2, unsigned n_actions) {
  unsigned c3 = 2u, k0 = key.x, k1 = key.y;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const unsigned hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const unsigned hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const unsigned n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  return (int)(c0 % n_actions);
}

// ------------------------------------------------------------------ one environment
// Orders LDS accesses across the waves of an environment's workgroup (a
// barrier) when there is more than one, else within the wave.
template <int W>
__device__ __forceinline__ void sync_all() {
  if constexpr (W > 1) __syncthreads();
  else wave_sync();
}

// Runs env e through its pushes: one explicit push (step mode) or a list of
// contour pushes (rollout mode, with a reward after each push).
//
// Body lanes: L lanes of the lead wave carry each body (lane b L + j), four
// in the 16-box layout and two in the 31-box one.  All of them hold its whole
// state, and together its first four table contacts (contact j + L ts in slot
// ts): a table contact's only body is the lanes' own, so its update needs no
// memory, and the body's sum over these contacts is a DPP exchange among
// the L lanes.  The other contacts (pairs, the pusher, a box's fifth and
// later table corner) are row contacts: four lanes each, or one per lane and
// slot, their velocities gathered from and their impulse rows left in LDS,
// where the body lanes add them after the table contacts, the even and the
// odd entries of the body's contact list separately, as ever.
//
// Bound: the vector ALU and the LDS pipe, each about half busy before (2076
// VALU instructions and 2061 LDS cycles per env-substep at 4096 x 15, 3866
// cycles of a CU), most of them in the ten iterations, whose every contact
// gathered four velocities from LDS, left three rows there and had them read
// back.  Nineteen of twenty contacts are table contacts: normal z, tangents
// -y and x, nothing on side a.  With the terms that are exactly zero left out
// (the same bits) and the body in the same lanes such a contact costs 28
// instructions instead of 61 and no LDS, and an environment of which no box
// touches another iterates without LDS at all.  4096 x 15: 3.15 -> 2.19 ms;
// 700 x 27: 2.66 -> 1.85; 1024 x 15 on two waves: 1.50 -> 1.32; 64 x 9, one
// wave per SIMD: 1.19 -> 1.10.  With row contacts in quads of lanes (below):
// 2.09, 1.73, 1.18 and 0.97 ms; with what followed, 1.76, 1.35, 1.12 and 0.88.
// Now it is the vector ALU where a SIMD has three environments, and the chain
// of dependent instructions, a substep after the other, where it has one.
//
// With W > 1 waves per environment the second wave tests the broadphase pairs
// while the lead finds the table contacts, takes every second narrowphase pass
// (of four or eight pairs), and updates row contacts while the lead updates its
// lanes' table contacts: of more than 16 every second slot of 64, and up to 16
// in quads, all of them, in the 31-box layout.  The results are bitwise those of
// W = 1.  Uniform
// decisions (push validity, rewards, overflow) are taken by every wave from
// the same LDS data, so all waves run the same loops and meet at the same
// barriers.
//
// The cost pass and pmbs_sim_collide end in the first substep, after its
// contacts: their kernels hold no more than that.
enum class Run { STEP, COST, COLLIDE };
template <int K, int W, int NB, Run RUN>
__device__ __forceinline__ void run_env(Smem<K, W, NB>& s, const StepArgs& g, const int e) {
  using S = Smem<K, W, NB>;
  constexpr int C = S::C, PLANE = S::PLANE, MB = S::MB;
  constexpr int L = NB == 16 ? 4 : 2;   // lanes per body
  constexpr int TS = 4 / L;             // table contacts per lane
  constexpr bool SPLIT = W > 1 && TS > 1;   // the second wave updates the quads of row contacts
  const Params& p = g.p;
  // opaque: what follows from the lane number is formed anew for each env
  // and substep; kept over them it fills the registers with addresses
  const int lane = opaque(threadIdx.x & 63);
  const int wid = W > 1 ? (int)(threadIdx.x >> 6) : 0;
  const bool lead = wid == 0;
  // scalar where there are barriers on either side of its branch, which whole
  // waves then take
  const bool row_wave = W > 1 && __builtin_amdgcn_readfirstlane(wid) != 0;
  const int b = (unsigned)lane / L, j = (unsigned)lane % L;
  const int base = g.env_offset[e];
  const int nb = g.env_offset[e + 1] - base;
  const bool active = lead && b < nb;  // a lane of the lead wave that owns a body
  const bool first = active && j == 0;
  const int N = g.stride;
  const float dt = p.dt;
  const bool rollout = g.actions != nullptr;
  const int act0 = rollout ? g.act_offset[e] : 0;
  int n_push = rollout ? g.act_offset[e + 1] - act0 : 1;
  const int src = (rollout && g.src_slot) ? g.src_slot[e] : -1;
  const int PS = g.pool_stride;

  // ---- load (SoA rows; the lanes of a body read the same words), from the
  // env arrays or from the state pool slot of the node being expanded
  f3 x = mk(0, 0, 0), v = mk(0, 0, 0), w = mk(0, 0, 0), h = mk(0, 0, 0), invI = mk(0, 0, 0);
  float q0 = 1, q1 = 0, q2 = 0, q3 = 0, invm = 0, mu = 0;
  if (active) {
    const int i = base + b;
    const float* st = src >= 0 ? g.pool + (size_t)src * 13 * PS : g.state;
    const int SN = src >= 0 ? PS : N;
    const int si = src >= 0 ? b : i;
    const float* bc = g.bconst;
    const int BN = g.bc_base ? g.bc_stride : N;
    const int bi = g.bc_base ? g.bc_base[e] + b : i;
    x = mk(st[0 * SN + si], st[1 * SN + si], st[2 * SN + si]);
    q0 = st[3 * SN + si]; q1 = st[4 * SN + si]; q2 = st[5 * SN + si]; q3 = st[6 * SN + si];
    v = mk(st[7 * SN + si], st[8 * SN + si], st[9 * SN + si]);
    w = mk(st[10 * SN + si], st[11 * SN + si], st[12 * SN + si]);
    h = mk(bc[0 * BN + bi], bc[1 * BN + bi], bc[2 * BN + bi]);
    invm = bc[3 * BN + bi];
    invI = mk(bc[4 * BN + bi], bc[5 * BN + bi], bc[6 * BN + bi]);
    mu = bc[7 * BN + bi];
  }
  const f3 ph = mk(p.phx, p.phy, p.phz);
  const float mu_table = 0.5f * (p.mu_plane + mu);
  // what no substep changes: half extents, and the pusher entry (index nb)
  if (first) s.half[b] = f4(h, invm);
  if (lead && lane == 0) {
    s.half[nb] = f4(ph, 0.0f);
    s.iwa[nb] = make_float4(0, 0, 0, 0);
    s.iwb[nb] = make_float4(0, 0, p.mu_pusher, 0);
    s.ang[nb] = make_float4(0, 0, 0, 0);
    s.cnt[nb] = 1;
  }

  // frames of the bodies (centre, rotation)
  f3 c0, c1, c2;
  auto write_body_frames = [&](int b, bool first, float moved) {
    quat_cols(q0, q1, q2, q3, &c0, &c1, &c2);
    if (first) {
      s.pos[b] = f4(x, moved);
      st3(&s.col[0][b], c0);
      st3(&s.col[1][b], c1);
      st3(&s.col[2][b], c2);
      s.quat[b] = make_float4(q0, q1, q2, q3);
    }
  };

  bool deferred = false;
  uint32_t status = 0u;
  float last_r = 0.0f;
  int n_rewards = 0;
  long long stat_nc = 0, stat_pairs = 0, stat_sub = 0;
  const int n_obj = nb + 1;
  // the lane's broadphase pairs, pass k's in bits 10 (k mod 3) .. of word k / 3
  const int n_tri = n_obj * (n_obj - 1) / 2;
  constexpr int PASSES = (S::MAX_PAIRS + 63) / 64;
  unsigned tri[(PASSES + 2) / 3];
#pragma unroll
  for (int k = 0; k < PASSES; ++k) {
    const unsigned ij = pair_of(64 * k + lane, n_obj) << (10 * (k % 3));
    tri[k / 3] = k % 3 ? tri[k / 3] | ij : ij;
  }

  // job 0 is the env's own simulation; job 1 (re-purposing) is one extra
  // simulation of another pair that spends the pushes left when job 0
  // reached reward 1 early
  int t_stop = -1, n_rewards_x = 0;
  for (int job = 0; job < 2; ++job) {
  for (int t = 0; t < n_push; ++t) {
  // ---- push begin (uniform across the workgroup)
  write_body_frames(b, first, 0.0f);
  if (lead) {
    for (int i = lane; i < n_tri; i += 64) s.apart[i] = -INFINITY;
  }
  sync_all<W>();
  // Pairs that a face axis keeps apart are left out of the candidates while
  // they provably stay so.  A body's `moved` grows each substep by a bound on
  // how far any point within `reach` of its centre can have moved: speed and
  // angular speed times reach, over dt, each 2-norm bounded by the sum of the
  // components, and the position stage's roundings (4.8e-7 of centre and reach
  // is 8 half ulps of each).  Along a face axis that turns with its box, a gap
  // shrinks by no more than the two bodies' bounds when reach is at least the
  // distance from either centre to any point of the other box: boxes whose
  // AABBs overlap are within sqrt(3) (2 R + 2 margin) + R of each other in that
  // sense, R the largest half diagonal.  With this a candidate list holds 2.5
  // of the 9.3 overlapping pairs of 21 boxes and 1.0 of 7.1 of 15; a sieve that
  // found the others anew took 1200 to 1500 cycles of a substep (1024 x 15: 1.17
  // -> 1.13 ms; 700 x 27: 1.44 -> 1.39).
  float reach = sqrtf(dot(ph, ph)), far = 0.0f;
  if (lane < nb) {
    const f3 hl = xyz(s.half[lane]);
    reach = fmaxf(reach, sqrtf(dot(hl, hl)));
    far = sum_abs(xyz(s.pos[lane]));
  }
  reach = uniform(4.5f * most32(reach) + 4.0f * p.margin);
  far = most32(far);
  // sums are rounded up, and grow with the distance from where the push began
  constexpr float MOVE_UP = 1.0f + 0x1p-20f;
  float move_round = 4.8e-7f * (far + reach);
  const float turn_reach = uniform(dt * reach);
  // the least gap that counts: the margin, and 8e-6 of reach for the roundings of two evaluations
  const float gap0 = uniform(p.margin + 8e-6f * reach);
  // a pair's apart value from a gap along a face axis and the sum of its `moved`
  auto apart_until = [&](float gap, float moved) { return gap - gap0 + moved * 0.999999f; };

  bool have_push;
  float4 push = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (rollout) {
    // contour push (Sec. IV-B): direction dir of n_dirs around object obj in
    // its yaw frame, starting beyond the footprint's ray-to-boundary
    // distance by the pusher half width plus the standoff, moving
    // push_length toward the object centre
    int act;
    if (job == 0) {
      act = g.actions[act0 + t];
    } else {
      const int4 xd = g.x_desc[e];
      act = t == 0 ? xd.y
                   : philox_action(g.x_key[e], (unsigned)xd.z, (unsigned)xd.y,
                                   (((unsigned)xd.w & 0xffffffu) << 8) | (unsigned)t, (unsigned)(nb * p.n_dirs));
    }
    const int obj = act / p.n_dirs, dir = act - obj * p.n_dirs;
    have_push = obj >= 0 && obj < nb;
    if (have_push) push = contour_start(s, obj, dir, p);
  } else {
    have_push = g.push != nullptr;
    if (have_push) push = g.push[e];
  }
  f3 pdir = mk(1, 0, 0);
  int n_move = 0;
  f3 xp = mk(0, 0, 10.0f);
  f3 pc0 = mk(1, 0, 0), pc1 = mk(0, 1, 0);
  if (have_push) {
    const PusherPose pq = pusher_pose(push, p);
    pdir = pq.dir;
    n_move = pq.n_move;
    xp = pq.x;
    pc0 = pq.c0;
    pc1 = pq.c1;
  }

  // validity of the start pose: SAT separation from every box must be > 0
  bool valid = false;
  if (have_push) {
    bool bad = false;
    if (lane < nb) {   // every wave tests the boxes from LDS: the same decision
      PusherPose pq;
      pq.x = xp;
      pq.c0 = pc0;
      pq.c1 = pc1;
      bad = !sat_clear(load_box(s, lane), pusher_box(pq, p), p.edge_eps);
    }
    valid = __ballot(bad) == 0;
  }
  if (!valid) {
    xp = mk(0, 0, 10.0f);
    pc0 = mk(1, 0, 0);
    pc1 = mk(0, 1, 0);
    n_move = 0;
  }
  if (have_push && !valid && (!rollout || t == 0) && job == 0) status |= PMBS_ENV_PUSH_INVALID;
  if (rollout && !valid) {
    // a discarded expansion push ends the rollout; a discarded random push
    // leaves the state and repeats the previous reward
    if (t == 0) break;
    if (lead && lane == 0) (job ? g.x_rewards : g.rewards)[(size_t)e * g.max_h + t] = last_r;
    if (job == 0) n_rewards = t + 1;
    else n_rewards_x = t + 1;
    continue;
  }
  // the pusher's rotation is fixed for the push
  if (lead && lane == 0) {
    st3(&s.col[0][nb], pc0);
    st3(&s.col[1][nb], pc1);
    st3(&s.col[2][nb], mk(0, 0, 1));
  }
  move_round = uniform(move_round + 4.8e-7f * sum_abs(xp));
  const f3 pext = uniform(aabb_ext(pc0, pc1, mk(0, 0, 1), ph, p.margin));
  pdir = uniform(pdir);
  n_move = __builtin_amdgcn_readfirstlane(n_move);

  const int n_sub = g.n_substeps;
  // impulses are carried within one push only: the row contacts' (nwarm of
  // them, in LDS) and the table contacts', in the lanes, whose corners are
  // the bits of corners
  int nwarm = 0;
  unsigned corners = 0u;
  TableContact tc[TS];
  int kk[TS];
#pragma unroll
  for (int ts = 0; ts < TS; ++ts) {
    tc[ts].ln = tc[ts].lt1 = tc[ts].lt2 = 0.0f;
    kk[ts] = 0;
  }
  int n_inc = 0, inc0 = 0;   // the lane's body's list of row contacts: length and start
  int n_near = 0;            // near pairs (the broadphase's wave), the lane's first of them
  unsigned near0 = 0u;   // (its number, i, j: 16 + 8 + 8 bits)
  for (int k = 0; k < n_sub; ++k) {
    const int lane = opaque(threadIdx.x & 63), b = (unsigned)lane / L, j = (unsigned)lane % L;
    const bool active = lead && b < nb, first = active && j == 0;
    // ---- 1. velocity stage
    const float step_move = fmaf(turn_reach, sum_abs(w), fmaf(dt, sum_abs(v), move_round));
    v.z -= p.gravity * dt;
    const float vs = (valid && k < n_move) ? p.push_speed : 0.0f;
    const f3 vp = pdir * vs;

    // ---- 2. frames and AABBs.  Half extents, and after the narrowphase
    // centre, rotation and orientation, are read back from LDS: held in
    // registers over the substep they spill.
    const int bl = active ? b : 0;
    h = xyz(s.half[bl]);
    const float moved = fmaf(s.pos[bl].w, MOVE_UP, step_move);
    f3 ga, gb, gpa, gpb;   // the grown AABBs of the lane's body and of the pusher
    if constexpr (S::KEEP) {
      ga = xyz(s.glo[bl]);
      gb = xyz(s.ghi[bl]);
      gpa = xyz(s.glo[nb]);
      gpb = xyz(s.ghi[nb]);
    }
    write_body_frames(b, first, moved);
    bool relist_near = false;
    {
      const f3 ext = aabb_ext(c0, c1, c2, h, p.margin);
      const f3 lo = x - ext, hi = x + ext;
      if (first) {
        s.u.n.x.box.lo[b] = f4(lo, moved);
        st3(&s.u.n.x.box.hi[b], hi);
      }
      const bool pusher = lead && lane == 0;
      const f3 plo = xp - pext, phi = xp + pext;
      if (pusher) {
        // the pusher does not turn
        const float m = 1.001f * fmaf((float)k, move_round, (float)min(k, n_move) * (fabsf(p.push_speed) * dt));
        s.pos[nb] = f4(xp, m);
        st3(&s.vel[nb], vp);
        s.u.n.x.box.lo[nb] = f4(plo, m);
        st3(&s.u.n.x.box.hi[nb], phi);
      }
      if constexpr (S::KEEP) {
        // the near list holds while every AABB stays inside its grown one
        // (then overlapping pairs are among the pairs of grown ones)
        auto within = [&](f3 l, f3 u, f3 a, f3 c) {
          return __ballot(l.x >= a.x) & __ballot(l.y >= a.y) & __ballot(l.z >= a.z) & __ballot(u.x <= c.x) &
                 __ballot(u.y <= c.y) & __ballot(u.z <= c.z);
        };
        relist_near = lead && (k == 0 || (__ballot(active) & ~within(lo, hi, ga, gb)) != 0ull ||
                               ~within(plo, phi, gpa, gpb) != 0ull);
        if (relist_near) {
          const f3 g3 = mk(SKIN, SKIN, SKIN);
          if (first) {
            st3(&s.glo[b], lo - g3);
            st3(&s.ghi[b], hi + g3);
          }
          if (pusher) {
            st3(&s.glo[nb], plo - g3);
            st3(&s.ghi[nb], phi + g3);
          }
        }
        if constexpr (W > 1)
          if (pusher) s.sh_near = relist_near ? 1 : 0;
      }
    }
    sync_all<W>();

    // ---- 3. broadphase (the second wave when there are two): pairs tested
    // directly, 64 per pass in lexicographic order, the overlapping ones
    // listed by ballot.  In the 16-box layout every pair (at most three
    // passes); in the 31-box one (up to eight) those of the near list, which
    // is one pass, and every pair's grown AABBs when that has to be listed
    // again: at a push's start and after 6 mm of motion, fifteen substeps of
    // the pusher's (22 objects: 1535 -> 520 cycles of a lone wave's substep;
    // 700 x 27: 1.52 -> 1.46 ms).
    int n_pairs = 0, n_cand = 0;   // overlapping pairs; those of them that are candidates
    if (W == 1 || wid == 1) {
      struct Boxes {
        unsigned ii, jj;
        float4 il, jl;
        f3 ih, jh;
        float apart;
      };
      auto load = [&](unsigned ii, unsigned jj, int number) {
        const auto& b4 = s.u.n.x.box;
        return Boxes{ii, jj, b4.lo[ii], b4.lo[jj], xyz(b4.hi[ii]), xyz(b4.hi[jj]), s.apart[number]};
      };
      auto load_tri = [&](int k2) {
        const unsigned ij = (unsigned)opaque((int)tri[k2 / 3]) >> (10 * (k2 % 3));
        const unsigned ii = ij & 31u, jj = (ij >> 5) & 31u;
        if constexpr (S::KEEP) return Boxes{ii, jj, s.glo[ii], s.glo[jj], xyz(s.ghi[ii]), xyz(s.ghi[jj]), 0.0f};
        else return load(ii, jj, 64 * k2 + lane);
      };
      // the overlapping ones of a pass after the n before them in out, without
      // those that are known to be apart (near pairs: all of them)
      auto list = [&](const Boxes& t, auto& out, int& n, bool near) {
        // one compare per ballot, joined in scalar registers
        unsigned long long hm = __ballot(t.ii < t.jj) & __ballot(t.il.x <= t.jh.x) & __ballot(t.jl.x <= t.ih.x) &
                                __ballot(t.il.y <= t.jh.y) & __ballot(t.jl.y <= t.ih.y) &
                                __ballot(t.il.z <= t.jh.z) & __ballot(t.jl.z <= t.ih.z);
        if (!near) {
          n_pairs += __popcll(hm);
          hm &= ~__ballot(t.il.w + t.jl.w < t.apart);
        }
        // rank among the lower lanes' hits (mbcnt)
        const int rk = __builtin_amdgcn_mbcnt_hi((unsigned)(hm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hm, 0u));
        if (__builtin_amdgcn_inverse_ballot_w64(hm)) out[n + rk] = (unsigned short)((t.ii << 8) | t.jj);
        n += __popcll(hm);
      };
      // every pair (of grown AABBs in the 31-box layout), two passes' corners
      // in flight together (past the last pair a lane has the pair (0, 0),
      // which is none)
      auto list_all = [&](auto& out, int& n, bool near) {
#pragma unroll
        for (int k2 = 0; k2 < PASSES; k2 += 2) {
          if (64 * k2 < n_tri) {
            const Boxes t0 = load_tri(k2);
            if (k2 + 1 < PASSES && 64 * (k2 + 1) < n_tri) {
              const Boxes t1 = load_tri(k2 + 1 < PASSES ? k2 + 1 : k2);
              __builtin_amdgcn_sched_barrier(0);
              list(t0, out, n, near);
              list(t1, out, n, near);
            } else {
              list(t0, out, n, near);
            }
          }
        }
      };
      if constexpr (S::KEEP) {
        // near pair p0 + lane, its pair number in the upper half
        auto numbered = [&](int p0) -> unsigned {
          if (p0 + lane >= n_near) return 0u;
          const unsigned pr = s.near[p0 + lane];
          return pr | (unsigned)number_of(pr >> 8, pr & 255u, n_obj) << 16;
        };
        if constexpr (W > 1) relist_near = __builtin_amdgcn_readfirstlane(s.sh_near) != 0;
        if (relist_near) {
          n_near = 0;
          list_all(s.near, n_near, true);
          wave_sync();
          near0 = numbered(0);
        }
        list(load((near0 >> 8) & 255u, near0 & 255u, near0 >> 16), s.pairs, n_cand, false);
        for (int p0 = 64; p0 < n_near; p0 += 64) {
          const unsigned pr = numbered(p0);
          list(load((pr >> 8) & 255u, pr & 255u, pr >> 16), s.pairs, n_cand, false);
        }
      } else {
        list_all(s.pairs, n_cand, false);
      }
    }

    // ---- 4a. table contacts (body order, corner order): the L lanes of a
    // body test its eight corners, two or four each, and every lane gets the
    // corners within the margin as a byte
    unsigned mask = 0u;
    int nt = 0;                  // the body's table contacts
    int n_table = 0, n_held = 0, n_extra = 0;
    if (lead) {
#pragma unroll
      for (int m = 0; m < 8 / L; ++m) {
        const int kc = j + L * m;
        const float sx = (kc & 1) ? h.x : -h.x, sy = (kc & 2) ? h.y : -h.y, sz = (kc & 4) ? h.z : -h.z;
        const float vz = x.z + (c0.z * sx + c1.z * sy + c2.z * sz);
        if (vz <= p.margin) mask |= 1u << kc;
      }
      mask |= (unsigned)__builtin_amdgcn_mov_dpp((int)mask, Q_XOR1, 0xf, 0xf, true);
      if (L == 4) mask |= (unsigned)__builtin_amdgcn_mov_dpp((int)mask, Q_XOR2, 0xf, 0xf, true);
      mask = active ? mask : 0u;
      nt = __popc(mask);
#pragma unroll
      for (int ts = 0; ts < TS; ++ts) n_held += __popcll(__ballot(j + L * ts < nt));
      n_table = n_held;
      if (__ballot(nt > 4) != 0ull) {
        // boxes flatter than the margin: corners past the fourth become row
        // contacts, the first of the list; the table contacts past the
        // capacity are dropped in list order
        const int off = wave_excl_scan(j == 0 ? nt : 0, &n_table) - (j == 0 ? 0 : nt);
        if (n_table > C) {
          nt = min(max(C - off, 0), nt);
          while (__popc(mask) > nt) mask &= ~(1u << (31 - __clz((int)mask)));
        }
        n_held = 0;
#pragma unroll
        for (int ts = 0; ts < TS; ++ts) n_held += __popcll(__ballot(j + L * ts < nt));
        const int xo = wave_excl_scan(j == 0 ? max(nt - 4, 0) : 0, &n_extra);
        if (first && nt > 4) {
          unsigned m = mask;
          for (int r = 0; m; ++r) {
            const int kc = __builtin_ctz(m);
            m &= m - 1;
            if (r < 4) continue;
            const float sx = (kc & 1) ? h.x : -h.x, sy = (kc & 2) ? h.y : -h.y, sz = (kc & 4) ? h.z : -h.z;
            const f3 vtx = x + mk(c0.x * sx + c1.x * sy + c2.x * sz, c0.y * sx + c1.y * sy + c2.y * sz,
                                  c0.z * sx + c1.z * sy + c2.z * sz);
            const int c = xo + r - 4;
            s.u.n.stage[c][0] = f4(vtx - mk(0, 0, 0.5f * vtx.z), vtx.z);
            s.u.n.stage[c][1] = make_float4(0, 0, 1, 0);
            s.cab[c] = PLANE | (b << 8) | (kc << 16);
          }
        }
      }
    }
    if constexpr (W > 1) {
      // every wave needs the pair list and the table contacts
      if (wid == 1 && lane == 0) s.sh_pairs = n_pairs | n_cand << 16;
      if (lead && lane == 0) {
        s.sh_table = n_table;
        s.sh_held = n_held;
        s.sh_extra = n_extra;
      }
      __syncthreads();
      n_cand = __builtin_amdgcn_readfirstlane(s.sh_pairs);
      n_pairs = n_cand & 0xffff;
      n_cand >>= 16;
      n_table = __builtin_amdgcn_readfirstlane(s.sh_table);
      n_held = __builtin_amdgcn_readfirstlane(s.sh_held);
      n_extra = __builtin_amdgcn_readfirstlane(s.sh_extra);
    } else {
      wave_sync();
    }
    const int row_cap = C - n_held;   // row contacts that fit the capacity
    int n_rows = n_extra;

    // ---- 4b. box-box and pusher-box contacts, candidate pairs in
    // lexicographic order, a pass of four pairs (LP = 16 lanes each) or of eight
    // (LP = 8): lane k evaluates candidate axis k (0-2 faces of A, 3-5 faces of
    // B, 6-14 edge crosses A_i x B_j) and, of eight lanes, axis k + 8; clipping
    // follows only when some pair of the pass has no axis that keeps it apart.
    // With W waves a round is W passes, wave w taking the w-th; the round's
    // contacts keep the order.  Bound by the pass's chain of LDS round trips and
    // dependent instructions: about 1000 cycles of a lone wave for the axes, and
    // 2000 more with a contact to clip, so that listing the pairs that a face
    // axis separates beforehand, eight lanes a pair, takes longer than it saves
    // once those that stay apart are no candidates (700 x 27: 1.38 ms with such a
    // sieve, 1.35 without).
    auto narrow_pass = [&](auto lanes_per_pair, int r0) {
      constexpr int LP = decltype(lanes_per_pair)::value, GROUPS = 64 / LP;
      const int ln = opaque(lane);
      const int grp = ln / LP, gl = ln % LP;
      const int pi = r0 + GROUPS * wid + grp;
      const bool has = pi < n_cand;
      const unsigned pr = has ? s.pairs[pi] : 0u;
      const int ia = pr >> 8, ib = pr & 255;
      const unsigned long long gm = ((1ull << LP) - 1ull) << (LP * grp);
      bool keep = false, face = false;
      f3 P = mk(0, 0, 0), nref = mk(0, 0, 1), n = mk(0, 0, 0);
      float psep = 0.0f, bs = 0.0f;
      int best = -1;
      {
        const Box A = load_box(s, ia), B = load_box(s, ib);
        const f3 d = B.c - A.c;
        struct Candidate {
          f3 L;
          float sv;
          bool edge;   // a usable edge axis
        };
        auto candidate = [&](int k) {
          // axes i of A and j of B by k, two bits each: i 0 1 2 - - - 0 0 0 1
          // 1 1 2 2 2 -, j - - - 0 1 2 0 1 2 0 1 2 0 1 2 -
          const f3 ua = lds_axis(s, ia, (0x2a540024u >> (2 * k)) & 3u);
          const f3 ub = lds_axis(s, ib, (0x24924900u >> (2 * k)) & 3u);
          const f3 v = cross(ua, ub);
          const float l2 = dot(v, v);
          const f3 L = sel(k < 3, ua, sel(k < 6, ub, v * rsq(l2)));
          return Candidate{L, fabsf(dot(d, L)) - radius_along(A, L) - radius_along(B, L),
                           k >= 6 && k < 15 && l2 >= p.edge_eps * p.edge_eps};
        };
        const Candidate q0 = candidate(gl), q1 = LP == 8 ? candidate(gl + 8) : q0;
        const bool over = ((gl < 6 || q0.edge) && q0.sv > p.margin) || (LP == 8 && q1.edge && q1.sv > p.margin);
        const bool out = (__ballot(over) & gm) != 0ull;
        // the contact axis: the candidates in order, the kept one replaced
        // only by a later one that exceeds it by tau_face (faces) or tau_edge
        // (edges); the edges are gone through only when one exceeds the
        // faces' choice
        bs = group_value<LP, 0>(q0.sv);
        best = 0;
        auto scan = [&](float sk, int k, float tau) {
          if (sk > bs + tau) {
            bs = sk;
            best = k;
          }
        };
        scan(group_value<LP, 1>(q0.sv), 1, p.tau_face);
        scan(group_value<LP, 2>(q0.sv), 2, p.tau_face);
        scan(group_value<LP, 3>(q0.sv), 3, p.tau_face);
        scan(group_value<LP, 4>(q0.sv), 4, p.tau_face);
        scan(group_value<LP, 5>(q0.sv), 5, p.tau_face);
        // a face axis keeps the boxes apart for a while (but the first
        // substep's orientations may not be unit quaternions yet)
        if (has && gl == 0 && bs > gap0 && k > 0)
          s.apart[number_of(ia, ib, n_obj)] = apart_until(bs, s.pos[ia].w + s.pos[ib].w);
        const float least = bs + p.tau_edge;
        if (__ballot(has && ((q0.edge && q0.sv > least) || (LP == 8 && q1.edge && q1.sv > least))) != 0ull) {
          const float e0 = q0.edge ? q0.sv : -INFINITY, e1 = LP == 8 ? (q1.edge ? q1.sv : -INFINITY) : e0;
          scan(group_value<LP, 6>(e0), 6, p.tau_edge);
          scan(group_value<LP, 7>(e0), 7, p.tau_edge);
          scan(group_value<LP, 8 % LP>(e1), 8, p.tau_edge);
          scan(group_value<LP, 9 % LP>(e1), 9, p.tau_edge);
          scan(group_value<LP, 10 % LP>(e1), 10, p.tau_edge);
          scan(group_value<LP, 11 % LP>(e1), 11, p.tau_edge);
          scan(group_value<LP, 12 % LP>(e1), 12, p.tau_edge);
          scan(group_value<LP, 13 % LP>(e1), 13, p.tau_edge);
          scan(group_value<LP, 14 % LP>(e1), 14, p.tau_edge);
        }
        // every lane of the group takes the kept axis from its lane, pointing from A to B
        const int from = ((ln & (64 - LP)) + best % LP) << 2;
        auto take = [&](float x) {
          return __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(x)));
        };
        const f3 Lo = LP == 8 ? sel(best < 8, q0.L, q1.L) : q0.L;
        const f3 Lb = mk(take(Lo.x), take(Lo.y), take(Lo.z));
        if (!has || out) best = -1;
        else n = sel(dot(d, Lb) >= 0.0f, Lb, neg(Lb));
      }
      if (__ballot(best >= 0) != 0ull) {
        // face axis: reference face of the axis owner, incident face of the
        // other box (most anti-parallel, ties to +x, -x, +y, -y, +z, -z), its
        // four corners one per lane, clipped by the reference face's side
        // planes +u, -u, +v, -v
        face = best >= 0 && best < 6;
        f3 fref = mk(0, 0, 0), u = mk(1, 0, 0), w = mk(0, 1, 0);
        float hu = 0.0f, hw = 0.0f;
        int np = 0;
        if (face) {
          const bool a_ref = best < 3;
          const int k = a_ref ? best : best - 3;
          const int ku = k == 2 ? 0 : k + 1, kv = k == 0 ? 2 : k - 1;
          // reference box ir (the axis owner) and incident box ii, read from
          // LDS at the indices found (no selects over both boxes' registers)
          const int ir = a_ref ? ia : ib, ii = a_ref ? ib : ia;
          const float* const hr = reinterpret_cast<const float*>(&s.half[ir]);
          nref = sel(a_ref, n, neg(n));
          fref = xyz(s.pos[ir]) + nref * hr[k];
          u = lds_axis(s, ir, ku);
          w = lds_axis(s, ir, kv);
          hu = hr[ku];
          hw = hr[kv];
          const f3 i0 = lds_axis(s, ii, 0), i1 = lds_axis(s, ii, 1), i2 = lds_axis(s, ii, 2);
          const f3 ic = xyz(s.pos[ii]);
          const float c0 = dot(i0, nref), c1 = dot(i1, nref), c2 = dot(i2, nref);
          int fb = 0;
          float bd = c0;
          if (-c0 < bd) { bd = -c0; fb = 1; }
          if (c1 < bd) { bd = c1; fb = 2; }
          if (-c1 < bd) { bd = -c1; fb = 3; }
          if (c2 < bd) { bd = c2; fb = 4; }
          if (-c2 < bd) { bd = -c2; fb = 5; }
          const int m = fb >> 1, mp = m == 2 ? 0 : m + 1, mq = m == 0 ? 2 : m - 1;
          const float sg = (fb & 1) ? -1.0f : 1.0f;
          const float* const hi = reinterpret_cast<const float*>(&s.half[ii]);
          const f3 am = lds_axis(s, ii, m), ap = lds_axis(s, ii, mp), aq = lds_axis(s, ii, mq);
          const float hm = hi[m], hp = hi[mp], hq = hi[mq];
          const f3 fc = ic + am * (sg * hm);
          const f3 ep = ap * hp, eq = aq * hq;
          // corner gl of the incident face: signs (+,+), (-,+), (-,-), (+,-) of
          // its two half edges (the lanes from 4 on repeat corner 3); a product with +-1
          // is exact, so each sum rounds once as a plain sum or difference
          const float spp = (gl == 1 || gl == 2) ? -1.0f : 1.0f, sqq = gl >= 2 ? -1.0f : 1.0f;
          P = fc + (ep * spp + eq * sqq);
          np = 4;
        }
        np = clip_group<LP>(s, &P, np, fref, u, 1.0f, hu, 0, grp, gl, lane, wid);
        np = clip_group<LP>(s, &P, np, fref, u, -1.0f, hu, 1, grp, gl, lane, wid);
        np = clip_group<LP>(s, &P, np, fref, w, 1.0f, hw, 0, grp, gl, lane, wid);
        np = clip_group<LP>(s, &P, np, fref, w, -1.0f, hw, 1, grp, gl, lane, wid);
        // contacts: kept polygon points (face) or one edge-edge point
        psep = dot(nref, P - fref);
        keep = face ? (gl < np && psep <= p.margin) : (best >= 6 && gl == 0);
      }
      const unsigned long long km = __ballot(keep);
      const unsigned long long below = (1ull << lane) - 1ull;
      int before = 0, round_total = __popcll(km);
      if constexpr (W > 1) {
        // kept contacts of every wave's pass: the earlier passes come first
        const int par = (r0 / (GROUPS * W)) & 1;
        if (lane == 0) s.rcount[par][wid] = round_total;
        __syncthreads();
        round_total = 0;
#pragma unroll
        for (int w2 = 0; w2 < W; ++w2) {
          const int m = s.rcount[par][w2];
          before += w2 < wid ? m : 0;
          round_total += m;
        }
      }
      const int off = n_rows + before + __popcll(km & below);
      if (keep && off < row_cap) {
        const int ab = ia | (ib << 8);
        if (face) {
          s.u.n.stage[off][0] = f4(P - nref * (0.5f * psep), psep);
          s.u.n.stage[off][1] = f4(n, 0.0f);
          s.cab[off] = ab | (__popcll(km & below & gm) << 16);
        } else {
          s.u.n.stage[off][0] = f4(edge_point(s, ia, ib, best, n), bs);
          s.u.n.stage[off][1] = f4(n, 0.0f);
          s.cab[off] = ab;
        }
      }
      n_rows += round_total;
    };
    // Up to one pass of sixteen lanes a pair per wave takes that, the shorter
    // chain (4096 x 15 1.66 ms, 1.70 with eight lanes always); more go eight to
    // a pass, which takes hardly longer (60 substeps of 1024 x 8 touching cubes,
    // 16 pairs: 1.12 -> 0.95 ms; 1024 x 30 in a pile, 138: 14.8 -> 11.6; 700 x 27
    // 1.33 -> 1.24).
    if (n_cand > 4 * W)
      for (int r0 = 0; r0 < n_cand; r0 += 8 * W) narrow_pass(std::integral_constant<int, 8>{}, r0);
    else if (n_cand > 0)
      narrow_pass(std::integral_constant<int, 16>{}, 0);
    const int nc_raw = n_table + n_rows - n_extra;
    if (nc_raw > C) {
      status |= PMBS_ENV_CONTACT_OVERFLOW;
      if (g.overflow_list) {
        // nothing of this env has been written yet: hand it to a larger class
        deferred = true;
        break;
      }
    }
    const int nc = nc_raw < C ? nc_raw : C;
    n_rows = n_rows < row_cap ? n_rows : row_cap;
    if constexpr (W > 1) n_rows = __builtin_amdgcn_readfirstlane(n_rows);
    if constexpr (RUN == Run::COST) {
      // The work estimate of the env's push from its start pose; nothing else
      // is written.  A substep with row contacts costs about 2.6 times one
      // without (the solver's ten iterations through LDS and a live
      // narrowphase pass), so what counts is for how many of them there are
      // row contacts: all, when there are some at the start; else from where
      // the pusher, moving straight on, meets the first box.  Measured per env
      // at 4096 x 15 (alone on a SIMD, us): 339 +- 23 without row contacts, 915
      // +- 75 with them throughout; a key of contacts, pairs and validity ranked
      // the envs with a correlation of 0.48 to these times, and the batch
      // ended with heavy envs that had started last (2.07 ms).
      float from = n_rows > 0 ? 0.0f : (float)n_sub;   // first substep with row contacts
      if (valid && n_rows == 0 && lane < nb) {
        const Box B = load_box(s, lane);
        const f3 side = mk(-pdir.y, pdir.x, 0.0f), d = B.c - xp;
        if (fabsf(dot(d, side)) <= radius_along(B, side) + p.phy && dot(d, pdir) > 0.0f) {
          const float way = fmaxf(dot(d, pdir) - radius_along(B, pdir) - p.phx - p.margin, 0.0f);
          const float k_hit = way * p.inv_dt / p.push_speed;
          if (k_hit <= (float)n_move) from = fminf(from, k_hit);
        }
      }
      for (int o = 32; o > 0; o >>= 1) from = fminf(from, __shfl_xor(from, o, 64));
      // in units of 1/120 of such a substep-long push's extra work
      const int key = (int)(120.0f * (1.0f - from / (float)n_sub)) + 4 * n_rows + n_pairs;
      if (lead && lane == 0) g.cost_key[e] = key;
      return;
    }
    stat_nc += nc;
    stat_pairs += n_pairs;
    stat_sub += 1;
    sync_all<W>();   // every wave's contacts are in the staging array
    x = xyz(s.pos[bl]);
    h = xyz(s.half[bl]);
    c0 = xyz(s.col[0][bl]);
    c1 = xyz(s.col[1][bl]);
    c2 = xyz(s.col[2][bl]);

    if constexpr (RUN == Run::COLLIDE) {
      // the whole list: table contacts at their rank, then the staged pairs
      float* out = g.dbg_contacts + (size_t)e * C * 9;
      auto put = [&](int c, int a, int bb, f3 pt, f3 n, float sep) {
        out[c * 9 + 0] = a == PLANE ? -1.0f : (float)a;
        out[c * 9 + 1] = (float)bb;
        out[c * 9 + 2] = pt.x; out[c * 9 + 3] = pt.y; out[c * 9 + 4] = pt.z;
        out[c * 9 + 5] = n.x; out[c * 9 + 6] = n.y; out[c * 9 + 7] = n.z;
        out[c * 9 + 8] = sep;
      };
      if (lead) {
        int tot;
        const int off = wave_excl_scan(j == 0 ? nt : 0, &tot);
        const int off_b = off - (j == 0 ? 0 : nt);
        if (active) {   // lane j the body's contacts j, j + L, ...
          int c = off_b;
          for (unsigned m = mask; m; m &= m - 1, ++c) {
            if ((c - off_b) % L != j) continue;
            const int kc = __builtin_ctz(m);
            const float sx = (kc & 1) ? h.x : -h.x, sy = (kc & 2) ? h.y : -h.y, sz = (kc & 4) ? h.z : -h.z;
            const f3 vtx = x + mk(c0.x * sx + c1.x * sy + c2.x * sz, c0.y * sx + c1.y * sy + c2.y * sz,
                                  c0.z * sx + c1.z * sy + c2.z * sz);
            put(c, PLANE, b, vtx - mk(0, 0, 0.5f * vtx.z), mk(0, 0, 1), vtx.z);
          }
        }
        for (int c = n_extra + lane; c < n_rows; c += 64) {
          const float4 s0 = s.u.n.stage[c][0], s1 = s.u.n.stage[c][1];
          const int ab = s.cab[c];
          put(tot + c - n_extra, ab & 255, (ab >> 8) & 255, xyz(s0), xyz(s1), s0.w);
        }
        if (lane == 0) {
          g.dbg_count[e] = nc;
          g.env_status[e] = status;
        }
      }
      return;
    }

    // The rest of the substep is the lead wave's, but for the row contacts that
    // the second wave prepares and updates while the lead updates its lanes'
    // table contacts.  Up to 16 of them it takes in quads, in the 31-box layout
    // (22 objects: 1100 -> 1000 cycles an iteration; rollouts of 256 x 21 6.10 ->
    // 5.94 ms); with one table contact per lane, as in the 16-box layout, two
    // barriers an iteration cost what the split gives (1024 x 15, two waves a
    // SIMD: 1.12 -> 1.14 ms): no split there.  Of more than 16 it takes every
    // second slot of 64, the first among them.
    const bool split = W > 1 && (n_rows > 16 || (SPLIT && n_rows > 0));
    if (row_wave) {
      if constexpr (W > 1) if (split) {
        const int lane = opaque(threadIdx.x & 63);
        __syncthreads();   // the bodies' data and the contact counts
        if (n_rows > 16) {
          solve_rows<0, 2>(s, lane, n_rows, nwarm, n_extra, p, []() { __syncthreads(); }, []() {},
                                  []() { __syncthreads(); }, []() {});
        } else if constexpr (SPLIT) {
          QuadContact qc = begin_quad(s, lane, n_rows, nwarm, n_extra, p);
          wave_sync();
          put_quad(s, lane, qc, qc.lam);
          __syncthreads();
          for (int it = 0; it < p.iters; ++it) {
            __syncthreads();   // the iteration-start velocities
            put_quad(s, lane, qc, update_quad(s, qc, []() {}));
            __syncthreads();   // the impulse rows
          }
          keep_quad(s, lane, n_rows, qc);
        }
      }
      if constexpr (W > 1) nwarm = n_rows;
    } else {
    // world inverse inertia Iw^-1 = R diag(invI) R^T: diagonal, off-diagonal (xy, xz, yz)
    f3 md, mo;
    {
      const float r00 = c0.x, r01 = c1.x, r02 = c2.x;
      const float r10 = c0.y, r11 = c1.y, r12 = c2.y;
      const float r20 = c0.z, r21 = c1.z, r22 = c2.z;
      md.x = r00 * invI.x * r00 + r01 * invI.y * r01 + r02 * invI.z * r02;
      md.y = r10 * invI.x * r10 + r11 * invI.y * r11 + r12 * invI.z * r12;
      md.z = r20 * invI.x * r20 + r21 * invI.y * r21 + r22 * invI.z * r22;
      mo.x = r00 * invI.x * r10 + r01 * invI.y * r11 + r02 * invI.z * r12;
      mo.y = r00 * invI.x * r20 + r01 * invI.y * r21 + r02 * invI.z * r22;
      mo.z = r10 * invI.x * r20 + r11 * invI.y * r21 + r12 * invI.z * r22;
    }
    // ---- 5. per-body lists of row contacts in contact-index order (CSR):
    // every row contact sets its bit in the masks of its two bodies; a
    // body's list length is its bit count; every contact then writes itself
    // at its rank among the set bits.  Kept from the previous substep when
    // neither the row contacts' keys nor any body's corners changed.
    const int lane = opaque(threadIdx.x & 63);
    const int nh = nt < 4 ? nt : 4;   // the body's contacts in its lanes: the first of its list
    const bool moved = __ballot(mask != corners) != 0ull;   // some body's corner set changed
    if (n_rows > 0) {
      bool same_list = n_rows == nwarm && !moved;
      if (same_list) {
        bool diff = false;
#pragma unroll
        for (int sl = 0; sl < K; ++sl) {
          const int c = 64 * sl + lane;
          if (c < n_rows) diff = diff || contact_key<S>(s.cab[c]) != s.wkey[c];
        }
        same_list = __ballot(diff) == 0ull;
      }
      if (!same_list) {
        constexpr int MW = 2 * K;  // mask words per body: slot sl, lane half
        unsigned* const im = &s.u.n.x.incm[0][0];
        for (int i = lane; i < S::NOBJ * MW; i += 64) im[i] = 0u;
        wave_sync();
        int ca[K], cb[K];
        const unsigned bit = 1u << (lane & 31);
#pragma unroll
        for (int sl = 0; sl < K; ++sl) {
          const int c = 64 * sl + lane;
          const int ab = c < n_rows ? s.cab[c] : -1;
          ca[sl] = c < n_rows && (ab & 255) < nb ? (ab & 255) : -1;
          cb[sl] = c < n_rows && ((ab >> 8) & 255) < nb ? ((ab >> 8) & 255) : -1;
          const int wd = 2 * sl + (lane >> 5);
          if (ca[sl] >= 0) atomicOr(&s.u.n.x.incm[ca[sl]][wd], bit);
          if (cb[sl] >= 0) atomicOr(&s.u.n.x.incm[cb[sl]][wd], bit);
        }
        wave_sync();
        n_inc = 0;
        if (active) {
#pragma unroll
          for (int wd = 0; wd < MW; ++wd) n_inc += __popc(s.u.n.x.incm[b][wd]);
        }
        int tot;
        inc0 = wave_excl_scan(j == 0 ? n_inc : 0, &tot) - (j == 0 ? 0 : n_inc);
        if (first) {
          s.cnt[b] = nh + n_inc;
          s.lstart[b] = inc0;
        }
        wave_sync();
#pragma unroll
        for (int sl = 0; sl < K; ++sl) {
          const int c = 64 * sl + lane;
          const int wd = 2 * sl + (lane >> 5);
#pragma unroll
          for (int side = 0; side < 2; ++side) {
            const int jb = side ? cb[sl] : ca[sl];
            if (jb >= 0) {
              int r = s.lstart[jb] + __popc(s.u.n.x.incm[jb][wd] & (bit - 1u));
#pragma unroll
              for (int w2 = 0; w2 < MW; ++w2)
                if (w2 < wd) r += __popc(s.u.n.x.incm[jb][w2]);
              s.inc[r] = (unsigned short)(((unsigned)c * 16u) | side);
            }
          }
        }
      }
      // the bodies' data that the row contacts read
      if (first && n_inc > 0) {
        s.iwa[b] = make_float4(md.x, md.y, md.z, mo.x);
        s.iwb[b] = make_float4(mo.y, mo.z, mu, 0.0f);
      }
    } else {
      n_inc = 0;
    }
    // a corner set that changed, or table contacts among the rows: last
    // substep's table impulses go through LDS (once per change; a resting or
    // sliding box keeps its corners for many substeps)
    const bool relist = moved || n_extra > 0;
    if (relist) {
      wave_sync();
#pragma unroll
      for (int ts = 0; ts < TS; ++ts)
        if (active)
          s.u.n.x.lam[4 * b + j + L * ts] = make_float4(tc[ts].ln, tc[ts].lt1, tc[ts].lt2, __int_as_float((int)corners));
      wave_sync();
#pragma unroll
      for (int ts = 0; ts < TS; ++ts) {
        const int i = j + L * ts;   // the lane's contact: corner number i of the set
        unsigned m = mask;
#pragma unroll
        for (int r = 0; r < 3; ++r) m = r < i ? m & (m - 1u) : m;
        kk[ts] = m ? __builtin_ctz(m) : 0;
        tc[ts].ln = tc[ts].lt1 = tc[ts].lt2 = 0.0f;
        if (i < nt && (corners >> kk[ts] & 1u)) {
          const int o = __popc(corners & ((1u << kk[ts]) - 1u));
          if (o < 4) {
            const float4 l = s.u.n.x.lam[4 * b + o];
            tc[ts].ln = l.x;
            tc[ts].lt1 = l.y;
            tc[ts].lt2 = l.z;
          } else {
            const int wi = warm_index(s, (b << 8) | kk[ts], nwarm);
            if (wi >= 0) {
              tc[ts].ln = s.wl[0][wi];
              tc[ts].lt1 = s.wl[1][wi];
              tc[ts].lt2 = s.wl[2][wi];
            }
          }
        }
      }
      corners = mask;
    }

    if constexpr (W > 1)
      if (split) __syncthreads();   // to the row wave

    // ---- 6. prep of the lanes' table contacts (an absent one has zero
    // masses, so its impulses stay zero)
    const float cbn = (float)(nh + n_inc);
#pragma unroll
    for (int ts = 0; ts < TS; ++ts) {
      TableContact& q = tc[ts];
      const bool on = j + L * ts < nt;
      const int kc = kk[ts];
      const float sx = (kc & 1) ? h.x : -h.x, sy = (kc & 2) ? h.y : -h.y, sz = (kc & 4) ? h.z : -h.z;
      const f3 vtx = x + mk(c0.x * sx + c1.x * sy + c2.x * sz, c0.y * sx + c1.y * sy + c2.y * sz,
                            c0.z * sx + c1.z * sy + c2.z * sz);
      const f3 pt = vtx - mk(0, 0, 0.5f * vtx.z);
      const float sep = vtx.z;
      q.rb = pt - x;
      const f3 em = table_masses(q.rb, md, mo);
      q.kn = on ? rcp(cbn * (invm + em.x)) : 0.0f;
      q.kt1 = on ? rcp(cbn * (invm + em.y)) : 0.0f;
      q.kt2 = on ? rcp(cbn * (invm + em.z)) : 0.0f;
      q.vstar = sep > 0.0f ? -sep * p.inv_dt : p.beta * fmaxf(-sep - p.slop, 0.0f) * p.inv_dt;
    }
    // ---- 7. projected Jacobi, I iterations.  A body's velocity changes by M
    // times the sum of its contacts' impulses (M: inverse mass, world inverse
    // inertia), added as two partial sums over the even and the odd entries of its
    // contact list, each in list order: lanes j of even and odd parity hold
    // them, the table contacts' terms first (entries 0-3), then the rows.
    f3 P[TS];
    auto row_at = [&](unsigned off) {
      return xyz(*reinterpret_cast<const float4*>(reinterpret_cast<const char*>(&s.u.imp[0][0]) + off));
    };
    auto add_signed = [](f3 a, float sg, f3 val) {
      return mk(fmaf(sg, val.x, a.x), fmaf(sg, val.y, a.y), fmaf(sg, val.z, a.z));
    };
    auto apply = [&](f3 lin, f3 ang) {
      v = mk(fmaf(invm, lin.x, v.x), fmaf(invm, lin.y, v.y), fmaf(invm, lin.z, v.z));
      w = mk(fmaf(md.x, ang.x, fmaf(mo.x, ang.y, fmaf(mo.y, ang.z, w.x))),
             fmaf(mo.x, ang.x, fmaf(md.y, ang.y, fmaf(mo.z, ang.z, w.y))),
             fmaf(mo.y, ang.x, fmaf(mo.z, ang.y, fmaf(md.z, ang.z, w.z))));
    };
    // the table contacts' terms of the lane's parity
    auto table_sums = [&](f3* lin, f3* ang) {
      if constexpr (L == 4) {
        const f3 T = cross(tc[0].rb, P[0]);
        *lin = P[0] + quad<Q_XOR2>(P[0]);
        *ang = T + quad<Q_XOR2>(T);
      } else {
        *lin = P[0] + P[TS - 1];
        *ang = cross(tc[0].rb, P[0]) + cross(tc[TS - 1].rb, P[TS - 1]);
      }
    };
    // an update in two halves: the new impulses up to the friction disc's
    // root, and the rest
    float t_ln[TS], t_lt1[TS], t_lt2[TS], t_root[TS];
    auto table_begin = [&]() {
#pragma unroll
      for (int ts = 0; ts < TS; ++ts) {
        const TableContact& q = tc[ts];
        const f3 u = cross_add(w, q.rb, v);
        t_ln[ts] = fmaxf(q.ln + q.kn * (q.vstar - u.z), 0.0f);
        t_lt1[ts] = q.lt1 + q.kt1 * u.y;
        t_lt2[ts] = q.lt2 - q.kt2 * u.x;
        t_root[ts] = rsq(t_lt1[ts] * t_lt1[ts] + t_lt2[ts] * t_lt2[ts]);
      }
    };
    auto table_end = [&]() {
#pragma unroll
      for (int ts = 0; ts < TS; ++ts) {
        TableContact& q = tc[ts];
        // onto the friction disc: scale by min(1, lim / |lt|) (a zero
        // tangential impulse gives inf or nan, and the min keeps 1)
        const float lim = mu_table * t_ln[ts];
        const float sc = fminf(lim * t_root[ts], 1.0f);
        const float lt1 = t_lt1[ts] * sc, lt2 = t_lt2[ts] * sc;
        P[ts] = mk(lt2 - q.lt2, q.lt1 - lt1, t_ln[ts] - q.ln);
        q.ln = t_ln[ts];
        q.lt1 = lt1;
        q.lt2 = lt2;
      }
    };
    auto table_update = [&]() {
      table_begin();
      table_end();
    };
#pragma unroll
    for (int ts = 0; ts < TS; ++ts) P[ts] = mk(tc[ts].lt2, -tc[ts].lt1, tc[ts].ln);
    if (n_rows == 0) {
      // table contacts alone: every body by itself, nothing through LDS
      auto sums = [&]() {
        f3 lin, ang;
        table_sums(&lin, &ang);
        apply(lin + quad<Q_XOR1>(lin), ang + quad<Q_XOR1>(ang));
      };
      sums();
      // two per trip: the new impulses of one are the next one's old ones
      // without copies
      int it = 0;
      for (; it + 1 < p.iters; it += 2) {
        table_update();
        sums();
        table_update();
        sums();
      }
      if (it < p.iters) {
        table_update();
        sums();
      }
    } else {
      // the lane's entries of its body's list: parity j & 1; with four lanes
      // per body lanes 0 and 1 add the linear rows and lanes 2 and 3 the
      // angular ones, with two lanes both.  The first four entries stay in
      // registers as row offsets and signs; one past the end of the list
      // points at the zero row, whose term (-1 times +0) changes no sum.
      constexpr int RG = 4;
      const unsigned zrow = (unsigned)(reinterpret_cast<const char*>(&s.zero) - reinterpret_cast<const char*>(&s.u.imp[0][0]));
      static_assert(sizeof(s.u) + sizeof(float4) <= 0x10000, "impulse rows and the zero row need 16-bit codes");
      const bool ang_lane = L == 4 && j >= 2;
      const int k0 = (j ^ nh) & 1;
      unsigned radr[RG], rada[L == 2 ? RG : 1];
      float rsg[RG];
      auto row_lin = [&](unsigned code) { return code & 0xfffeu; };
      auto row_ang = [&](unsigned code) { return (code & 0xfffeu) + (1u + (code & 1u)) * (unsigned)(C * 16); };
#pragma unroll
      for (int u = 0; u < RG; ++u) {
        const int i = k0 + 2 * u;
        const bool in = i < n_inc;
        const unsigned code = in ? s.inc[inc0 + i] : 0u;
        rsg[u] = in && (code & 1u) ? 1.0f : -1.0f;
        radr[u] = in ? (ang_lane ? row_ang(code) : row_lin(code)) : zrow;
        if constexpr (L == 2) rada[u] = in ? row_ang(code) : zrow;
      }
      const bool rows2 = __ballot(n_inc > k0 + 4) != 0ull;   // some lane has a third entry
      const bool rows4 = __ballot(n_inc > k0 + 2 * RG) != 0ull;
      auto sums = [&]() {
        f3 lin, ang;
        if constexpr (L == 4) {
          const f3 r0 = row_at(radr[0]), r1 = row_at(radr[1]);
          __builtin_amdgcn_sched_barrier(0);
          table_sums(&lin, &ang);   // while the loads are in flight
          f3 a = sel(ang_lane, ang, lin);
          a = add_signed(a, rsg[0], r0);
          a = add_signed(a, rsg[1], r1);
          if (rows2) {
            const f3 r2 = row_at(radr[2]), r3 = row_at(radr[3]);
            a = add_signed(a, rsg[2], r2);
            a = add_signed(a, rsg[3], r3);
            if (rows4)
              for (int i = k0 + 2 * RG; i < n_inc; i += 2) {
                const unsigned code = s.inc[inc0 + i];
                a = add_signed(a, (code & 1u) ? 1.0f : -1.0f, row_at(ang_lane ? row_ang(code) : row_lin(code)));
              }
          }
          a = a + quad<Q_XOR1>(a);
          apply(quad<Q_LOW>(a), quad<Q_HIGH>(a));
        } else {
          const f3 r0 = row_at(radr[0]), r1 = row_at(radr[1]), t0 = row_at(rada[0]), t1 = row_at(rada[1]);
          __builtin_amdgcn_sched_barrier(0);
          table_sums(&lin, &ang);
          lin = add_signed(lin, rsg[0], r0);
          lin = add_signed(lin, rsg[1], r1);
          ang = add_signed(ang, rsg[0], t0);
          ang = add_signed(ang, rsg[1], t1);
          if (rows2) {
            const f3 r2 = row_at(radr[2]), r3 = row_at(radr[3]), t2 = row_at(rada[2]), t3 = row_at(rada[3]);
            lin = add_signed(lin, rsg[2], r2);
            lin = add_signed(lin, rsg[3], r3);
            ang = add_signed(ang, rsg[2], t2);
            ang = add_signed(ang, rsg[3], t3);
            if (rows4)
              for (int i = k0 + 2 * RG; i < n_inc; i += 2) {
                const unsigned code = s.inc[inc0 + i];
                const float sg = (code & 1u) ? 1.0f : -1.0f;
                lin = add_signed(lin, sg, row_at(row_lin(code)));
                ang = add_signed(ang, sg, row_at(row_ang(code)));
              }
          }
          apply(lin + quad<Q_XOR1>(lin), ang + quad<Q_XOR1>(ang));
        }
      };
      // lane 0 of a body with row contacts publishes its linear, lane 1 its
      // angular velocity (as y, z, x, y: components q + 1 and q + 2 adjacent)
      float4* const vslot = j == 0 ? &s.vel[b < MB ? b : 0] : &s.ang[b < MB ? b : 0];
      const bool publisher = active && j < 2 && n_inc > 0;
      auto publish = [&]() {
        if (publisher) *vslot = j == 0 ? make_float4(v.x, v.y, v.z, 0.0f) : make_float4(w.y, w.z, w.x, w.y);
        wave_sync();   // the iteration-start velocities
      };
      // The row contacts' prep, then their warm start: the impulses carried
      // over from the previous substep (the impulse rows share LDS with the
      // staging array that the prep reads).  Up to 16 take a quad of lanes
      // each, more a lane each: most environments have none or a few, and a
      // quad's lanes share the three rows of an update (38 instructions
      // instead of 61, and a third of the prep's masses).
      wave_sync();
      if (n_rows <= 16) {
        if constexpr (SPLIT) {
          __syncthreads();   // the rows of the impulses carried over
          sums();
          for (int it = 0; it < p.iters; ++it) {
            publish();
            __syncthreads();
            // between the barriers, while the row wave is busy: the compiler
            // would move register work to either side of them
            hold(v);
            hold(w);
            table_update();
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) hold(P[ts]);
            __syncthreads();
            sums();
          }
        } else {
          QuadContact qc = begin_quad(s, lane, n_rows, nwarm, n_extra, p);
          wave_sync();
          put_quad(s, lane, qc, qc.lam);
          wave_sync();
          sums();
          for (int it = 0; it < p.iters; ++it) {
            publish();
            const float dl = update_quad(s, qc, [&]() {
              __builtin_amdgcn_sched_barrier(0);
              table_begin();   // while the loads are in flight
              __builtin_amdgcn_sched_barrier(0);
              table_end();     // between the steps of the rows' chain
            });
            put_quad(s, lane, qc, dl);
            wave_sync();   // the impulse rows
            sums();
          }
          keep_quad(s, lane, n_rows, qc);
        }
      } else {
        // the same sums where a body has many rows: its lane's first 12 entries
        // stay in registers, a row's offset and bit 0 for a term to subtract, and
        // are loaded in groups, all of a group in flight together (18 rows a body:
        // 2000 -> 1000 cycles against one entry after the other).  In the
        // 512-contact class, that of piles, 16 (1024 x 16 in a pile, 20 rows a
        // body: 5.80 -> 5.65 ms; towers with 8 a body 1 to 2 % slower).
        constexpr int E = K == 8 ? 16 : 12, G = 4;
        unsigned entry[E];
        bool group[E / G];   // some lane has an entry in the group
#pragma unroll
        for (int u = 0; u < E; ++u) {
          if (u % G == 0) group[u / G] = __ballot(n_inc > k0 + 2 * u) != 0ull;
          entry[u] = zrow | 1u;
          if (group[u / G]) {
            const int i = k0 + 2 * u;
            const unsigned code = s.inc[i < n_inc ? inc0 + i : 0];
            if (i < n_inc) entry[u] = (ang_lane ? row_ang(code) : row_lin(code)) | (~code & 1u);
          }
        }
        const bool longer = __ballot(n_inc > k0 + 2 * E) != 0ull;
        auto sums_many = [&]() {
          f3 lin, ang, a;
          f3 r[G], t[L == 2 ? G : 1];
          auto load = [&](int u0) {
#pragma unroll
            for (int u = 0; u < G; ++u) {
              const unsigned off = entry[u0 + u] & ~1u;
              r[u] = row_at(off);
              if constexpr (L == 2)
                t[u] = row_at(off == zrow ? zrow : off + (2u - (entry[u0 + u] & 1u)) * (unsigned)(C * 16));
            }
          };
          auto add = [&](int u0) {
#pragma unroll
            for (int u = 0; u < G; ++u) {
              const float sg = __uint_as_float(0x3f800000u | entry[u0 + u] << 31);
              if constexpr (L == 4) {
                a = add_signed(a, sg, r[u]);
              } else {
                lin = add_signed(lin, sg, r[u]);
                ang = add_signed(ang, sg, t[u]);
              }
            }
          };
          load(0);
          __builtin_amdgcn_sched_barrier(0);
          table_sums(&lin, &ang);   // while the loads are in flight
          a = sel(ang_lane, ang, lin);
          add(0);
#pragma unroll
          for (int u0 = G; u0 < E; u0 += G)
            if (group[u0 / G]) {
              load(u0);
              add(u0);
            }
          if (longer)
            for (int i = k0 + 2 * E; i < n_inc; i += 2) {
              const unsigned code = s.inc[inc0 + i];
              const float sg = (code & 1u) ? 1.0f : -1.0f;
              if constexpr (L == 4) {
                a = add_signed(a, sg, row_at(ang_lane ? row_ang(code) : row_lin(code)));
              } else {
                lin = add_signed(lin, sg, row_at(row_lin(code)));
                ang = add_signed(ang, sg, row_at(row_ang(code)));
              }
            }
          if constexpr (L == 4) {
            a = a + quad<Q_XOR1>(a);
            apply(quad<Q_LOW>(a), quad<Q_HIGH>(a));
          } else {
            apply(lin + quad<Q_XOR1>(lin), ang + quad<Q_XOR1>(ang));
          }
        };
        if constexpr (W == 1) {
          solve_rows<0, 1>(s, lane, n_rows, nwarm, n_extra, p, []() { wave_sync(); }, sums_many, publish, table_update);
        } else {
          solve_rows<1, 2>(s, lane, n_rows, nwarm, n_extra, p, []() { __syncthreads(); }, sums_many, [&]() {
            publish();
            __syncthreads();
            hold(v);   // as above
            hold(w);
          }, [&]() {
            table_update();
#pragma unroll
            for (int ts = 0; ts < TS; ++ts) hold(P[ts]);
          });
        }
      }
    }
    nwarm = n_rows;

    // ---- 8. position stage
    x = fma3(v, dt, xyz(s.pos[bl]));
    {
      const float4 q = s.quat[bl];
      q0 = q.x;
      q1 = q.y;
      q2 = q.z;
      q3 = q.w;
      float dw = -(w.x * q1 + w.y * q2 + w.z * q3);
      float dx = q0 * w.x + (w.y * q3 - w.z * q2);
      float dy = q0 * w.y + (w.z * q1 - w.x * q3);
      float dz = q0 * w.z + (w.x * q2 - w.y * q1);
      float hd = 0.5f * dt;
      q0 += hd * dw; q1 += hd * dx; q2 += hd * dy; q3 += hd * dz;
      const float il = rsq(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
      q0 *= il; q1 *= il; q2 *= il; q3 *= il;
    }
    }  // lead
    xp = fma3(vp, dt, xp);
    wave_sync();
  }
  if (deferred) break;

  if (rollout) {
    // ---- reward after the push: clearance of the target's footprint, by
    // every wave from the frames in LDS (the same stopping decision); the L
    // lanes of a body share its vertices
    write_body_frames(b, first, 0.0f);
    sync_all<W>();
    const int tg = g.target[e];
    const int lane = opaque(threadIdx.x & 63), b = (unsigned)lane / L, j = (unsigned)lane % L;
    const bool active = lead && b < nb;
    float d2 = INFINITY;
    if (b < nb && b != tg && tg >= 0 && tg < nb) {
      const Foot T = foot_of(xyz(s.pos[tg]), xyz(s.col[0][tg]), xyz(s.col[1][tg]), xyz(s.col[2][tg]), xyz(s.half[tg]));
      const Foot J = foot_of(xyz(s.pos[b]), xyz(s.col[0][b]), xyz(s.col[1][b]), xyz(s.col[2][b]), xyz(s.half[b]));
      d2 = foot_distance2<L>(T, J, j);
    }
    for (int o = 32; o > 0; o >>= 1) d2 = fminf(d2, __shfl_xor(d2, o, 64));
    const float d = sqrtf(d2);
    const float r = d > g.width ? 1.0f : d / g.width;
    last_r = r;
    if (job == 0) n_rewards = t + 1;
    else n_rewards_x = t + 1;
    if (lead && lane == 0) (job ? g.x_rewards : g.rewards)[(size_t)e * g.max_h + t] = r;
    // the expanded child's state goes to its pool slot
    const int cs = (t == 0 && job == 0 && g.child_slot) ? g.child_slot[e] : -1;
    if (cs >= 0 && active && j < 2) {
      float* dst = g.pool + (size_t)cs * 13 * PS + opaque(b);
      if (j == 0) {
        dst[0 * PS] = x.x; dst[1 * PS] = x.y; dst[2 * PS] = x.z;
        dst[7 * PS] = v.x; dst[8 * PS] = v.y; dst[9 * PS] = v.z;
      } else {
        dst[3 * PS] = q0; dst[4 * PS] = q1; dst[5 * PS] = q2; dst[6 * PS] = q3;
        dst[10 * PS] = w.x; dst[11 * PS] = w.y; dst[12 * PS] = w.z;
      }
    }
    sync_all<W>();   // every wave has read the frames before they change
    if (r >= 1.0f) {
      if (job == 0) t_stop = t;
      break;
    }
  }
  }  // pushes
  if (deferred) break;
  // re-purposing: the extra simulation starts from its node's pool slot
  if (job == 1 || !g.x_desc || t_stop < 0 || t_stop + 1 >= n_push) break;
  // the pushes left, at most the extra pair's own horizon (top byte of w)
  n_push = min(n_push - t_stop - 1, (int)((unsigned)g.x_desc[e].w >> 24));
  last_r = 0.0f;
  if (active) {
    const float* st = g.pool + (size_t)g.x_desc[e].x * 13 * PS + opaque(b);
    x = mk(st[0 * PS], st[1 * PS], st[2 * PS]);
    q0 = st[3 * PS]; q1 = st[4 * PS]; q2 = st[5 * PS]; q3 = st[6 * PS];
    v = mk(st[7 * PS], st[8 * PS], st[9 * PS]);
    w = mk(st[10 * PS], st[11 * PS], st[12 * PS]);
  }
  }  // jobs

  if (deferred) {
    if (lead && lane == 0) g.overflow_list[atomicAdd(g.overflow_count, 1)] = e;
    return;
  }
  // outputs: the lead wave's
  if (!lead) return;
  if (rollout && lane == 0 && g.reward_count) g.reward_count[e] = n_rewards;
  if (rollout && lane == 0 && g.x_count) g.x_count[e] = n_rewards_x;
  if (rollout && !g.write_state) {
    if (lane == 0) {
      g.env_status[e] = status;
      if (g.stats) {
        g.stats[3 * e] = stat_nc;
        g.stats[3 * e + 1] = stat_pairs;
        g.stats[3 * e + 2] = stat_sub;
      }
    }
    return;
  }

  // ---- write back
  bool bad = false;
  if (active && j < 2) {
    const int i = opaque(base + b);
    float* st = g.state;
    if (j == 0) {
      st[0 * N + i] = x.x; st[1 * N + i] = x.y; st[2 * N + i] = x.z;
      st[7 * N + i] = v.x; st[8 * N + i] = v.y; st[9 * N + i] = v.z;
      bad = !(isfinite(x.x) && isfinite(x.y) && isfinite(x.z) && isfinite(v.x) && isfinite(v.y) && isfinite(v.z));
    } else {
      st[3 * N + i] = q0; st[4 * N + i] = q1; st[5 * N + i] = q2; st[6 * N + i] = q3;
      st[10 * N + i] = w.x; st[11 * N + i] = w.y; st[12 * N + i] = w.z;
      bad = !(isfinite(q0) && isfinite(q1) && isfinite(q2) && isfinite(q3) && isfinite(w.x) && isfinite(w.y) &&
              isfinite(w.z));
    }
  }
  if (__ballot(bad) != 0) status |= PMBS_ENV_NONFINITE;
  if (lane == 0) {
    g.env_status[e] = status;
    if (g.stats) {
      g.stats[3 * e] = stat_nc;
      g.stats[3 * e + 1] = stat_pairs;
      g.stats[3 * e + 2] = stat_sub;
    }
  }
}

// ------------------------------------------------------------------ block -> work item
// Workgroups go to the eight XCDs in turn (block i on XCD i mod 8) and each
// XCD has its own L2.  Neighbouring envs share the cache lines of every SoA
// row, so XCD x gets one contiguous run of the n items: block i takes item
// start(i mod 8) + i / 8 (a permutation of 0..n-1 for any n).
__device__ __forceinline__ int xcd_start(int x, int n) {
  const int q = n / 8, r = n - q * 8;
  return x * q + (x < r ? x : r);
}
__device__ __forceinline__ int xcd_item(int bid, int n) { return xcd_start(bid % 8, n) + bid / 8; }

// ------------------------------------------------------------------ the step kernel
// One workgroup per environment.  Without a work queue block i runs work item
// env_base + xcd_item(i); with one, blocks pull work items from the device counter
// until it passes n_envs (every block reaches that exit).  order[] maps
// work items to environments (longest horizon first for uneven rollouts).
// With XCD queues (xcd_queues, a grid of at least eight blocks) block i
// pulls from counter queue[i mod 8] the items of XCD i mod 8's own
// contiguous run, order[start(x) ..], so each XCD's L2 holds its own envs'
// state rows, as without a queue.
// The table's LDS entries: the same for every env, and no phase writes
// them, so a workgroup sets them once.
template <class S>
__device__ __forceinline__ void init_plane(S& s, const Params& p) {
  constexpr int PLANE = S::PLANE;
  if (threadIdx.x == 0) {
    s.pos[PLANE] = make_float4(0, 0, 0, 0);
    s.col[0][PLANE] = make_float4(1, 0, 0, 0);
    s.col[1][PLANE] = make_float4(0, 1, 0, 0);
    s.col[2][PLANE] = make_float4(0, 0, 1, 0);
    s.half[PLANE] = make_float4(0, 0, 0, 0);
    s.iwa[PLANE] = make_float4(0, 0, 0, 0);
    s.iwb[PLANE] = make_float4(0, 0, p.mu_plane, 0);
    s.vel[PLANE] = make_float4(0, 0, 0, 0);
    s.ang[PLANE] = make_float4(0, 0, 0, 0);
    s.cnt[PLANE] = 1;
    s.zero = make_float4(0, 0, 0, 0);
  }
}

// Three waves per SIMD for the kernel of the many small environments, at 168
// registers: 4096 x 15 takes 1.76 ms so, 1.98 with two (no spills), and took
// 2.61 with four where three took 2.19.  Its 53 spilled registers a lane are
// most of what the launch moves through HBM, 1 % of a copy's rate.
template <int K, int W, int NB>
__global__ __launch_bounds__(64 * W, K == 2 && NB == 16 && W == 1 ? 3 : 2) void step_kernel(StepArgs g) {
  __shared__ Smem<K, W, NB> s;
  __shared__ int next;
  init_plane(s, g.p);
  int n_work = g.work_count ? *g.work_count : g.n_envs;
  int* queue = g.queue;
  int seg = 0;
  if (g.xcd_queues) {
    const int x = blockIdx.x % 8;
    seg = xcd_start(x, n_work);
    n_work = xcd_start(x + 1, n_work) - seg;
    queue += x;
  }
  int wi = g.queue ? 0 : g.env_base + xcd_item(blockIdx.x, gridDim.x);
  for (;;) {
    if (g.queue) {
      if (threadIdx.x == 0) next = atomicAdd(queue, 1);
      __syncthreads();
      wi = __builtin_amdgcn_readfirstlane(next);
      __syncthreads();
    }
    if (wi >= n_work) break;
    run_env<K, W, NB, Run::STEP>(s, g, __builtin_amdgcn_readfirstlane(g.order ? g.order[seg + wi] : wi));
    if (!g.queue) break;
    __syncthreads();
  }
}

// The cost pass of a queued step: one block per env runs the push begin
// and the first substep's collision detection and writes the env's work
// estimate to cost_key (the rest of run_env is not compiled in).
template <int K, int W, int NB>
__global__ __launch_bounds__(64 * W, 2) void cost_kernel(StepArgs g) {
  __shared__ Smem<K, W, NB> s;
  init_plane(s, g.p);
  const int e = g.env_base + xcd_item(blockIdx.x, gridDim.x);
  if (e < g.n_envs) run_env<K, W, NB, Run::COST>(s, g, e);
}

// pmbs_sim_collide: one block per env writes its contact list at the current
// poses (4096 x 5, 128 contacts: 27.5 us by the step kernel at three waves per
// SIMD, 23.0 so; 4096 x 21, 512 contacts 77.5 and 69.3).
template <int K, int NB>
__global__ __launch_bounds__(64, 2) void collide_kernel(StepArgs g) {
  __shared__ Smem<K, 1, NB> s;
  init_plane(s, g.p);
  const int e = xcd_item(blockIdx.x, gridDim.x);
  if (e < g.n_envs) run_env<K, 1, NB, Run::COLLIDE>(s, g, e);
}

// Schedule of a queued step: each XCD's contiguous run of envs (xcd_start)
// by descending work estimate, a counting sort of the estimates clamped to
// [0, ORDER_BINS).  Equal estimates come in the order of the LDS atomics
// (an env's result does not depend on when it runs).  Block x of eight
// (ORDER_BINS threads each) sorts run x into order[start(x) ..] and clears
// the XCD's queue counter queue[x].
constexpr int ORDER_BINS = 1024;
__global__ __launch_bounds__(ORDER_BINS) void order_kernel(const int* __restrict__ key, int n, int* __restrict__ order,
                                                          int* queue) {
  __shared__ int start[ORDER_BINS];
  __shared__ int wsum[ORDER_BINS / 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int e0 = xcd_start(blockIdx.x, n), e1 = xcd_start(blockIdx.x + 1, n);
  order += e0;
  auto bin = [&](int e) {
    const int k = key[e];
    return k < 0 ? 0 : (k >= ORDER_BINS ? ORDER_BINS - 1 : k);
  };
  start[t] = 0;
  __syncthreads();
  for (int e = e0 + t; e < e1; e += ORDER_BINS) atomicAdd(&start[bin(e)], 1);
  __syncthreads();
  // thread t owns bin ORDER_BINS - 1 - t (largest first): the envs of
  // larger bins come before its own
  const int r = ORDER_BINS - 1 - t;
  const int c = start[r];
  int v = c;
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(v, d, 64);
    if (lane >= d) v += y;
  }
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  int before = 0;
  for (int k = 0; k < w; ++k) before += wsum[k];
  start[r] = before + v - c;
  __syncthreads();
  for (int e = e0 + t; e < e1; e += ORDER_BINS) order[atomicAdd(&start[bin(e)], 1)] = e;
  if (t == 0) queue[blockIdx.x] = 0;
}

__global__ void zero_kernel(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ------------------------------------------------------------------ state pool
// env e <-> pool slot slots[e] (slot < 0: env left alone).  Pool slot layout
// [13][pool_stride]; env bodies are the packed rows env_offset[e]...
__global__ __launch_bounds__(64) void pool_kernel(PoolArgs g) {
  const int e = xcd_item(blockIdx.x, gridDim.x);
  if (e >= g.n_envs) return;
  const int slot = g.slots[e];
  if (slot < 0 || slot >= g.pool_slots) return;
  const int base = g.env_offset[e];
  const int nb = g.env_offset[e + 1] - base;
  if (nb > g.pool_stride) return;
  float* pool = g.pool + (size_t)slot * 13 * g.pool_stride;
  for (int t = threadIdx.x; t < 13 * nb; t += 64) {
    const int r = t / nb, i = t - r * nb;
    float* env_p = g.state + (size_t)r * g.stride + base + i;
    float* pool_p = pool + (size_t)r * g.pool_stride + i;
    if (g.to_pool) *pool_p = *env_p;
    else *env_p = *pool_p;
  }
}

// ------------------------------------------------------------------ reward
__device__ __forceinline__ Foot load_foot(const float* st, int SN, int si, const float* bc, int BN, int bi) {
  f3 c0, c1, c2;
  quat_cols(st[3 * SN + si], st[4 * SN + si], st[5 * SN + si], st[6 * SN + si], &c0, &c1, &c2);
  return foot_of(mk(st[0 * SN + si], st[1 * SN + si], st[2 * SN + si]), c0, c1, c2,
                 mk(bc[0 * BN + bi], bc[1 * BN + bi], bc[2 * BN + bi]));
}

// One wave per environment, four lanes per box: bound by the ALU (192 point
// to segment distances with a correctly rounded divide per pair of boxes), and
// by the lanes in use, so a box's 16 vertex turns are split over four lanes
// and one square root follows the wave's minimum.  4096 x 15: 41.8 us with a
// lane per box and a root per distance, 9.9 us now.
__global__ __launch_bounds__(64) void reward_kernel(RewardArgs g) {
  const int e = xcd_item(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x;
  if (e >= g.n_envs) return;
  const int base = g.env_offset[e];
  const int nb = g.env_offset[e + 1] - base;
  const int t = g.target[e];
  const bool from_pool = g.pool != nullptr;
  const float* st = from_pool ? g.pool + (size_t)g.slots[e] * 13 * g.pool_stride : g.state;
  const int SN = from_pool ? g.pool_stride : g.stride;
  const int s0 = from_pool ? 0 : base;
  const int BN = g.bc_base ? g.bc_stride : g.stride;
  const int b0 = g.bc_base ? g.bc_base[e] : base;
  float d = INFINITY;
  if (t >= 0 && t < nb) {
    const Foot T = load_foot(st, SN, s0 + t, g.bconst, BN, b0 + t);
    for (int i = lane; i < 4 * nb; i += 64) {   // four lanes per box share its vertices
      const int k = i >> 2;
      if (k == t) continue;
      const Foot J = load_foot(st, SN, s0 + k, g.bconst, BN, b0 + k);
      d = fminf(d, foot_distance2<4>(T, J, i & 3));
    }
  } else {
    d = NAN;
  }
  for (int off = 32; off > 0; off >>= 1) d = fminf(d, __shfl_xor(d, off, 64));
  d = sqrtf(d);
  if (lane == 0) {
    if (g.clearance) g.clearance[e] = d;
    g.reward[e] = d > g.width ? 1.0f : d / g.width;
  }
}

// ------------------------------------------------------------------ start-pose validity
// Frames of one environment's boxes, as the step kernel holds them in LDS.
struct Frames {
  float4 pos[MAXB];
  float4 col[3][MAXB];
  float4 half[MAXB];
};

// Start-pose validity of every contour push (Sec. IV-B: pushes that cannot
// start because of a collision are discarded): bit a mod 32 of word a / 32 is
// set when the pusher at action a's start pose clears every box by sat_clear.
//
// Four waves per environment: the boxes' frames from the env state (or pool
// slot src_slot[e]; < 0 skips the env), computed as the step kernel computes
// them, then a thread per action for its pusher, then every (action, box) pair,
// box j by wave j mod 4.  The ALU bounds it: 15 axes for each of 8 nb * nb
// pairs, of which few are near each other.  So the pairs go through three
// sieves, a wave's own list of pairs packed after each: the pusher's two
// horizontal axes, lane = action (the pusher's own radii formed once; most of
// the pairs end here), then the other four face axes, then the nine edge axes,
// lane = pair.  1024 x 21: 45 to 64 -> 19 us; 64 x 11: 32 -> 10.6, with a lane
// per push walking all the boxes before.  Workgroups loop over the envs (the
// count may come from device memory).
constexpr int VALID_WAVES = PMBS_VALID_WORDS / 2, VALID_ACTIONS = 32 * PMBS_VALID_WORDS;
struct ValidShared {
  Frames f;
  float4 centre[VALID_ACTIONS];    // pusher centre (x, y), radii along its first two axes
  float4 axes[VALID_ACTIONS];      // its first two axes (x, y each; z = 0)
  unsigned short list[VALID_WAVES][VALID_ACTIONS * (MAXB / VALID_WAVES + 1)];   // action | box << 8
  unsigned hit[PMBS_VALID_WORDS];  // actions that meet a box
};

__device__ __forceinline__ Box action_box(float4 centre, float4 axes, const Params& p) {
  Box b;
  b.c = mk(centre.x, centre.y, p.pusher_z);
  b.a0 = mk(axes.x, axes.y, 0.0f);
  b.a1 = mk(axes.z, axes.w, 0.0f);
  b.a2 = mk(0, 0, 1);
  b.h = mk(p.phx, p.phy, p.phz);
  return b;
}

__global__ __launch_bounds__(64 * VALID_WAVES) void valid_kernel(ValidArgs g) {
  static_assert(MAXB <= 256 && VALID_ACTIONS <= 256, "a pair is 8 + 8 bits");
  __shared__ ValidShared s;
  const Params& p = g.p;
  const int n = g.count ? g.count[0] + g.count[1] : g.n_envs;
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  unsigned short* const list = s.list[wid];
  for (int e = blockIdx.x; e < n; e += gridDim.x) {
    const int src = g.src_slot ? g.src_slot[e] : -1;
    if (g.src_slot && src < 0) continue;
    const int base = g.env_offset[e];
    const int nb = g.env_offset[e + 1] - base;
    if (t < nb) {
      const float* st = src >= 0 ? g.pool + (size_t)src * 13 * g.pool_stride : g.state;
      const int SN = src >= 0 ? g.pool_stride : g.stride;
      const int si = src >= 0 ? lane : base + lane;
      const int BN = g.bc_base ? g.bc_stride : g.stride;
      const int bi = g.bc_base ? g.bc_base[e] + lane : base + lane;
      f3 c0, c1, c2;
      quat_cols(st[3 * SN + si], st[4 * SN + si], st[5 * SN + si], st[6 * SN + si], &c0, &c1, &c2);
      s.f.pos[lane] = make_float4(st[0 * SN + si], st[1 * SN + si], st[2 * SN + si], 0.0f);
      s.f.col[0][lane] = f4(c0, 0.0f);
      s.f.col[1][lane] = f4(c1, 0.0f);
      s.f.col[2][lane] = f4(c2, 0.0f);
      s.f.half[lane] = make_float4(g.bconst[0 * BN + bi], g.bconst[1 * BN + bi], g.bconst[2 * BN + bi], 0.0f);
    }
    if (t < PMBS_VALID_WORDS) s.hit[t] = 0u;
    __syncthreads();
    const int n_act = min(nb * p.n_dirs, VALID_ACTIONS);
    if (t < n_act) {
      const int obj = t / p.n_dirs, dir = t - obj * p.n_dirs;
      const Box P = pusher_box(pusher_pose(contour_start(s.f, obj, dir, p), p), p);
      s.centre[t] = make_float4(P.c.x, P.c.y, radius_along(P, P.a0), radius_along(P, P.a1));
      s.axes[t] = make_float4(P.a0.x, P.a0.y, P.a1.x, P.a1.y);
    }
    __syncthreads();
    int kept = 0;
    for (int j = wid; j < nb; j += VALID_WAVES) {
      const Box A = load_box(s.f, j);
      for (int a0 = 0; a0 < n_act; a0 += 64) {
        const int a = min(a0 + lane, n_act - 1);
        const float4 pc = s.centre[a];
        const Box P = action_box(pc, s.axes[a], p);
        const f3 d = P.c - A.c;
        const bool apart = fabsf(dot(d, P.a0)) - radius_along(A, P.a0) - pc.z > 0.0f ||
                           fabsf(dot(d, P.a1)) - radius_along(A, P.a1) - pc.w > 0.0f;
        const bool keep = a0 + lane < n_act && !apart;
        const unsigned long long m = __ballot(keep);
        if (keep) list[kept + __popcll(m & below)] = (unsigned short)(a | j << 8);
        kept += __popcll(m);
      }
    }
    // a list is packed in place: what is written lies at or before the 64
    // entries that were just read
    wave_sync();
    int left = 0;
    for (int i0 = 0; i0 < kept; i0 += 64) {
      const int v = list[min(i0 + lane, kept - 1)];
      const Box A = load_box(s.f, v >> 8), P = action_box(s.centre[v & 255], s.axes[v & 255], p);
      const f3 d = P.c - A.c;
      float best = gap_along(A, P, d, P.a2);
#pragma unroll
      for (int k = 0; k < 3; ++k) best = fmaxf(best, gap_along(A, P, d, axis(A, k)));
      const bool keep = i0 + lane < kept && !(best > 0.0f);
      const unsigned long long m = __ballot(keep);
      wave_sync();
      if (keep) list[left + __popcll(m & below)] = (unsigned short)v;
      left += __popcll(m);
      wave_sync();
    }
    for (int i0 = 0; i0 < left; i0 += 64) {
      const int v = list[min(i0 + lane, left - 1)], a = v & 255;
      const Box A = load_box(s.f, v >> 8), P = action_box(s.centre[a], s.axes[a], p);
      if (i0 + lane < left && !edges_clear(A, P, p.edge_eps)) atomicOr(&s.hit[a >> 5], 1u << (a & 31));
    }
    __syncthreads();
    if (t < PMBS_VALID_WORDS) {
      const int m = n_act - 32 * t;
      g.out[(size_t)e * PMBS_VALID_WORDS + t] = ~s.hit[t] & (m >= 32 ? ~0u : m > 0 ? (1u << m) - 1u : 0u);
    }
  }
}

// ------------------------------------------------------------------ launchers
hipError_t launch_valid(const ValidArgs& a, hipStream_t stream, int grid) {
  const int g = grid > 0 ? grid : a.n_envs;
  if (g <= 0) return hipSuccess;
  hipLaunchKernelGGL(valid_kernel, dim3(g), dim3(64 * VALID_WAVES), 0, stream, a);
  return hipGetLastError();
}

// Calls f(kernel tag) for the kernel of a contact class (128, 256 or 512
// contacts: 2, 4 or 8 slots of row contacts per lane), a workgroup shape (1
// or 2 waves per environment; the 512-contact class has one) and the largest
// body count: at most 16 boxes, which is what four lanes a body leave room for,
// take the 16-box layout (128 contacts: 4096 x 15 1.76 ms, 2.25 in the 31-box
// layout; 1024 x 15 1.12 and 1.24; 64 x 9 0.88 and 0.98.  256 contacts, 60
// substeps of 1024 x 10 cubes in two touching towers: 1.34 and 1.51; 4096 x 8
// touching cubes, eight workgroups a CU and five: 3.13 and 4.48).
template <int K_, int W_, int NB_>
struct Shape {
  static constexpr int K = K_, W = W_, NB = NB_;
};
template <class F>
static auto with_shape(int max_contacts, int waves, int max_nb, F f) {
  if (max_nb > 16) {
    if (max_contacts > 256) return f(Shape<8, 1, 32>{});
    if (max_contacts > 128) return waves == 2 ? f(Shape<4, 2, 32>{}) : f(Shape<4, 1, 32>{});
    return waves == 2 ? f(Shape<2, 2, 32>{}) : f(Shape<2, 1, 32>{});
  }
  if (max_contacts > 256) return f(Shape<8, 1, 16>{});
  if (max_contacts > 128) return waves == 2 ? f(Shape<4, 2, 16>{}) : f(Shape<4, 1, 16>{});
  return waves == 2 ? f(Shape<2, 2, 16>{}) : f(Shape<2, 1, 16>{});
}

static hipError_t launch_shape(const StepArgs& a, int max_contacts, hipStream_t stream, int grid, int waves, int max_nb) {
  return with_shape(max_contacts, waves, max_nb, [&](auto t) {
    using T = decltype(t);
    hipLaunchKernelGGL((step_kernel<T::K, T::W, T::NB>), dim3(grid), dim3(64 * T::W), 0, stream, a);
    return hipGetLastError();
  });
}

hipError_t launch_step(const StepArgs& a, int max_contacts, hipStream_t stream, int waves, int max_nb) {
  const int n = a.n_envs - a.env_base;
  return n <= 0 ? hipSuccess : launch_shape(a, max_contacts, stream, n, waves, max_nb);
}

hipError_t launch_step_class(const StepArgs& a, int max_contacts, hipStream_t stream, int grid, int waves, int max_nb) {
  if (grid <= 0 || !a.queue) return hipErrorInvalidValue;
  return launch_shape(a, max_contacts, stream, grid, waves, max_nb);
}

hipError_t launch_cost(const StepArgs& a, int max_contacts, hipStream_t stream, int waves, int max_nb) {
  const int n = a.n_envs - a.env_base;
  if (n <= 0 || !a.cost_key) return n <= 0 ? hipSuccess : hipErrorInvalidValue;
  StepArgs c = a;
  if (c.n_substeps < 1) c.n_substeps = 1;   // the estimate comes from the first substep
  return with_shape(max_contacts, waves, max_nb, [&](auto t) {
    using T = decltype(t);
    hipLaunchKernelGGL((cost_kernel<T::K, T::W, T::NB>), dim3(n), dim3(64 * T::W), 0, stream, c);
    return hipGetLastError();
  });
}

hipError_t launch_collide(const StepArgs& a, int max_contacts, hipStream_t stream, int max_nb) {
  if (a.n_envs <= 0 || !a.dbg_count || !a.dbg_contacts) return a.n_envs <= 0 ? hipSuccess : hipErrorInvalidValue;
  StepArgs c = a;
  c.n_substeps = 1;
  return with_shape(max_contacts, 1, max_nb, [&](auto t) {
    using T = decltype(t);
    hipLaunchKernelGGL((collide_kernel<T::K, T::NB>), dim3(c.n_envs), dim3(64), 0, stream, c);
    return hipGetLastError();
  });
}

hipError_t launch_order(const int* key, int n, int* order, int* queue, hipStream_t stream) {
  if (n <= 0 || !key || !order || !queue) return hipErrorInvalidValue;
  hipLaunchKernelGGL(order_kernel, dim3(8), dim3(ORDER_BINS), 0, stream, key, n, order, queue);
  return hipGetLastError();
}

hipError_t launch_zero(int* p, int n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3((n + 63) / 64), dim3(64), 0, stream, p, n);
  return hipGetLastError();
}

int step_blocks_per_cu(int max_contacts, int waves, int max_nb) {
  return with_shape(max_contacts, waves, max_nb, [&](auto t) {
    using T = decltype(t);
    int n = 0;
    const hipError_t e =
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, step_kernel<T::K, T::W, T::NB>, 64 * T::W, 0);
    return e == hipSuccess ? n : 0;
  });
}

hipError_t launch_pool(const PoolArgs& a, hipStream_t stream) {
  if (a.n_envs <= 0) return hipSuccess;
  hipLaunchKernelGGL(pool_kernel, dim3(a.n_envs), dim3(64), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_reward(const RewardArgs& a, hipStream_t stream) {
  if (a.n_envs <= 0) return hipSuccess;
  hipLaunchKernelGGL(reward_kernel, dim3(a.n_envs), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace pmbs
