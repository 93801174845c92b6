// trace.hip -- BVH traversal, G-buffer and thin-lens distributed ray trace.
//
// Traversal: both children of a node are box-tested from one record, the
// nearer is visited first.  The wave-coherent walk (G-buffer) reads 64-byte
// records with full-precision boxes through the scalar cache; the per-lane
// walk (lens rays) reads 44 bytes with half-precision boxes and keeps a
// stack per lane whose first HDOF_LDS_STACK entries live in LDS (entry i of
// lane t at stk[i][t], so a wave's pushes hit 64 distinct banks) and the
// rest in a short private spill array.
// Triangles: watertight ray/triangle test (Woop, Benthin, Wald, JCGT 2013),
// ties broken towards the lowest input triangle index.
//
// G-buffer: 16x16-pixel blocks, each wave an 8x8 quadrant (coherent primary
// rays); blocks remapped so each XCD works on a contiguous band of the image
// and keeps its part of the BVH in its own L2.
// Thin-lens trace: queue of (pixel, sample) entries built from the mask's
// counts and offsets; the waves of a persistent grid pop entries from device
// counters, so the host never reads the ray count; results per entry,
// then a per-pixel reduction in fixed sample order (deterministic).
#include "hdof_internal.h"

#include <hip/hip_ext.h>

namespace {

struct Ray {
  V3 O, D;
  V3 inv, oinv;  // 1/D and -O/D for the slab test
  // watertight test in the ray's sheared frame (Woop, Benthin, Wald): rows
  // of the map v -> ((v-O)[kx] - Sx (v-O)[kz], (v-O)[ky] - Sy (v-O)[kz],
  // Sz (v-O)[kz]) as dense 3-vectors, with the origin term folded in
  V3 mx, my, mz;
  float ox, oy, oz;
};

__device__ inline float safe_inv(float d) {
  float a = fabsf(d) > 1e-30f ? d : copysignf(1e-30f, d);
  return 1.0f / a;
}

__device__ inline V3 unit(int k) { return V3{k == 0 ? 1.0f : 0.0f, k == 1 ? 1.0f : 0.0f, k == 2 ? 1.0f : 0.0f}; }

// What make_ray divides for: the inverse direction and the shear of the
// axes (kx, ky, kz), kz the direction's largest component and (kx, ky)
// ordered by its sign.
struct RayPre {
  V3 O, D, inv;
  float Sx, Sy;
  int axes;  // kz | kx << 2
};

__device__ inline RayPre ray_pre(V3 O, V3 D) {
  RayPre q;
  q.O = O;
  q.D = D;
  q.inv = V3{safe_inv(D.x), safe_inv(D.y), safe_inv(D.z)};
  float ax = fabsf(D.x), ay = fabsf(D.y), az = fabsf(D.z);
  int kz = ax > ay ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
  int kx = kz == 2 ? 0 : kz + 1;
  int ky = kx == 2 ? 0 : kx + 1;
  float dz = comp(D, kz);
  if (dz < 0.0f) {
    int t = kx;
    kx = ky;
    ky = t;
  }
  q.Sx = comp(D, kx) / dz;
  q.Sy = comp(D, ky) / dz;
  q.axes = kz | kx << 2;
  return q;
}

// (the inverse direction's kz component is 1 / dz: the largest component of
// a direction is above safe_inv's threshold)
__device__ inline Ray ray_of(const RayPre& q) {
  Ray r;
  r.O = q.O;
  r.D = q.D;
  r.inv = q.inv;
  r.oinv = V3{-q.O.x * q.inv.x, -q.O.y * q.inv.y, -q.O.z * q.inv.z};
  const int kz = q.axes & 3, kx = q.axes >> 2, ky = 3 - kx - kz;
  const float Sz = comp(q.inv, kz);
  const V3 ez = unit(kz);
  r.mx = V3{kx == 0 ? 1.0f : (kz == 0 ? -q.Sx : 0.0f), kx == 1 ? 1.0f : (kz == 1 ? -q.Sx : 0.0f),
            kx == 2 ? 1.0f : (kz == 2 ? -q.Sx : 0.0f)};
  r.my = V3{ky == 0 ? 1.0f : (kz == 0 ? -q.Sy : 0.0f), ky == 1 ? 1.0f : (kz == 1 ? -q.Sy : 0.0f),
            ky == 2 ? 1.0f : (kz == 2 ? -q.Sy : 0.0f)};
  r.mz = V3{Sz * ez.x, Sz * ez.y, Sz * ez.z};
  r.ox = dot3(r.mx, q.O);
  r.oy = dot3(r.my, q.O);
  r.oz = dot3(r.mz, q.O);
  return r;
}

__device__ inline Ray make_ray(V3 O, V3 D) { return ray_of(ray_pre(O, D)); }

// slab test of one child box against [0, tmax]; conservative by 2 gamma(3)
__device__ inline bool box_hit(const Ray& r, float lox, float hix, float loy, float hiy, float loz,
                               float hiz, float tmax, float& tnear) {
  float tx0 = fmaf(lox, r.inv.x, r.oinv.x), tx1 = fmaf(hix, r.inv.x, r.oinv.x);
  float ty0 = fmaf(loy, r.inv.y, r.oinv.y), ty1 = fmaf(hiy, r.inv.y, r.oinv.y);
  float tz0 = fmaf(loz, r.inv.z, r.oinv.z), tz1 = fmaf(hiz, r.inv.z, r.oinv.z);
  float tmin = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
  float tmx = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fminf(fmaxf(tz0, tz1), tmax));
  tnear = tmin;
  return tmin <= tmx * 1.0000004f;
}

// The same test when the signs of the ray's direction are known: (nx, ny,
// nz) are the box's planes the ray enters through and (fx, fy, fz) those it
// leaves through, so the per-axis min and max of box_hit are decided in
// advance.  For a box with lo <= hi on every axis the entry and exit
// distances equal box_hit's bit for bit (an fma with a fixed multiplier and
// addend is monotonic in its first operand).
__device__ inline bool box_hit_signed(const Ray& r, float nx, float fx, float ny, float fy, float nz, float fz,
                                      float tmax, float& tnear) {
  const float tx0 = fmaf(nx, r.inv.x, r.oinv.x), tx1 = fmaf(fx, r.inv.x, r.oinv.x);
  const float ty0 = fmaf(ny, r.inv.y, r.oinv.y), ty1 = fmaf(fy, r.inv.y, r.oinv.y);
  const float tz0 = fmaf(nz, r.inv.z, r.oinv.z), tz1 = fmaf(fz, r.inv.z, r.oinv.z);
  const float tmin = fmaxf(fmaxf(tx0, ty0), fmaxf(tz0, 0.0f));
  const float tmx = fminf(fminf(tx1, ty1), fminf(tz1, tmax));
  tnear = tmin;
  return tmin <= tmx * 1.0000004f;
}

// Half-precision boxes: a pair of planes (minimum, maximum) in units about
// the node's centre.  Rotated by 16 where the ray runs against the axis, a
// pair has the plane the ray enters through in its low half, and an fma
// that takes a half operand gives its distance.  A node that box_hit enters
// by its full boxes is entered here: with e = 2^-24, a plane's distance t
// there has one rounding (e t), here two, of the centre's distance and of
// the sum (2 e t, and e times the plane's offset from the centre, which the
// planes' margin covers), so both sides of the comparison may be 3 e nearer
// or farther and the 7 e of box_hit become 13 e: 1 + 2^-20.
__device__ inline float half_dist(unsigned pair, int hi, float sinv, float base) {
  unsigned short u = (unsigned short)(hi ? pair >> 16 : pair);
  _Float16 h;
  __builtin_memcpy(&h, &u, 2);
  return fmaf((float)h, sinv, base);
}

__device__ inline bool box_hit_half(unsigned x, unsigned y, unsigned z, V3 sinv, V3 base, int rx, int ry, int rz,
                                    float tmax, float& tnear) {
  x = __builtin_amdgcn_alignbit(x, x, rx);
  y = __builtin_amdgcn_alignbit(y, y, ry);
  z = __builtin_amdgcn_alignbit(z, z, rz);
  const float tmin = fmaxf(fmaxf(half_dist(x, 0, sinv.x, base.x), half_dist(y, 0, sinv.y, base.y)),
                           fmaxf(half_dist(z, 0, sinv.z, base.z), 0.0f));
  const float tmx = fminf(fminf(half_dist(x, 1, sinv.x, base.x), half_dist(y, 1, sinv.y, base.y)),
                          fminf(half_dist(z, 1, sinv.z, base.z), tmax));
  tnear = tmin;
  return tmin <= tmx * 1.00000095f;
}

struct Best {
  float t;
  int tri;   // leaf-order index, -1 = none
  int id;    // input index
};

// Woop-Benthin-Wald watertight test; updates best on a closer (or tied,
// lower input index) hit with t > 0.  Each vertex is mapped by the ray's
// shear exactly once per test, so two triangles sharing an edge evaluate
// the same 2D edge function for it (watertight); the z row is only needed
// for a triangle the ray passes through.
__device__ inline float shear(V3 m, float o, float4 v) { return fmaf(m.z, v.z, fmaf(m.y, v.y, m.x * v.x)) - o; }

__device__ inline void tri_test(const Ray& r, const float4* __restrict__ tris, int i, Best& b) {
  const float4 a = tris[3 * i], q = tris[3 * i + 1], c = tris[3 * i + 2];
  const float Ax = shear(r.mx, r.ox, a), Ay = shear(r.my, r.oy, a);
  const float Bx = shear(r.mx, r.ox, q), By = shear(r.my, r.oy, q);
  const float Cx = shear(r.mx, r.ox, c), Cy = shear(r.my, r.oy, c);
  float U = Cx * By - Cy * Bx;
  float V = Ax * Cy - Ay * Cx;
  float W = Bx * Ay - By * Ax;
  if (U == 0.0f || V == 0.0f || W == 0.0f) {
    U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
    V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
    W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
  }
  if ((U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f)) return;
  const float det = U + V + W;
  if (det == 0.0f) return;
  const float T = U * shear(r.mz, r.oz, a) + V * shear(r.mz, r.oz, q) + W * shear(r.mz, r.oz, c);
  const float t = T * __builtin_amdgcn_rcpf(det);
  if (!(t > 0.0f)) return;
  const int id = __float_as_int(a.w);
  if (t < b.t || (t == b.t && id < b.id)) {
    b.t = t;
    b.tri = i;
    b.id = id;
  }
}

__device__ inline void test_leaf(const Ray& r, const float4* __restrict__ tris, unsigned code, Best& b) {
  int first = (int)(code & HDOF_LEAF_FIRST_MASK);
  int cnt = (int)((code >> 27) & 0xF) + 1;
  for (int k = 0; k < cnt; ++k) tri_test(r, tris, first + k, b);
}

// Whether the ray meets the box of cnt triangles from the first on before
// tmax (r: inv and oinv).  The half boxes of a walk are wider than a leaf's
// own, and at the very edge of a triangle, a rounding either way, this test
// decides whether the ray meets the triangle.
__device__ inline bool tris_box_hit(const Ray& r, const float4* __restrict__ tris, int first, int cnt, float tmax) {
  V3 lo = V3{INFINITY, INFINITY, INFINITY}, hi = V3{-INFINITY, -INFINITY, -INFINITY};
  for (int k = 0; k < cnt; ++k) {
    const float4 a = tris[3 * (first + k)], q = tris[3 * (first + k) + 1], c = tris[3 * (first + k) + 2];
    lo = V3{fminf(lo.x, fminf(fminf(a.x, q.x), c.x)), fminf(lo.y, fminf(fminf(a.y, q.y), c.y)),
            fminf(lo.z, fminf(fminf(a.z, q.z), c.z))};
    hi = V3{fmaxf(hi.x, fmaxf(fmaxf(a.x, q.x), c.x)), fmaxf(hi.y, fmaxf(fmaxf(a.y, q.y), c.y)),
            fmaxf(hi.z, fmaxf(fmaxf(a.z, q.z), c.z))};
  }
  float tn;
  return box_hit(r, lo.x, hi.x, lo.y, hi.y, lo.z, hi.z, tmax, tn);
}

// this lane's bit of a wave's mask
__device__ __forceinline__ bool lane_of(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// the lanes of a wave's mask (__popcll's 64-bit result is compared by the
// vector ALU)
__device__ __forceinline__ int lanes(unsigned long long m) {
  int n;
  asm("s_bcnt1_i32_b64 %0, %1" : "=s"(n) : "s"(m) : "scc");
  return n;
}

// The same tests of a leaf that the whole wave visits, for the lanes of mask
// m: the records are scalar loads, and but for two branches that the wave
// takes as a whole (an edge function that is exactly 0 in some lane; no lane
// inside) the test is straight-line code, its result a select.  The same
// operations as tri_test, so the same hits bit for bit.
__device__ __forceinline__ void test_leaf_wave(const Ray& r, const float4* __restrict__ tris, unsigned code,
                                               unsigned long long m, Best& b) {
  int i = (int)(code & HDOF_LEAF_FIRST_MASK);
  const int end = i + (int)((code >> 27) & 0xF) + 1;
  for (; i < end; ++i) {
    const float4* p = (const float4*)((const char*)tris + 48u * (unsigned)i);
    const float4 a = p[0], q = p[1], c = p[2];
    const float Ax = shear(r.mx, r.ox, a), Ay = shear(r.my, r.oy, a);
    const float Bx = shear(r.mx, r.ox, q), By = shear(r.my, r.oy, q);
    const float Cx = shear(r.mx, r.ox, c), Cy = shear(r.my, r.oy, c);
    float U = Cx * By - Cy * Bx;
    float V = Ax * Cy - Ay * Cx;
    float W = Bx * Ay - By * Ax;
    const unsigned long long zm = __builtin_amdgcn_ballot_w64(U == 0.0f) | __builtin_amdgcn_ballot_w64(V == 0.0f) |
                                  __builtin_amdgcn_ballot_w64(W == 0.0f);
    if ((zm & m) != 0ull) {
      const bool zero = lane_of(zm);
      const float U2 = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
      const float V2 = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
      const float W2 = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
      U = zero ? U2 : U;
      V = zero ? V2 : V;
      W = zero ? W2 : W;
    }
    const unsigned long long in =
        ~(__builtin_amdgcn_ballot_w64(fminf(fminf(U, V), W) < 0.0f) &
          __builtin_amdgcn_ballot_w64(fmaxf(fmaxf(U, V), W) > 0.0f)) & m;
    if (in == 0ull) continue;
    const float det = U + V + W;
    const float T = U * shear(r.mz, r.oz, a) + V * shear(r.mz, r.oz, q) + W * shear(r.mz, r.oz, c);
    const float t = T * __builtin_amdgcn_rcpf(det);
    const int id = __float_as_int(a.w);
    const unsigned long long closer =
        __builtin_amdgcn_ballot_w64(t < b.t) |
        (__builtin_amdgcn_ballot_w64(t == b.t) & __builtin_amdgcn_ballot_w64(id < b.id));
    const bool hit = lane_of(in & closer & __builtin_amdgcn_ballot_w64(det != 0.0f) &
                             __builtin_amdgcn_ballot_w64(t > 0.0f));
    b.t = hit ? t : b.t;
    b.tri = hit ? i : b.tri;
    b.id = hit ? id : b.id;
  }
}

// Each internal node is entered at most once per ray, so more than n_nodes
// steps means a malformed tree: the ray stops and raises the device flag
// instead of looping.
struct Work {
  int visits, tests;
};

// What a wave of the persistent trace keeps in LDS: 64 ray slots (structure
// of arrays, a slot's fields SLOT_* of a ray that waits or is walked, then
// its hit in place of the shear), the slots no lane has taken yet, and the
// lanes' stacks (entry i of lane t at stk[i + 1][t], below it TRAV_DONE; one
// row more takes what a full stack is written in vain).
enum { SLOT_O, SLOT_D = 3, SLOT_INV = 6, SLOT_SX = 9, SLOT_SY, SLOT_AXES, SLOT_S1, SLOT_ENTRY, SLOT_DONE, SLOT_N };
#define SLOT_HIT SLOT_SX  // of a finished ray: distance, triangle, its input index
struct PoolLds {
  float f[SLOT_N][64];
  int list[64];
  int stk[HDOF_LDS_STACK + 2][64];
};
#define TRAV_DONE 0xFFFFFFFFu  // entry of a lane without a ray, or with a finished one (no leaf has this code)

// Orders the wave's LDS accesses as the program has them (the LDS executes
// one wave's accesses in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Slot i's ray, to be walked (state 0; 2: with its leaves' boxes tested).
__device__ __forceinline__ void slot_ray(PoolLds& L, int i, V3 O, V3 D, int state) {
  const RayPre q = ray_pre(O, D);
  const float f[SLOT_S1] = {O.x,     O.y,     O.z,  D.x,  D.y, D.z, q.inv.x,
                            q.inv.y, q.inv.z, q.Sx, q.Sy, __int_as_float(q.axes)};
#pragma unroll
  for (int k = 0; k < SLOT_S1; ++k) L.f[k][i] = f[k];
  L.f[SLOT_DONE][i] = __int_as_float(state);
}

__device__ __forceinline__ V3 slot_v3(const PoolLds& L, int f, int i) { return V3{L.f[f][i], L.f[f + 1][i], L.f[f + 2][i]}; }

// Wave-coherent traversal: the lanes of a wave walk one node sequence, the
// union of their own paths (primary rays of an 8x8 pixel quadrant are
// coherent).  Node records and leaf triangles are then wave-uniform loads,
// served by the scalar data cache instead of 64 vector fetches per node;
// the node stack is one VGPR holding entry i in lane i; a lane tests the
// boxes of every node the wave enters against its own closest hit, and the
// wave enters a child when any lane's ray reaches it.  Of two such
// children the one the wave's first lane reaches first is entered first.
// Each node is entered at most once per wave, so more than n_nodes steps
// raises the device flag and stops.
// Bound: instruction issue.  A visit took 56 scalar and 52 vector
// instructions; a child that no lane reaches is now the code -1, so that one
// scalar or tells the common case (two nodes to enter), addresses are 32-bit
// scalar offsets, and a leaf's tests have no lane-wise branches: 35 and 55
// (2.07M primary rays in 200k triangles, 38 visits a wave: 187 -> 152 us,
// 175 -> 139 and 142 -> 109 for other views; vector ALUs 72 % busy).  Tests
// specialised by the rays' common shear axis, 12 vector operations less per
// triangle: no faster, three times the code.
// FLIP >= 0: every live lane's direction has the signs FLIP gives (bit k
// set: axis k negative), so each slab's entry and exit planes are known at
// compile time (one copy of the loop per sign octant) and the box test
// needs no per-lane min and max of the two slab distances.  FLIP < 0: the
// general test.
template <bool COUNT, int FLIP>
__device__ inline Best traverse_wave(const float4* __restrict__ nodes, const float4* __restrict__ tris,
                                     int n_nodes, const Ray& r, bool live, int* __restrict__ flags, Work& wk) {
  // a lane without a ray starts with a negative closest-hit distance: every
  // box test then fails for it (entry distances are >= 0), so its results
  // need no masking
  Best b = Best{live ? INFINITY : -1.0f, -1, 0x7fffffff};
  const int lane = (int)(threadIdx.x & 63);
  int stackv = 0;  // entry i in lane i
  int sp = 0;
  int cur = 0;  // root (internal)
  for (int left = n_nodes;;) {
    if (left-- < 0) {
      if (live) atomicOr(flags, HDOF_FLAG_STACK_OVERFLOW);
      break;
    }
    if (COUNT && live) wk.visits++;
    const float4* nd = (const float4*)((const char*)nodes + ((unsigned)cur << 6));
    const float4 n0 = nd[0], n1 = nd[1], n2 = nd[2], n3 = nd[3];
    float t0, t1;
    bool h0, h1;
    if (FLIP >= 0) {
      constexpr bool fx = (FLIP & 1) != 0, fy = (FLIP & 2) != 0, fz = (FLIP & 4) != 0;
      h0 = box_hit_signed(r, fx ? n0.y : n0.x, fx ? n0.x : n0.y, fy ? n0.w : n0.z, fy ? n0.z : n0.w,
                          fz ? n2.y : n2.x, fz ? n2.x : n2.y, b.t, t0);
      h1 = box_hit_signed(r, fx ? n1.y : n1.x, fx ? n1.x : n1.y, fy ? n1.w : n1.z, fy ? n1.z : n1.w,
                          fz ? n2.w : n2.z, fz ? n2.z : n2.w, b.t, t1);
    } else {
      h0 = box_hit(r, n0.x, n0.y, n0.z, n0.w, n2.x, n2.y, b.t, t0);
      h1 = box_hit(r, n1.x, n1.y, n1.z, n1.w, n2.z, n2.w, b.t, t1);
    }
    const unsigned long long m0 = __builtin_amdgcn_ballot_w64(h0), m1 = __builtin_amdgcn_ballot_w64(h1);
    // a child's code, a leaf's negative; -1: reached by no lane
    const int c0 = m0 != 0ull ? __float_as_int(n3.x) : -1, c1 = m1 != 0ull ? __float_as_int(n3.y) : -1;
    if ((c0 | c1) >= 0) {
      const bool first0 = (__builtin_amdgcn_ballot_w64(t0 <= t1) & 1ull) != 0ull;
      const int nearc = first0 ? c0 : c1, farc = first0 ? c1 : c0;
      if (sp < 64) {
        stackv = lane == sp ? farc : stackv;
        ++sp;
      } else if (live) {
        atomicOr(flags, HDOF_FLAG_STACK_OVERFLOW);
      }
      cur = nearc;
      continue;
    }
    if (c0 < -1) {
      test_leaf_wave(r, tris, (unsigned)c0, m0, b);
      if (COUNT && h0) wk.tests += (int)(((unsigned)c0 >> 27) & 0xF) + 1;
    }
    if (c1 < -1) {
      test_leaf_wave(r, tris, (unsigned)c1, m1, b);
      if (COUNT && h1) wk.tests += (int)(((unsigned)c1 >> 27) & 0xF) + 1;
    }
    cur = max(c0, c1);
    if (cur < 0) {
      if (sp == 0) break;
      --sp;
      cur = __builtin_amdgcn_readlane(stackv, sp);
    }
  }
  return b;
}

// The wave's traversal: the signed form when the live lanes' directions
// share their signs on every axis (nearly every wave of pixel-adjacent
// rays), else the general one.  Both return the same closest hit.
template <bool COUNT>
__device__ inline Best traverse_wave_any(const float4* __restrict__ nodes, const float4* __restrict__ tris,
                                         int n_nodes, const Ray& r, bool live, int* __restrict__ flags, Work& wk) {
  const unsigned long long lm = __ballot(live);
  const unsigned long long sx = __ballot(live && signbit(r.inv.x)), sy = __ballot(live && signbit(r.inv.y)),
                           sz = __ballot(live && signbit(r.inv.z));
  if ((sx == 0ull || sx == lm) && (sy == 0ull || sy == lm) && (sz == 0ull || sz == lm)) {
    const int flip = (sx != 0ull ? 1 : 0) | (sy != 0ull ? 2 : 0) | (sz != 0ull ? 4 : 0);
    switch (flip) {
      case 0: return traverse_wave<COUNT, 0>(nodes, tris, n_nodes, r, live, flags, wk);
      case 1: return traverse_wave<COUNT, 1>(nodes, tris, n_nodes, r, live, flags, wk);
      case 2: return traverse_wave<COUNT, 2>(nodes, tris, n_nodes, r, live, flags, wk);
      case 3: return traverse_wave<COUNT, 3>(nodes, tris, n_nodes, r, live, flags, wk);
      case 4: return traverse_wave<COUNT, 4>(nodes, tris, n_nodes, r, live, flags, wk);
      case 5: return traverse_wave<COUNT, 5>(nodes, tris, n_nodes, r, live, flags, wk);
      case 6: return traverse_wave<COUNT, 6>(nodes, tris, n_nodes, r, live, flags, wk);
      default: return traverse_wave<COUNT, 7>(nodes, tris, n_nodes, r, live, flags, wk);
    }
  }
  return traverse_wave<COUNT, -1>(nodes, tris, n_nodes, r, live, flags, wk);
}

// Two-sided Lambertian face normal + point light, no shadow ray; with a
// specular table (k_s, shininess per input triangle) a Blinn-Phong lobe
// k_s I max(0, n.h)^shininess / max(d^2, 1e-4) is added while the light is
// on the viewer's side, h the unit half vector of the light direction and
// the direction back along the ray; ys = the lobe's luminance.
__device__ inline void shade(const float4* __restrict__ tris, const float* __restrict__ albedo,
                             const float2* __restrict__ spec, const LightK& li, V3 O, V3 D, const Best& b, V3& L,
                             V3& n, V3& alb, float& ys) {
  float4 a = tris[3 * b.tri], q = tris[3 * b.tri + 1], c = tris[3 * b.tri + 2];
  V3 e1 = V3{q.x - a.x, q.y - a.y, q.z - a.z};
  V3 e2 = V3{c.x - a.x, c.y - a.y, c.z - a.z};
  V3 nn = cross3(e1, e2);
  float il = rsqrtf(dot3(nn, nn));
  nn = il * nn;
  if (dot3(nn, D) > 0.0f) nn = V3{-nn.x, -nn.y, -nn.z};
  V3 P = V3{fmaf(b.t, D.x, O.x), fmaf(b.t, D.y, O.y), fmaf(b.t, D.z, O.z)};
  V3 l = li.p - P;
  float d2 = dot3(l, l);
  float cosv = d2 > 0.0f ? dot3(nn, l) * rsqrtf(d2) : 0.0f;
  float irr = fmaxf(0.0f, cosv) / fmaxf(d2, 1e-4f);
  const float* al = albedo + 3 * (size_t)b.id;
  alb = V3{al[0], al[1], al[2]};
  L = V3{alb.x * fmaf(li.I.x, irr, li.ka.x), alb.y * fmaf(li.I.y, irr, li.ka.y),
         alb.z * fmaf(li.I.z, irr, li.ka.z)};
  n = nn;
  ys = 0.0f;
  if (spec) {
    const float2 m = spec[b.id];
    if (m.x > 0.0f && cosv > 0.0f) {
      const float il2 = rsqrtf(d2), iD = rsqrtf(dot3(D, D));
      const V3 h = V3{fmaf(l.x, il2, -D.x * iD), fmaf(l.y, il2, -D.y * iD), fmaf(l.z, il2, -D.z * iD)};
      const float hh = dot3(h, h);
      const float nh = hh > 0.0f ? fmaxf(0.0f, dot3(nn, h) * rsqrtf(hh)) : 0.0f;
      const float f = m.x * powf(nh, m.y) / fmaxf(d2, 1e-4f);
      L = V3{fmaf(f, li.I.x, L.x), fmaf(f, li.I.y, L.y), fmaf(f, li.I.z, L.z)};
      ys = f * fmaf(0.2126f, li.I.x, fmaf(0.7152f, li.I.y, 0.0722f * li.I.z));
    }
  }
}

// PACK (frames with 16-pixel post-filter tiles): also the post-filter's
// packed texel (shaded rgb, signed CoC of the stored depth) and the block's
// maximum CoC radius, the block being the post-filter tile.
// spec_out (nullable): the specular luminance plane.
// One 16x16-pixel block lb of the image of camera k (its outputs planar
// [C][H][W] from the given pointers).
template <bool COUNT, bool PACK>
__device__ inline void gbuffer_block(const float4* __restrict__ nodes, const float4* __restrict__ tris, int n_nodes,
                                     const float* __restrict__ albedo, const float2* __restrict__ spec,
                                     float* __restrict__ spec_out, const CamK& k, const LensK& l, const LightK& li,
                                     int lb, float* __restrict__ depth, float* __restrict__ normal,
                                     float* __restrict__ alb_out, float* __restrict__ color, int* __restrict__ tri_id,
                                     int* __restrict__ flags, unsigned long long* __restrict__ counters,
                                     float4* __restrict__ pack, float* __restrict__ tile_r) {
  __shared__ float wmax[4];
  const int bx_n = (k.W + 15) >> 4;
  const int bx = lb % bx_n, by = lb / bx_n;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int x = bx * 16 + (wave & 1) * 8 + (lane & 7), y = by * 16 + (wave >> 1) * 8 + (lane >> 3);
  const bool live = x < k.W && y < k.H;
  V3 v = pixel_dir(k, live ? x : 0, live ? y : 0);
  Ray r = make_ray(k.e, V3{l.S1 * v.x, l.S1 * v.y, l.S1 * v.z});
  Work wk{0, 0};
  Best b = traverse_wave_any<COUNT>(nodes, tris, n_nodes, r, live, flags, wk);
  float rr = 0.0f;
  if (live) {
    if (COUNT) {
      atomicAdd(&counters[0], 1ull);
      atomicAdd(&counters[1], (unsigned long long)wk.visits);
      atomicAdd(&counters[2], (unsigned long long)wk.tests);
    }
    const size_t N = (size_t)k.W * k.H, p = (size_t)y * k.W + x;
    float z = HDOF_ZMAX, ys = 0.0f;
    V3 L = V3{0.0f, 0.0f, 0.0f};
    if (b.tri >= 0) {
      V3 n, a;
      shade(tris, albedo, spec, li, r.O, r.D, b, L, n, a, ys);
      z = b.t * l.S1;
      normal[p] = n.x;
      normal[N + p] = n.y;
      normal[2 * N + p] = n.z;
      alb_out[p] = a.x;
      alb_out[N + p] = a.y;
      alb_out[2 * N + p] = a.z;
      tri_id[p] = b.id;
    } else {
      for (int c = 0; c < 3; ++c) {
        normal[c * N + p] = 0.0f;
        alb_out[c * N + p] = 0.0f;
      }
      tri_id[p] = -1;
    }
    depth[p] = z;
    if (spec_out) spec_out[p] = ys;
    color[p] = L.x;
    color[N + p] = L.y;
    color[2 * N + p] = L.z;
    if (PACK) {
      const float c = coc_px(l, z);
      pack[p] = make_float4(L.x, L.y, L.z, c);
      rr = 0.5f * fabsf(c);
    }
  }
  if (PACK) {
    for (int o = 32; o > 0; o >>= 1) rr = fmaxf(rr, __shfl_xor(rr, o));
    if (lane == 0) wmax[wave] = rr;
    __syncthreads();
    if (t == 0) tile_r[lb] = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
  }
}

template <bool COUNT, bool PACK>
__global__ __launch_bounds__(256) void k_gbuffer(const float4* __restrict__ nodes,
                                                 const float4* __restrict__ tris, int n_nodes,
                                                 const float* __restrict__ albedo,
                                                 const float2* __restrict__ spec, float* __restrict__ spec_out,
                                                 CamK k, LensK l,
                                                 LightK li, float* __restrict__ depth,
                                                 float* __restrict__ normal, float* __restrict__ alb_out,
                                                 float* __restrict__ color, int* __restrict__ tri_id,
                                                 int* __restrict__ flags,
                                                 unsigned long long* __restrict__ counters,
                                                 float4* __restrict__ pack, float* __restrict__ tile_r) {
  const int nb = ((k.W + 15) >> 4) * ((k.H + 15) >> 4);
  gbuffer_block<COUNT, PACK>(nodes, tris, n_nodes, albedo, spec, spec_out, k, l, li, xcd_block(blockIdx.x, nb),
                             depth, normal, alb_out, color, tri_id, flags, counters, pack, tile_r);
}

// Writes the queue entries of a wave's 64 pixels, consecutive from p - lane
// (s entries holding p from o on; those outside [0, cap) dropped).  Called by
// whole waves; `own` is the wave's.  The pixels' entries follow one another
// in the queue (row-major offsets), so the lanes note their pixel's entries
// in LDS and the wave writes them lane by entry: by the pixels' lanes, each
// store touched a line per lane, s times over.  Bound: memory.  8.3M entries
// of 16 per pixel: 40 -> 10 us.  Pixels whose entries do not follow one
// another (offsets of a caller's own), or too few to share, write their own.
// (Not for frames and batches, whose few traced pixels it gained nothing.)
#define QW_N 512
__device__ inline void queue_write(uint8_t* own, int s, long o, int p, long cap, int* __restrict__ queue) {
  const int lane = threadIdx.x & 63;
  const unsigned long long am = __builtin_amdgcn_ballot_w64(s > 0);
  if (am == 0ull) return;
  const int first = __ffsll(am) - 1;
  const long o0 = (long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(o >> 32), first) << 32) |
                         (unsigned)__builtin_amdgcn_readlane((int)o, first));
  // each lane's entries start where the lanes' before it end
  int before = s;
  for (int i = 1; i < 64; i <<= 1) {
    const int n = __shfl_up(before, i);
    if (lane >= i) before += n;
  }
  const int n = __builtin_amdgcn_readlane(before, 63);
  before -= s;
  if (n < 128 || __builtin_amdgcn_ballot_w64(s > 0 && o != o0 + before) != 0ull) {
    for (int j = 0; j < s; ++j)
      if (o + j >= 0 && o + j < cap) queue[o + j] = p;
    return;
  }
  for (int c = 0; c < n; c += QW_N) {
    const int j1 = min(s, c + QW_N - before);
    for (int j = max(0, c - before); j < j1; ++j) own[before + j - c] = (uint8_t)lane;
    wave_order();
    for (int i = lane; i < QW_N && c + i < n; i += 64) {
      const long e = o0 + c + i;
      if (e >= 0 && e < cap) queue[e] = p - lane + own[i];
    }
    wave_order();
  }
}

// queue entries: pixel index repeated spp times at its offset; also resets
// the persistent trace's work counters (same stream, runs before the trace).
// Batched: offsets are view-local, *ebase is the view's first queue entry
// and the stored index is the pixel's position in the batch (pxbase + p).
// Entries outside [0, cap) are dropped: inconsistent offsets never write out
// of bounds.
__global__ __launch_bounds__(256) void k_queue_fill(const uint8_t* __restrict__ spp, const int* __restrict__ offsets,
                                                    int N, const int* __restrict__ ebase, int pxbase, long cap,
                                                    int* __restrict__ queue, int* __restrict__ counter) {
  __shared__ uint8_t own[4][QW_N];
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p < 8 * HDOF_SEG_STRIDE) counter[p] = 0;
  const int s = p < N ? spp[p] : 0;
  const long o = s > 0 ? (long)offsets[p] + (ebase ? *ebase : 0) : 0;
  queue_write(own[threadIdx.x >> 6], s, o, pxbase + p, cap, queue);
}

// Persistent trace.  The queue is cut into `segments` contiguous segments
// (bands of image rows; whole views in a batch), one per group of XCDs
// (blocks are dispatched round-robin over the 8 XCDs): a wave takes work
// from its own segment first, so each XCD's L2 holds the part of the BVH its
// rays touch, then moves on to the other segments.  Every wave exits once
// all segments are drained and its rays are done.
using ViewK = BatchView;  // the device copy of a batch's view table

struct TraceArgs {
  const float4* nodes;
  const float4* hnodes;
  const float* unit;
  const float4* tris;
  int n_nodes;
  const float* albedo;
  const float2* spec;  // nullable: Lambertian
  LightK li;
  const int* queue;
  const int* offsets;
  const int* total_p;
  int* counter;
  float* ray_col;
  float* ray_z;
  int* ray_id;
  size_t cap;
  int* flags;
  unsigned long long* counters;
  int refill, segments;
  int ray_quantum, n_cu, bpc;  // ray_quantum > 0: blocks kept per CU = ceil(rays / ray_quantum) in [1, bpc]
  ViewK v0;                // the view of a plain frame
  const ViewK* views;      // batch: device table of views
  const int* entry_base;   // batch: first queue entry of each view
  int n_views;
};

// The ray of queue entry ee of a segment ending at hi: its pixel from the
// queue, its sample index from the pixel's first entry, the lens sample
// from the view's counters.  False for an entry past hi or a corrupt pixel
// index.  pxb (batch): the first batch pixel of each view.
template <bool BATCH>
__device__ inline bool entry_ray(const TraceArgs& A, const int* pxb, int ee, int hi, V3& O, V3& D, float& S1) {
  const int g = ee < hi ? A.queue[ee] : -1;
  bool ok;
  int p, j;
  const ViewK* vk = &A.v0;
  if (BATCH) {
    // view of batch pixel g: last view whose first pixel is <= g
    int v = 0;
    for (int step = HDOF_MAX_VIEWS / 2; step >= 1; step >>= 1)
      if (v + step < A.n_views && pxb[v + step] <= g) v += step;
    vk = &A.views[v];
    p = g - pxb[v];
    ok = g >= 0 && p < vk->k.W * vk->k.H;
    j = ok ? ee - A.entry_base[v] - A.offsets[g] : 0;
  } else {
    p = g;
    ok = g >= 0 && g < A.v0.k.W * A.v0.k.H;
    j = ok ? ee - A.offsets[g] : 0;
  }
  if (!ok) return false;
  const CamK k = vk->k;
  const LensK l = vk->l;
  lens_ray(k, l, p % k.W, p / k.W, (uint32_t)j, vk->view, vk->seed, vk->frame, O, D);
  S1 = l.S1;
  return true;
}

// Shade the closest hit of a finished ray and store entry e's result.
__device__ inline void store_ray(const TraceArgs& A, V3 O, V3 D, const Best& b, float S1, int e) {
  float z = HDOF_ZMAX;
  V3 L = V3{0.0f, 0.0f, 0.0f};
  if (b.tri >= 0) {
    V3 n, a;
    float ys;
    shade(A.tris, A.albedo, A.spec, A.li, O, D, b, L, n, a, ys);
    z = b.t * S1;
  }
  A.ray_col[e] = L.x;
  A.ray_col[A.cap + e] = L.y;
  A.ray_col[2 * A.cap + e] = L.z;
  A.ray_z[e] = z;
  if (A.ray_id) A.ray_id[e] = b.tri >= 0 ? b.id : -1;
}

// The G-buffers of a batch in one launch (packed texels and tile radii
// too): the launch's blocks, in XCD-contiguous order over the whole batch,
// are the views' 16x16-pixel blocks one view after another; blk_base[v] is
// view v's first block (blk_base[n] the total), which is also its first
// post-filter tile.  A view's planes start at its first batch pixel.
struct GbBatch {
  int n;
  int blk_base[HDOF_MAX_VIEWS + 1];
};

__global__ __launch_bounds__(256) void k_gbuffer_batch(const float4* __restrict__ nodes,
                                                       const float4* __restrict__ tris, int n_nodes,
                                                       const float* __restrict__ albedo, LightK li,
                                                       const ViewK* __restrict__ views, GbBatch gbb,
                                                       float* __restrict__ depth, float* __restrict__ normal,
                                                       float* __restrict__ alb_out, float* __restrict__ color,
                                                       int* __restrict__ tri_id, int* __restrict__ flags,
                                                       float4* __restrict__ pack, float* __restrict__ tile_r) {
  const int g = xcd_block(blockIdx.x, gbb.blk_base[gbb.n]);
  const int v = batch_view_of(gbb.blk_base, gbb.n, g);
  const ViewK& vk = views[v];
  const size_t pb = (size_t)vk.px_base;
  gbuffer_block<false, true>(nodes, tris, n_nodes, albedo, nullptr, nullptr, vk.k, vk.l, li, g - gbb.blk_base[v],
                             depth + pb, normal + 3 * pb, alb_out + 3 * pb, color + 3 * pb, tri_id + pb, flags,
                             nullptr, pack + pb, tile_r + gbb.blk_base[v]);
}

// The blocks of the persistent trace that take part: with a ray quantum (a
// frame overlapping the trace with the post-filter gather) only the first
// ceil(total * n_cu / ray_quantum) blocks, one block per CU for every
// ray_quantum rays on average, so a light trace leaves CUs to the gather,
// but at least one block per CU and one per 64 rays (half a batch for each
// wave) while that is no more than 7 per CU, or while all blocks' waves can
// hold the whole queue as one batch each: fewer blocks make a longer trace,
// which the frame then waits for.  (Frames of 640x360 with 218k rays at 1.6 /
// 3.6 / 10 blocks per CU: 337 / 279 / 250 us; 1400x1050 with 693k at 5 / 7 /
// 10: 483 / 454 / 462; 400x300 with 73k at 1 / 3.6 / 4.5: 157 / 117 / 119.)
// Below 3 rays per 8 pixels the lower bounds but the first are left out.
// Large frames then wait for the gather, and more blocks beside it slow them
// (without / with the bounds, us: 1080p, 571k rays, 358 / 379; 370k, 337 /
// 365; 1440p, 0.10 to 0.34 rays per pixel, 543 / 570, 599 / 629, 696 / 714,
// 699 / 702).  The line is one of that size: smaller frames below it wait for
// the trace all the same and would gain by the bounds (960x540 with 141k
// rays 309 / 234, 168k 247 / 196; 1280x720 with 187k 332 / 271, 310k 367 /
// 286; 1080p with 287k rays of a wider scene 435 / 409).  The frames above
// the line have 0.39 to 3.8 rays per pixel.
// The first blocks are kept, so every queue segment keeps its blocks.
__device__ inline int kept_blocks(const TraceArgs& A, int total) {
  const long all = (long)A.bpc * A.n_cu;
  if (A.ray_quantum <= 0) return (int)all;
  const long light = ((long)total * A.n_cu + A.ray_quantum - 1) / A.ray_quantum;
  const bool few = 8l * total < 3l * A.v0.k.W * A.v0.k.H;
  const long most = few ? 0 : (total <= HDOF_TRACE_BLOCK * all ? all : 7l * A.n_cu);
  return (int)min(all, max(max((long)A.n_cu, light), min(most, (long)total / 64)));
}

// the kept blocks' waves whose own queue segment is seg
__device__ inline int waves_of(int kept, int segments, int seg) {
  return (kept - seg + segments - 1) / segments * (HDOF_TRACE_BLOCK / 64);
}

// The trace's arguments read anew from the kernel's argument segment (its
// only argument): what a refill derives from them is then not kept in
// registers through the traversal (141 vector registers otherwise).
__device__ __forceinline__ const TraceArgs* fresh_args() {
  const __attribute__((address_space(4))) char* p =
      (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return (const TraceArgs*)p;
}

// Entries handed out: per queue segment (one per XCD, the block's
// blockIdx.x mod segments) an atomic counter of entries taken; a wave whose
// segment runs dry moves on to the next and stops once it has found every
// segment dry.  (A look at all counters before each take, to skip the dry
// ones, makes every wave read the same lines: 241 -> 377 us on 947k rays.)
// Bound: the vector-memory path.  A dwordx4 load of 64 lanes takes a CU 16
// clocks whatever the mask (its data return was 87 % busy with four of them
// per node, the vector ALUs 71 %), so what counts is load instructions per
// ray: three per node since the boxes are halves, and more lanes in each.
// On 1.75M rays of a 1080p frame, alone: 533 -> 411 us; 8.3M rays of every
// pixel of 960x540 with their queue and reduction: 1617 -> 1447 us; the 1M
// triangles' 4.7M rays: 591 -> 526 us.  With the stack's top read beside the
// node, the far child written unconditionally and the choice between near,
// far and top made by masks instead of branches (each was a compare, a
// change of the exec mask and, for the pop, a second LDS wait): 368, 1304
// and 456 us.
// A wave holds up to 64 rays in LDS slots.  Each is set up, and once hit
// shaded and stored, by one lane each, 64 at a time; a lane that has
// finished a ray takes the next waiting slot, which costs the wave a few LDS
// reads instead of a ray's set-up (Philox block, lens sample, divisions), so
// lanes need not idle until the whole batch is done.  When no slot waits and
// the idle lanes number `refill` (at most HDOF_REFILL_MAX), the finished
// slots are shaded and refilled from the queue.
// (refill at 16 / 24 / 40 / 48 idle lanes: 528 / 493 / 462 / 442 us: rays of
// neighbouring entries that start together share their first loads' lines.)
// Traversal: box steps enter internal nodes (of two children that the ray
// reaches within the closest hit so far, the nearer becomes the entry and
// the other is pushed); a leaf step tests the entry's triangles.  The wave
// takes box steps while HDOF_MIN_BOX lanes have them to take, then the leaf
// step of the lanes that wait at a leaf (until the last lane, 8 or 20:
// 509 / 442 / 489 us).
// (five waves per SIMD: at 98 registers the batched form had four, and its
// batch took 7.37 ms instead of 7.27)
template <bool COUNT, bool BATCH>
__global__ __launch_bounds__(HDOF_TRACE_BLOCK, 5) void k_trace(TraceArgs A) {
  __shared__ PoolLds lds[HDOF_TRACE_BLOCK / 64];
  __shared__ int pxb[BATCH ? HDOF_MAX_VIEWS + 1 : 1];
  int spill[HDOF_SPILL_STACK];
  const int t = threadIdx.x, lane = t & 63;
  PoolLds& L = lds[__builtin_amdgcn_readfirstlane(t >> 6)];
  if (BATCH) {
    for (int v = t; v < A.n_views; v += HDOF_TRACE_BLOCK) pxb[v] = A.views[v].px_base;
    __syncthreads();
  }
  int total = *A.total_p;
  if (total < 0) total = 0;
  if ((size_t)total > A.cap) {
    if (blockIdx.x == 0 && t == 0) atomicOr(A.flags, HDOF_FLAG_CAPACITY);
    total = (int)A.cap;
  }
  const int kept = kept_blocks(A, total);
  if ((int)blockIdx.x >= kept) return;
  // A queue of which no wave gets more than one batch is shared out evenly,
  // without the counters (28k rays of 96x64 pixels: 148 -> 100 us; 218k of
  // 640x360: 163 -> 129): the largest segment over the fewest waves.
  const bool single = kept >= A.segments && ((long)total + A.segments - 1) / A.segments <=
                                                64l * waves_of(kept, A.segments, A.segments - 1);
  const int share = ((int)blockIdx.x / A.segments) * (HDOF_TRACE_BLOCK / 64) + __builtin_amdgcn_readfirstlane(t >> 6);
  const int refill = min(A.refill, HDOF_REFILL_MAX);
  const float unit = *A.unit;
  bool held = false, drained = false;  // held: the lane's slot holds a ray
  int seg = blockIdx.x % A.segments, tried = 0;
  int next = 0, count = 0;  // the waiting slots are list[next .. count)
  // the lane's ray: its slot (-1: none), the entry to visit next (a node, or
  // a leaf code), the stack's top (a row of stk, row 0 its bottom), the
  // closest hit
  // (as a byte offset from lds: the stack is addressed with no arithmetic)
  const int tp0 = (int)((t >> 6) * sizeof(PoolLds) + offsetof(PoolLds, stk)) + 4 * lane;
  const int tp_full = tp0 + 256 * HDOF_LDS_STACK;  // the last row's
  const auto stk = [&](int at) -> int& { return *(int*)((char*)lds + at); };
  int slot = -1, tp = tp0;
  unsigned cur = TRAV_DONE;
  Best b = Best{INFINITY, -1, 0x7fffffff};
  unsigned long long strict = 0ull;  // lanes that test their leaves' boxes
  // box steps since a ray of the wave was last done, and what they are bounded by
  unsigned stall = 0;
  const unsigned stall_max = (unsigned)min(64ll * (A.n_nodes + 1ll), 0xfffffff0ll);
  Work wk{0, 0};
  stk(tp0) = (int)TRAV_DONE;
  for (;;) {
    const unsigned long long idle = __builtin_amdgcn_ballot_w64(slot < 0);
    const unsigned long long lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    if (next >= count && (int)__popcll(idle) >= (drained ? 64 : refill)) {
      wave_order();
      const TraceArgs& B = *fresh_args();
      bool redo = false;
      const int state = __float_as_int(L.f[SLOT_DONE][lane]);
      if (held && (state & 1)) {
        const Best h = Best{L.f[SLOT_HIT][lane], __float_as_int(L.f[SLOT_HIT + 1][lane]),
                            __float_as_int(L.f[SLOT_HIT + 2][lane])};
        const V3 O = slot_v3(L, SLOT_O, lane), D = slot_v3(L, SLOT_D, lane);
        // A hit on a triangle whose leaf's box the ray misses (at an edge) is
        // none for a walk by full boxes.  A ray that misses the triangle's
        // own box is walked again with every leaf's box tested, as full boxes
        // do, so the hits are those of full boxes (without it 4 of 18M rays
        // differed; the check costs the trace 1 to 2 %).  Far from the origin
        // the full boxes' own rounding decides more hits, and two walks by
        // them in another order differ too: 5 of 461k rays at 10^4 units, as
        // many as differ here.
        if (state == 1 && h.tri >= 0) {
          Ray q;
          q.inv = slot_v3(L, SLOT_INV, lane);
          q.oinv = V3{-O.x * q.inv.x, -O.y * q.inv.y, -O.z * q.inv.z};
          redo = !tris_box_hit(q, B.tris, h.tri, 1, INFINITY);
        }
        if (!redo) store_ray(B, O, D, h, L.f[SLOT_S1][lane], __float_as_int(L.f[SLOT_ENTRY][lane]));
        held = redo;
      }
      const bool any_redo = __builtin_amdgcn_ballot_w64(redo) != 0ull;
      if (any_redo && redo) slot_ray(L, lane, slot_v3(L, SLOT_O, lane), slot_v3(L, SLOT_D, lane), 2);
      if (drained && !any_redo) break;
      const unsigned long long fm = __builtin_amdgcn_ballot_w64(!held);
      int want = (int)__popcll(fm);
      const int nseg = B.segments;
      const int lo = (int)((long)total * seg / nseg), hi = (int)((long)total * (seg + 1) / nseg);
      int base = 0;
      if (drained) {  // only rays to be walked again
        want = 0;
      } else if (single) {
        // the wave's only batch: its share of the segment
        const int nw = waves_of(kept, nseg, seg);
        base = lo + (int)((long)(hi - lo) * share / nw);
        want = min(want, lo + (int)((long)(hi - lo) * (share + 1) / nw) - base);
        drained = true;
      } else {
        if (lane == 0) base = atomicAdd(&B.counter[seg * HDOF_SEG_STRIDE], want);
        base = __builtin_amdgcn_readfirstlane(base) + lo;
        if (base + want >= hi) {  // this segment is used up: go on to the next one
          seg = seg + 1 == nseg ? 0 : seg + 1;
          drained = ++tried == nseg;
        }
      }
      bool got = false;
      const int nth = (int)__popcll(fm & lt_mask);
      if (!held && nth < want) {
        const int e = base + nth;
        V3 O, D;
        float S1;
        got = entry_ray<BATCH>(B, pxb, e, hi, O, D, S1);
        if (got) {
          L.f[SLOT_S1][lane] = S1;
          L.f[SLOT_ENTRY][lane] = __int_as_float(e);
          slot_ray(L, lane, O, D, 0);
          held = true;
        }
      }
      got = got || redo;
      const unsigned long long gm = __builtin_amdgcn_ballot_w64(got);
      if (got) L.list[__popcll(gm & lt_mask)] = lane;
      next = 0;
      count = (int)__popcll(gm);
      wave_order();
    }
    if (next < count) {  // hand the waiting slots to the idle lanes
      const int i = next + (int)__popcll(idle & lt_mask);
      const bool fresh = slot < 0 && i < count;
      if (fresh) {
        slot = L.list[i];
        b = Best{INFINITY, -1, 0x7fffffff};
        cur = 0;  // root
        tp = tp0;
      }
      strict |= __builtin_amdgcn_ballot_w64(fresh && __float_as_int(L.f[SLOT_DONE][slot < 0 ? lane : slot]) == 2);
      next = min(count, next + (int)__popcll(idle));
    }
    const int sl = slot < 0 ? lane : slot;
    const Ray r = ray_of(RayPre{slot_v3(L, SLOT_O, sl), V3{0.f, 0.f, 0.f}, slot_v3(L, SLOT_INV, sl),
                                L.f[SLOT_SX][sl], L.f[SLOT_SY][sl], __float_as_int(L.f[SLOT_AXES][sl])});
    const V3 sinv = V3{r.inv.x * unit, r.inv.y * unit, r.inv.z * unit};
    const int rx = signbit(r.inv.x) ? 16 : 0, ry = signbit(r.inv.y) ? 16 : 0, rz = signbit(r.inv.z) ? 16 : 0;
    for (;;) {  // walk until lanes can be given rays
      const unsigned long long busy = __builtin_amdgcn_ballot_w64(slot >= 0);
      for (;;) {
        const bool inner = !(cur & HDOF_LEAF_BIT);
        const unsigned long long im = __builtin_amdgcn_ballot_w64(inner);
        if (lanes(im) < (im == busy ? 1 : HDOF_MIN_BOX)) break;
        // each internal node is entered at most once per ray: more steps
        // than the wave's rays can take before one of them is done mean a
        // malformed tree, and the rays stop here
        if (++stall > stall_max) {
          if (lane == 0) atomicOr(A.flags, HDOF_FLAG_STACK_OVERFLOW);
          cur = TRAV_DONE;
          break;
        }
        if (inner) {
          // no branch but a uniform one: the stack's top (below the first
          // entry: TRAV_DONE) is read with the node, and the other child is
          // written above it whether it will be used or not
          if (COUNT) wk.visits++;
          const char* nd = (const char*)A.hnodes + (cur << 4);
          const float4 n0 = *(const float4*)nd, n1 = *(const float4*)(nd + 16);
          const float3 n2 = *(const float3*)(nd + 32);
          const bool deep = __builtin_amdgcn_ballot_w64(tp >= tp_full) != 0ull;
          const int ti = min(tp, tp_full);
          unsigned top = (unsigned)stk(ti);
          const V3 base = V3{fmaf(n0.x, sinv.x, r.oinv.x), fmaf(n0.y, sinv.y, r.oinv.y), fmaf(n0.z, sinv.z, r.oinv.z)};
          float t0, t1;
          const unsigned long long h0 = __builtin_amdgcn_ballot_w64(
              box_hit_half(__float_as_uint(n1.x), __float_as_uint(n1.z), __float_as_uint(n2.x), sinv, base, rx, ry, rz,
                           b.t, t0));
          const unsigned long long h1 = __builtin_amdgcn_ballot_w64(
              box_hit_half(__float_as_uint(n1.y), __float_as_uint(n1.w), __float_as_uint(n2.y), sinv, base, rx, ry, rz,
                           b.t, t1));
          const unsigned long long le = __builtin_amdgcn_ballot_w64(t0 <= t1);
          const bool near0 = lane_of(h0 & (~h1 | le)), both = lane_of(h0 & h1), any = lane_of(h0 | h1);
          const unsigned c0 = __float_as_uint(n2.z), c1 = __float_as_uint(n0.w);
          const unsigned far = near0 ? c1 : c0;
          stk(ti + 256) = (int)far;
          if (deep) {  // entries in the spill array
            const int e = (tp - tp_full) >> 8;
            if (e > 0) top = (unsigned)spill[e - 1];
            if (both && e >= 0) {
              if (e < HDOF_SPILL_STACK)
                spill[e] = (int)far;
              else
                atomicOr(A.flags, HDOF_FLAG_STACK_OVERFLOW), tp -= 256;
            }
          }
          cur = any ? (near0 ? c0 : c1) : top;
          tp += both ? 256 : 0;
          tp -= any ? 0 : 256;
        }
      }
      if ((cur & HDOF_LEAF_BIT) && cur != TRAV_DONE) {
        unsigned top = (unsigned)stk(min(tp, tp_full));
        if (strict == 0ull || !lane_of(strict) ||
            tris_box_hit(r, A.tris, (int)(cur & HDOF_LEAF_FIRST_MASK), (int)((cur >> 27) & 0xF) + 1, b.t))
          test_leaf(r, A.tris, cur, b);
        if (COUNT) wk.tests += (int)((cur >> 27) & 0xF) + 1;
        const int e = (tp - tp_full) >> 8;
        if (e > 0) top = (unsigned)spill[e - 1];
        cur = top;
        tp -= 256;
      }
      const bool done = slot >= 0 && cur == TRAV_DONE;
      if (done) {  // the stack is empty: the ray's hit goes to its slot
        L.f[SLOT_HIT][slot] = b.t;
        L.f[SLOT_HIT + 1][slot] = __int_as_float(b.tri);
        L.f[SLOT_HIT + 2][slot] = __int_as_float(b.id);
        L.f[SLOT_DONE][slot] = __int_as_float(strict != 0ull && lane_of(strict) ? 3 : 1);
        slot = -1;
        if (COUNT) {  // a second walk is no other ray, but its work counts
          if (!lane_of(strict)) atomicAdd(&A.counters[3], 1ull);
          atomicAdd(&A.counters[4], (unsigned long long)wk.visits);
          atomicAdd(&A.counters[5], (unsigned long long)wk.tests);
          wk = Work{0, 0};
        }
      }
      const unsigned long long dm = __builtin_amdgcn_ballot_w64(done);
      if (dm != 0ull) stall = 0;
      strict &= ~dm;
      // (also met by a wave that was given no ray at all)
      const int nidle = (int)__popcll(__builtin_amdgcn_ballot_w64(slot < 0));
      if (nidle >= (next < count ? HDOF_HAND_OUT : (drained ? 64 : refill))) break;
    }
  }
}

// Wave-coherent form: a wave takes 64 consecutive entries of its segment at
// a time (the samples of a few neighbouring pixels, whose rays differ by
// their lens offsets) and walks the union of their paths with wave-uniform
// node loads (traverse_wave_any), then shades and stores them; no per-lane
// refill and no LDS stack.  Same hand-out of entries as k_trace, so the
// same results.
template <bool COUNT, bool BATCH>
__global__ __launch_bounds__(HDOF_TRACE_BLOCK, HDOF_TRACE_WAVES_PER_EU) void k_trace_wave(TraceArgs A) {
  __shared__ int pxb[HDOF_MAX_VIEWS + 1];
  const int t = threadIdx.x, lane = t & 63;
  if (BATCH) {
    for (int v = t; v < A.n_views; v += HDOF_TRACE_BLOCK) pxb[v] = A.views[v].px_base;
    __syncthreads();
  }
  int total = *A.total_p;
  if (total < 0) total = 0;
  if ((size_t)total > A.cap) {
    if (blockIdx.x == 0 && t == 0) atomicOr(A.flags, HDOF_FLAG_CAPACITY);
    total = (int)A.cap;
  }
  if ((int)blockIdx.x >= kept_blocks(A, total)) return;
  const int nseg = A.segments;
  int seg = blockIdx.x % nseg, tried = 0;
  while (tried < nseg) {
    const int lo = (int)((long)total * seg / nseg), hi = (int)((long)total * (seg + 1) / nseg);
    int base = 0;
    if (lane == 0) base = atomicAdd(&A.counter[seg * HDOF_SEG_STRIDE], 64);
    base = __shfl(base, 0) + lo;
    if (base >= hi) {  // this segment is used up: go on to the next one
      seg = seg + 1 == nseg ? 0 : seg + 1;
      ++tried;
      continue;
    }
    const int e = base + lane;
    V3 O = V3{0.0f, 0.0f, 0.0f}, D = V3{0.0f, 0.0f, 1.0f};
    float S1 = A.v0.l.S1;
    const bool live = entry_ray<BATCH>(A, pxb, e, hi, O, D, S1);
    const Ray r = make_ray(O, D);
    Work wk{0, 0};
    const Best b = traverse_wave_any<COUNT>(A.nodes, A.tris, A.n_nodes, r, live, A.flags, wk);
    if (live) {
      store_ray(A, r.O, r.D, b, S1, e);
      if (COUNT) {
        atomicAdd(&A.counters[3], 1ull);
        atomicAdd(&A.counters[4], (unsigned long long)wk.visits);
        atomicAdd(&A.counters[5], (unsigned long long)wk.tests);
      }
    }
  }
}

// A ray's terms in its pixel's sums (om: its lens sample's weight, 1 without
// spherical aberration; w: the share of the near plane) and the sums.
struct RtRay {
  float R, G, B, c, w, om;
  float pw;  // FARPOS: the far share of a ray that hit, at the point P
  V3 P;
};

struct RtSums {
  float Nw = 0.f, Fw = 0.f, Sw = 0.f, scn = 0.f, scf = 0.f;
  float snr = 0.f, sng = 0.f, snb = 0.f, sfr = 0.f, sfg = 0.f, sfb = 0.f, sy = 0.f, sy2 = 0.f;
  float Pw = 0.f, px = 0.f, py = 0.f, pz = 0.f;
  template <bool FARPOS>
  __device__ __forceinline__ void add(const RtRay& q) {
    const float wf = q.om - q.w;
    if (FARPOS) {
      Pw += q.pw;
      px = fmaf(q.pw, q.P.x, px);
      py = fmaf(q.pw, q.P.y, py);
      pz = fmaf(q.pw, q.P.z, pz);
    }
    Sw += q.om;
    Nw += q.w;
    Fw += wf;
    scn = fmaf(q.w, fabsf(q.c), scn);
    scf = fmaf(wf, fabsf(q.c), scf);
    snr = fmaf(q.w, q.R, snr);
    sng = fmaf(q.w, q.G, sng);
    snb = fmaf(q.w, q.B, snb);
    sfr = fmaf(wf, q.R, sfr);
    sfg = fmaf(wf, q.G, sfg);
    sfb = fmaf(wf, q.B, sfb);
    const float Y = fmaf(0.2126f, q.R, fmaf(0.7152f, q.G, 0.0722f * q.B));
    sy = fmaf(q.om, Y, sy);
    sy2 = fmaf(q.om * Y, Y, sy2);
  }
};

struct RtIn {
  const float *ray_col, *ray_z;
  size_t cap;
  LensK l;
  CamK k;
  uint32_t seed, frame, view;
};

// the share of the near plane of a ray with CoC c
__device__ __forceinline__ float rt_near(float c) { return clamp01(fmaf(-c, 0.35355339059327376f, 0.5f)); }

__device__ __forceinline__ float4 rt_load(const RtIn& A, size_t e) {
  return make_float4(A.ray_col[e], A.ray_col[A.cap + e], A.ray_col[2 * A.cap + e], A.ray_z[e]);
}

// An entry (colour and depth), the j-th ray of pixel p.  RAYS (FARPOS, or
// spherical aberration): the ray is regenerated from its counters (t = z /
// S1, since the direction's forward component is S1).
template <bool FARPOS, bool RAYS>
__device__ __forceinline__ RtRay rt_ray(const RtIn& A, const float4& in, int p, int j) {
  RtRay q;
  q.R = in.x;
  q.G = in.y;
  q.B = in.z;
  const float z = in.w;
  q.c = coc_px(A.l, z);
  q.om = 1.0f;
  V3 O, D;
  if (RAYS)
    lens_ray(A.k, A.l, p % A.k.W, p / A.k.W, (uint32_t)j, A.view, A.seed, A.frame, O, D, &q.om);
  q.w = q.om * rt_near(q.c);
  q.pw = 0.f;
  q.P = V3{0.f, 0.f, 0.f};
  if (FARPOS && z < HDOF_ZMAX) {
    const float t = z * A.l.invS1;
    q.pw = q.om - q.w;
    q.P = V3{fmaf(t, D.x, O.x), fmaf(t, D.y, O.y), fmaf(t, D.z, O.z)};
  }
  return q;
}

// One wave's staged entries (colour and CoC, structure of arrays, index i at
// i + i / 64: pixels of 4, 8 or 16 entries then read from different banks).
#define RTS_T 64
#define RTS_N 256  // (128: trace and reduction of 8.3M rays 12 us slower)
#define RTS_AT(i) ((i) + ((i) >> 6))
// Above RTS_SPP entries a pixel few of the wave's lanes have entries in a
// chunk, and add them one by one: worth it only where other waves fill the
// time.  Counts of 255, pixels' lanes / staged: 64x64 pixels 240 / 2790 us,
// 320x180 401 / 2195, 480x270 2282 / 1202, 640x360 3611 / 2027; 32: 17 / 52,
// 35 / 36, 288 / 31, 426 / 44; 16: 9 / 10, 11 / 11, 24 / 12, 93 / 16.
#define RTS_SPP 16
#define RTS_BLOCKS 256  // of 256 pixels: a wave for each SIMD
struct RtStage {
  float v[4][RTS_AT(RTS_N)];
};

// The sums of the wave's 64 pixels p (consecutive, one per lane; s entries
// from o on, all inside the queue).  STAGE: their entries lie together in the
// queue (row-major offsets), so the wave reads them lane by entry and the
// pixels' lanes add them up from LDS in the order of their rays: read by the
// pixels' lanes, every load touches a line per lane, s times over.  Bound:
// memory.  8.3M rays of every pixel of 960x540: 243 -> 27 us (133 MB of
// entries, 19 MB of planes).  A pixel's lane reads its own entries where a
// wave has fewer than RTS_T, where they are spread over more than 64
// pixels can have (offsets of a caller's own), and where a small image has
// many per pixel.  Not staged: frames and
// batches, whose reduction runs beside the post-filter's gather (the kernel
// alone 313 -> 236 us for sixteen views and 38 -> 36 for a 1080p frame, but
// the whole calls 7.31 -> 7.34 ms and 692 -> 697 us: the gather keeps the LDS
// and sets the pace), and regenerated rays (RAYS: their arithmetic is the
// larger part; staged per entry 106 -> 137 us for 4.7M rays).
template <bool FARPOS, bool RAYS, bool STAGE>
__device__ __forceinline__ RtSums rt_sums(RtStage* S, const RtIn& A, int p, int s, long o) {
  RtSums t;
  const unsigned long long am = __builtin_amdgcn_ballot_w64(s > 0);
  if (am == 0ull) return t;
  const int lane = threadIdx.x & 63, first = __ffsll(am) - 1;
  const long o0 = (long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(o >> 32), first) << 32) |
                         (unsigned)__builtin_amdgcn_readlane((int)o, first));
  const long rel = s > 0 ? o - o0 : 0;
  int lo = 0, hi = -1;
  if (STAGE && __builtin_amdgcn_ballot_w64(rel > (1l << 24) || rel < -(1l << 24)) == 0ull) {
    lo = s > 0 ? (int)rel : 0x7fffffff;
    hi = s > 0 ? (int)rel + s : -0x7fffffff;
    for (int i = 32; i > 0; i >>= 1) {
      lo = min(lo, __shfl_xor(lo, i));
      hi = max(hi, __shfl_xor(hi, i));
    }
  }
  if (hi - lo > 64 * 255 || hi - lo < RTS_T || (hi - lo > 64 * RTS_SPP && gridDim.x < RTS_BLOCKS)) {
    for (int j = 0; j < s; ++j) t.add<FARPOS>(rt_ray<FARPOS, RAYS>(A, rt_load(A, (size_t)(o + j)), p, j));
    return t;
  }
  const int d = (int)rel;
  for (int c = lo; c < hi; c += RTS_N) {
    float4 in[RTS_N / 64];  // all of a chunk's loads before their use
#pragma unroll
    for (int b = 0; b < RTS_N / 64; ++b) in[b] = rt_load(A, (size_t)(o0 + min(c + b * 64 + lane, hi - 1)));
#pragma unroll
    for (int b = 0; b < RTS_N / 64; ++b) {
      const int at = RTS_AT(b * 64 + lane);
      S->v[0][at] = in[b].x;
      S->v[1][at] = in[b].y;
      S->v[2][at] = in[b].z;
      S->v[3][at] = coc_px(A.l, in[b].w);
    }
    wave_order();
    const int j0 = max(0, c - d), j1 = min(s, c + RTS_N - d);  // this lane's entries of the chunk
    for (int j = j0; j < j1; ++j) {
      const int at = RTS_AT(d + j - c);
      const float c = S->v[3][at];
      t.add<FARPOS>(RtRay{S->v[0][at], S->v[1][at], S->v[2][at], c, rt_near(c), 1.0f, 0.f, V3{0.f, 0.f, 0.f}});
    }
    wave_order();
  }
  return t;
}

// per-pixel near/far split, hit ratio and luminance moments, fixed order;
// batched: *ebase is the view's first queue entry
// FARPOS: also the far-weighted mean hit point of the pixel's rays that hit
// and its weight, 4 planes.
// VAR (whole frames): the variance history update of the pixel as well,
// from the moments just formed.
// coc_nf (nullable, 2 planes): the average CoC size of the near rays and of
// the far rays, sum w |c| / sum w and sum (1 - w) |c| / sum (1 - w).
// Called by whole waves, the lanes' pixels consecutive; p >= N: none.
template <bool FARPOS, bool VAR, bool RAYS, bool STAGE>
__device__ __forceinline__ void rt_reduce_px(RtStage* S, const RtIn& A, int p,
                                             const uint8_t* __restrict__ spp, const int* __restrict__ offsets, int N,
                                             const int* __restrict__ ebase, float* __restrict__ cn,
                                             float* __restrict__ cf, float* __restrict__ h, float* __restrict__ m1,
                                             float* __restrict__ m2, float* __restrict__ far_pos, const VarFuse& vf,
                                             float* __restrict__ coc_nf) {
  const bool px = p < N;
  const int sp = px ? spp[p] : 0;
  int s = sp;
  // untraced pixels (most of them) do not read their offset
  const long o = s > 0 ? (long)offsets[p] + (ebase ? *ebase : 0) : 0;
  if (o < 0 || o + s > (long)A.cap) s = 0;  // inconsistent offsets: nothing was traced here
  const RtSums t = rt_sums<FARPOS, RAYS, STAGE>(S, A, p, s, o);
  if (!px) return;
  const float Nw = t.Nw, Fw = t.Fw, Sw = t.Sw;
  const float in_ = Nw > 0.f ? 1.0f / Nw : 0.f, if_ = Fw > 0.f ? 1.0f / Fw : 0.f;
  const float is = Sw > 0.f ? 1.0f / Sw : 0.f;
  const float ybar = t.sy * is, y2bar = t.sy2 * is;
  if (!vf.sparse_rt || sp > 0) {
    cn[p] = t.snr * in_;
    cn[N + p] = t.sng * in_;
    cn[2 * (size_t)N + p] = t.snb * in_;
    cf[p] = t.sfr * if_;
    cf[N + p] = t.sfg * if_;
    cf[2 * (size_t)N + p] = t.sfb * if_;
    h[p] = Nw * is;
    m1[p] = ybar;
    m2[p] = y2bar;
  }
  if (VAR && !(vf.in_place && sp == 0)) {  // in place: an untraced pixel's history is already there
    float a1 = vf.rm1[p], a2 = vf.rm2[p];
    uint8_t f = vf.rfl[p];
    if (sp > 0) {
      if (f & HDOF_HIST_VALID) {
        a1 = fmaf(vf.alpha, ybar, (1.0f - vf.alpha) * a1);
        a2 = fmaf(vf.alpha, y2bar, (1.0f - vf.alpha) * a2);
        f = HDOF_HIST_VALID;
      } else {
        a1 = ybar;
        a2 = y2bar;
        f = HDOF_HIST_VALID | HDOF_HIST_NEW;
      }
    }
    vf.m1[p] = a1;
    vf.m2[p] = a2;
    vf.fl[p] = f;
    if (!vf.in_place) vf.hz[p] = vf.depth[p];
  }
  if (FARPOS) {
    const float ip = t.Pw > 0.f ? 1.0f / t.Pw : 0.f;
    far_pos[p] = t.px * ip;
    far_pos[N + p] = t.py * ip;
    far_pos[2 * (size_t)N + p] = t.pz * ip;
    far_pos[3 * (size_t)N + p] = t.Pw;
  }
  if (coc_nf) {
    coc_nf[p] = t.scn * in_;
    coc_nf[N + p] = t.scf * if_;
  }
}

template <bool FARPOS, bool VAR, bool RAYS>
__global__ __launch_bounds__(256) void k_rt_reduce(RtIn A, const uint8_t* __restrict__ spp,
                                                   const int* __restrict__ offsets, int N,
                                                   const int* __restrict__ ebase, float* __restrict__ cn,
                                                   float* __restrict__ cf, float* __restrict__ h,
                                                   float* __restrict__ m1, float* __restrict__ m2,
                                                   float* __restrict__ far_pos, VarFuse vf,
                                                   float* __restrict__ coc_nf) {
  constexpr bool STAGE = !RAYS && !VAR;
  __shared__ RtStage stage[STAGE ? 4 : 1];
  rt_reduce_px<FARPOS, VAR, RAYS, STAGE>(stage + (STAGE ? threadIdx.x >> 6 : 0), A, blockIdx.x * 256 + threadIdx.x, spp, offsets, N, ebase, cn,
                            cf, h, m1, m2, far_pos, vf, coc_nf);
}

// The batched form's queue fill and reduction, one launch each over every
// view: blocks of HDOF_BATCH_PX_BLOCK pixels (256 threads, a pixel every
// 256), view v's from blk_base[v] (blk_base[n] the total), its pixels from
// its px_base and its queue entries from ebase[v].
struct PxBatch {
  int n;
  int blk_base[HDOF_MAX_VIEWS + 1];
};

__global__ void k_queue_fill_batch(const uint8_t* __restrict__ spp, const int* __restrict__ offsets,
                                   const ViewK* __restrict__ views, PxBatch b, const int* __restrict__ ebase,
                                   long cap, int* __restrict__ queue, int* __restrict__ counter) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < 8 * HDOF_SEG_STRIDE; i += blockDim.x) counter[i] = 0;
  const int v = batch_view_of(b.blk_base, b.n, blockIdx.x);
  const int N = views[v].k.W * views[v].k.H, pb = views[v].px_base;
  const int e0 = ebase[v];
  const int p0 = (blockIdx.x - b.blk_base[v]) * HDOF_BATCH_PX_BLOCK;
  for (int i = threadIdx.x; i < HDOF_BATCH_PX_BLOCK; i += blockDim.x) {
    const int p = p0 + i;
    if (p >= N) break;
    const int s = spp[pb + p];
    if (s == 0) continue;
    const long o = (long)offsets[pb + p] + e0;
    for (int j = 0; j < s; ++j)
      if (o + j >= 0 && o + j < cap) queue[o + j] = pb + p;
  }
}

// the trace planes are written at traced pixels only (the composite reads
// them nowhere else)
__global__ __launch_bounds__(256) void k_rt_reduce_batch(const uint8_t* __restrict__ spp,
                                                         const int* __restrict__ offsets,
                                                         const ViewK* __restrict__ views, PxBatch b,
                                                         const int* __restrict__ ebase,
                                                         const float* __restrict__ ray_col,
                                                         const float* __restrict__ ray_z, size_t cap,
                                                         float* __restrict__ cn, float* __restrict__ cf,
                                                         float* __restrict__ h, float* __restrict__ m1,
                                                         float* __restrict__ m2) {
  const int v = batch_view_of(b.blk_base, b.n, blockIdx.x);
  const int N = views[v].k.W * views[v].k.H;
  const size_t pb = (size_t)views[v].px_base;
  // (the rays' lens weights are not regenerated here: sa = 0)
  const RtIn A{ray_col, ray_z, cap, views[v].l, views[v].k, 0u, 0u, 0u};
  VarFuse vf{};
  vf.sparse_rt = 1;
  const int p0 = (blockIdx.x - b.blk_base[v]) * HDOF_BATCH_PX_BLOCK;
  for (int i = threadIdx.x; i < HDOF_BATCH_PX_BLOCK; i += 256)
    rt_reduce_px<false, false, false, false>(nullptr, A, p0 + i, spp + pb, offsets + pb, N, ebase + v, cn + 3 * pb,
                               cf + 3 * pb, h + pb, m1 + pb, m2 + pb, nullptr, vf, nullptr);
}

// batch: first queue entry of each view and the batch total
__global__ void k_view_scan(const int* __restrict__ totals, int n, int* __restrict__ ebase,
                            int* __restrict__ grand) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  long run = 0;
  for (int v = 0; v < n; ++v) {
    ebase[v] = (int)run;
    run += totals[v];
  }
  *grand = (int)min(run, (long)0x7fffffff);
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

template <bool BATCH>
void launch_trace_kernel(hdof_ctx* ctx, const TraceArgs& A, hipStream_t st) {
  const int grid = ctx->n_cu * ctx->tune.blocks_per_cu;
  void (*kern)(TraceArgs);
  // automatic form: by the scene's triangle count (n_nodes + 1 for the binary tree)
  const bool wave = ctx->tune.wave == 1 || (ctx->tune.wave == 2 && A.n_nodes + 1 >= HDOF_WAVE_AUTO_TRIS);
  if (wave)
    kern = ctx->count_on ? k_trace_wave<true, BATCH> : k_trace_wave<false, BATCH>;
  else
    kern = ctx->count_on ? k_trace<true, BATCH> : k_trace<false, BATCH>;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(HDOF_TRACE_BLOCK), 0, st, A);
}

__global__ void k_zero_f(float* __restrict__ a, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0.0f;
}

TraceArgs base_args(hdof_ctx* ctx, const hdof_scene* sc, const LightK& li, size_t cap) {
  TraceArgs A{};
  A.nodes = sc->nodes;
  A.hnodes = sc->hnodes;
  A.unit = sc->unit;
  A.tris = sc->tris;
  A.n_nodes = sc->n_nodes;
  A.albedo = sc->albedo;
  A.spec = (const float2*)sc->spec;
  A.li = li;
  A.queue = (const int*)ctx->queue.p;
  A.counter = (int*)ctx->work_counter.p;
  A.ray_col = (float*)ctx->ray_col.p;
  A.cap = cap;
  A.flags = ctx->d_flags;
  A.counters = ctx->d_counters;
  A.refill = ctx->tune.refill;
  A.segments = ctx->tune.segments;
  A.ray_quantum = ctx->trace_ray_quantum;
  A.n_cu = ctx->n_cu;
  A.bpc = ctx->tune.blocks_per_cu;
  return A;
}

}  // namespace

// done (nullable): an event the G-buffer's own dispatch completes (its
// completion signal, with no marker packet between it and the next kernel
// on st)
hdof_status launch_gbuffer(hdof_ctx* ctx, const hdof_scene* sc, const CamK& k, const LensK& l,
                           const LightK& li, hdof_gbuffer_bufs out, hipStream_t st, float4* pack, float* tile_r,
                           hipEvent_t done) {
  int nb = cdiv(k.W, 16) * cdiv(k.H, 16);
  auto kern = ctx->count_on ? (pack ? k_gbuffer<true, true> : k_gbuffer<true, false>)
                            : (pack ? k_gbuffer<false, true> : k_gbuffer<false, false>);
  if (done)
    hipExtLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, st, nullptr, done, 0, sc->nodes, sc->tris, sc->n_nodes,
                          sc->albedo, (const float2*)sc->spec, sc->spec ? out.spec : nullptr, k, l, li, out.depth,
                          out.normal, out.albedo, out.color, out.tri_id, ctx->d_flags, ctx->d_counters, pack,
                          tile_r);
  else
    hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, st, sc->nodes, sc->tris, sc->n_nodes, sc->albedo,
                       (const float2*)sc->spec, sc->spec ? out.spec : nullptr, k, l, li, out.depth, out.normal,
                       out.albedo, out.color, out.tri_id, ctx->d_flags, ctx->d_counters, pack, tile_r);
  // a Lambertian scene has no specular part: its plane is 0
  if (!sc->spec && out.spec) hipLaunchKernelGGL(k_zero_f, dim3(cdiv(k.W * k.H, 256)), dim3(256), 0, st, out.spec,
                                                k.W * k.H);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

hdof_status launch_gbuffer_batched(hdof_ctx* ctx, const hdof_scene* sc, const LightK& li, int n_views,
                                   const BatchView* hviews, const void* views_dev, hdof_gbuffer_bufs out,
                                   float4* pack, float* tile_r, hipStream_t st) {
  GbBatch gbb;
  gbb.n = n_views;
  gbb.blk_base[0] = 0;
  for (int v = 0; v < n_views; ++v)
    gbb.blk_base[v + 1] = gbb.blk_base[v] + cdiv(hviews[v].k.W, 16) * cdiv(hviews[v].k.H, 16);
  for (int v = n_views + 1; v <= HDOF_MAX_VIEWS; ++v) gbb.blk_base[v] = gbb.blk_base[n_views];
  hipLaunchKernelGGL(k_gbuffer_batch, dim3(gbb.blk_base[n_views]), dim3(256), 0, st, sc->nodes, sc->tris,
                     sc->n_nodes, sc->albedo, li, (const ViewK*)views_dev, gbb, out.depth, out.normal, out.albedo,
                     out.color, out.tri_id, ctx->d_flags, pack, tile_r);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

hdof_status reserve_trace(hdof_ctx* ctx, size_t cap, bool own_depth) {
  hdof_status s;
  if ((s = hdof_ensure(ctx->queue, sizeof(int) * cap)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->ray_col, sizeof(float) * 3 * cap)) != HDOF_OK) return s;
  if (own_depth && (s = hdof_ensure(ctx->ray_z, sizeof(float) * cap)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->work_counter, sizeof(int) * 8 * HDOF_SEG_STRIDE)) != HDOF_OK) return s;
  return HDOF_OK;
}

hdof_status launch_trace(hdof_ctx* ctx, const hdof_scene* sc, const CamK& k, const LensK& l,
                         const LightK& li, int spp_max, const uint8_t* spp, const int32_t* offsets,
                         const int32_t* total, uint32_t seed, uint32_t frame, uint32_t view,
                         hdof_rt_bufs out, int32_t* ray_id, float* ray_depth, float* far_pos, hipStream_t st,
                         const VarFuse* vf, bool queue_ready, float* coc_nf) {
  const int N = k.W * k.H;
  const size_t cap = (size_t)N * (size_t)spp_max;
  hdof_status s;
  if ((s = reserve_trace(ctx, cap, !ray_depth)) != HDOF_OK) return s;
  float* rz = ray_depth ? ray_depth : (float*)ctx->ray_z.p;
  if (!queue_ready)
    hipLaunchKernelGGL(k_queue_fill, dim3(cdiv(N, 256)), dim3(256), 0, st, spp, offsets, N, (const int*)nullptr,
                       0, (long)cap, (int*)ctx->queue.p, (int*)ctx->work_counter.p);
  hdof_prof_mark(ctx, 3, st);
  TraceArgs A = base_args(ctx, sc, li, cap);
  A.offsets = offsets;
  A.total_p = total;
  A.ray_z = rz;
  A.ray_id = ray_id;
  A.v0 = ViewK{k, l, seed, frame, view, 0};
  launch_trace_kernel<false>(ctx, A, st);
  hdof_prof_mark(ctx, 4, st);
  const VarFuse vz = vf ? *vf : VarFuse{};
  const bool rays = l.sa != 0.0f;
  auto kern = far_pos ? (vf ? k_rt_reduce<true, true, true> : k_rt_reduce<true, false, true>)
              : rays  ? (vf ? k_rt_reduce<false, true, true> : k_rt_reduce<false, false, true>)
                      : (vf ? k_rt_reduce<false, true, false> : k_rt_reduce<false, false, false>);
  const RtIn R{(const float*)ctx->ray_col.p, rz, cap, l, k, seed, frame, view};
  hipLaunchKernelGGL(kern, dim3(cdiv(N, 256)), dim3(256), 0, st, R, spp, offsets, N, (const int*)nullptr, out.c_near,
                     out.c_far, out.hit_ratio, out.lum_m1, out.lum_m2, far_pos, vz, coc_nf);
  if (!vf) hdof_prof_mark(ctx, 5, st);  // fused: the variance update stage is part of this one
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

// Batched trace: the views' masks have written per-view counts, view-local
// offsets and totals[v]; one scan gives each view's first queue entry, each
// view fills its part of the queue, ONE persistent launch traces all views,
// then each view reduces its own pixels.  `views` is the device copy of
// `hviews` (same order).
hdof_status launch_trace_batched(hdof_ctx* ctx, const hdof_scene* sc, const LightK& li, int spp_max,
                                 int n_views, const BatchView* hviews, const void* views_dev,
                                 const uint8_t* spp, const int32_t* offsets, const int32_t* totals,
                                 int32_t* ebase, int32_t* grand, hdof_rt_bufs* rt, hipStream_t st) {
  long npx = 0;
  for (int v = 0; v < n_views; ++v) npx += (long)hviews[v].k.W * hviews[v].k.H;
  const size_t cap = (size_t)npx * (size_t)spp_max;
  hdof_status s;
  if ((s = reserve_trace(ctx, cap, true)) != HDOF_OK) return s;
  PxBatch pxb{};
  pxb.n = n_views;
  for (int v = 0; v < n_views; ++v)
    pxb.blk_base[v + 1] = pxb.blk_base[v] + cdiv(hviews[v].k.W * hviews[v].k.H, HDOF_BATCH_PX_BLOCK);
  hipLaunchKernelGGL(k_view_scan, dim3(1), dim3(64), 0, st, totals, n_views, ebase, grand);
  hipLaunchKernelGGL(k_queue_fill_batch, dim3(pxb.blk_base[n_views]), dim3(256), 0, st, spp, offsets,
                     (const ViewK*)views_dev, pxb, (const int*)ebase, (long)cap, (int*)ctx->queue.p,
                     (int*)ctx->work_counter.p);
  TraceArgs A = base_args(ctx, sc, li, cap);
  A.offsets = offsets;
  A.total_p = grand;
  A.ray_z = (float*)ctx->ray_z.p;
  A.ray_id = nullptr;
  A.views = (const ViewK*)views_dev;
  A.entry_base = ebase;
  A.n_views = n_views;
  A.v0 = ViewK{hviews[0].k, hviews[0].l, 0, 0, 0, 0};
  launch_trace_kernel<true>(ctx, A, st);
  hipLaunchKernelGGL(k_rt_reduce_batch, dim3(pxb.blk_base[n_views]), dim3(256), 0, st, spp, offsets,
                     (const ViewK*)views_dev, pxb, (const int*)ebase, (const float*)ctx->ray_col.p,
                     (const float*)ctx->ray_z.p, cap, rt->c_near, rt->c_far, rt->hit_ratio, rt->lum_m1,
                     rt->lum_m2);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

size_t batch_view_bytes() { return sizeof(ViewK); }

void batch_view_pack(const BatchView* hv, int n, void* out) {
  ViewK* o = (ViewK*)out;
  for (int v = 0; v < n; ++v) o[v] = ViewK{hv[v].k, hv[v].l, hv[v].seed, hv[v].frame, hv[v].view, hv[v].px_base};
}
