// bvh.hip -- BVH build on the GPU (per scene, outside the frame).
//
// The paper traces through the driver's hardware BVH; CDNA4 has no ray
// tracing units, so the acceleration structure is built here:
//   centroid bounds -> 63-bit Morton codes -> LSD radix sort (8 x 8 bits)
//   -> PLOC clustering (Meister & Bittner, TVCG 2018): each cluster finds
//      its nearest neighbour by merged-box surface area within a window of
//      the Morton order, mutual pairs merge, clusters are compacted, until
//      one remains (a surface-area-aware tree rather than a pure Morton
//      split, which large triangles such as room walls would inflate)
//   -> depth-first numbering from subtree sizes; subtrees of at most
//      HDOF_BVH_LEAF triangles become leaves whose triangles are contiguous
//   -> traversal layout: per internal node the boxes of both children in
//      full (64 B, the wave-coherent walk) and in half precision about their
//      centre (48 B, the per-lane walk), triangles as 3 float4 in leaf order.
#include <cmath>
#include <utility>

#include "hdof_internal.h"
#include "ploc.h"

#define RS_THREADS 256
#define RS_ITEMS 4
#define RS_TILE (RS_THREADS * RS_ITEMS)
#define HDOF_BVH_LEAF 4
#define PLOC_R 16

namespace {

#define BOUNDS_BLOCKS 1024  // partial bounds at most

// the block's minima (6 values: minimum, -maximum) of `v`, in every thread
__device__ inline void block_min6(float v[6], float (*red)[RS_THREADS / 64]) {
  for (int a = 0; a < 6; ++a) {
    for (int o = 32; o > 0; o >>= 1) v[a] = fminf(v[a], __shfl_xor(v[a], o));
    if ((threadIdx.x & 63) == 0) red[a][threadIdx.x >> 6] = v[a];
  }
  __syncthreads();
  for (int a = 0; a < 6; ++a) v[a] = fminf(fminf(red[a][0], red[a][1]), fminf(red[a][2], red[a][3]));
}

// Per block: the centroids' bounds, and of its triangles of finite extent the
// number and the sum of the exponents of their largest extents.
__global__ __launch_bounds__(RS_THREADS) void k_centroid_bounds(const float* __restrict__ v, int n,
                                                                float* __restrict__ part, int2* __restrict__ sizes) {
  __shared__ float red[6][RS_THREADS / 64];
  __shared__ int2 size_red[RS_THREADS / 64];
  int2 sz = make_int2(0, 0);
  float m[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
  for (int i = blockIdx.x * RS_THREADS + threadIdx.x; i < n; i += gridDim.x * RS_THREADS) {
    const float* t = v + 9 * (size_t)i;
    float ext = 0.0f;
    for (int a = 0; a < 3; ++a) {
      float c = (t[a] + t[3 + a] + t[6 + a]) * (1.0f / 3.0f);
      m[a] = fminf(m[a], c);
      m[3 + a] = fminf(m[3 + a], -c);
      ext = fmaxf(ext, fmaxf(fmaxf(t[a], t[3 + a]), t[6 + a]) - fminf(fminf(t[a], t[3 + a]), t[6 + a]));
    }
    if (ext > 0.0f && ext < INFINITY) {
      int e;
      frexpf(ext, &e);
      sz.x += 1, sz.y += e;
    }
  }
  for (int o = 32; o > 0; o >>= 1) sz.x += __shfl_xor(sz.x, o), sz.y += __shfl_xor(sz.y, o);
  if ((threadIdx.x & 63) == 0) size_red[threadIdx.x >> 6] = sz;
  block_min6(m, red);
  if (threadIdx.x < 6) part[6 * blockIdx.x + threadIdx.x] = m[threadIdx.x];
  if (threadIdx.x == 0) {
    for (int w = 1; w < RS_THREADS / 64; ++w) sz.x += size_red[w].x, sz.y += size_red[w].y;
    sizes[blockIdx.x] = sz;
  }
}

__device__ inline uint64_t spread21(uint64_t x) {
  x &= 0x1FFFFF;
  x = (x | (x << 32)) & 0x1F00000000FFFFull;
  x = (x | (x << 16)) & 0x1F0000FF0000FFull;
  x = (x | (x << 8)) & 0x100F00F00F00F00Full;
  x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

// Morton codes of the centroids in the bounds that the partial ones reduce
// to; the albedo's copy and the mean exponent of the triangles' extents too
__global__ __launch_bounds__(RS_THREADS) void k_morton(const float* __restrict__ v, int n,
                                                       const float* __restrict__ part,
                                                       const int2* __restrict__ sizes, int nparts,
                                                       const float* __restrict__ albedo, uint64_t* __restrict__ keys,
                                                       int* __restrict__ vals, float* __restrict__ alb_out,
                                                       int* __restrict__ mean) {
  __shared__ float red[6][RS_THREADS / 64];
  float m[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
  for (int k = threadIdx.x; k < nparts; k += RS_THREADS)
    for (int a = 0; a < 6; ++a) m[a] = fminf(m[a], part[6 * k + a]);
  block_min6(m, red);
  const int i0 = blockIdx.x * RS_THREADS, i = i0 + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    long count = 0, sum = 0;
    for (int k = threadIdx.x; k < nparts; k += 64) count += sizes[k].x, sum += sizes[k].y;
    for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o), sum += __shfl_xor(sum, o);
    if (threadIdx.x == 0) *mean = count > 0 ? (int)floorf((float)sum / (float)count) : 1000;
  }
  for (int k = 0; k < 3; ++k) {
    const size_t j = 3 * (size_t)i0 + k * RS_THREADS + threadIdx.x;
    if (j < 3 * (size_t)n) alb_out[j] = albedo[j];
  }
  if (i >= n) return;
  const float* t = v + 9 * (size_t)i;
  uint64_t q[3];
  for (int a = 0; a < 3; ++a) {
    float c = (t[a] + t[3 + a] + t[6 + a]) * (1.0f / 3.0f);
    float ext = -m[3 + a] - m[a];
    float u = ext > 0.0f ? (c - m[a]) / ext : 0.5f;
    u = fminf(fmaxf(u, 0.0f), 1.0f);
    q[a] = (uint64_t)fminf(u * 2097152.0f, 2097151.0f);
  }
  keys[i] = (spread21(q[0]) << 2) | (spread21(q[1]) << 1) | spread21(q[2]);
  vals[i] = i;
}

// ---- LSD radix sort: histogram, scan, stable scatter ----------------------
__global__ void k_rs_hist(const uint64_t* __restrict__ keys, int n, int shift, int nblocks,
                          int* __restrict__ hist) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  int base = blockIdx.x * RS_TILE;
  for (int k = 0; k < RS_ITEMS; ++k) {
    int i = base + k * RS_THREADS + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255], 1);
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// inclusive scan of one value per thread of a block of four waves
__device__ inline int block_scan(int v, int* part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  if (lane == 63) part[wave] = v;
  __syncthreads();
  for (int w = 0; w < wave; ++w) v += part[w];
  return v;
}

// each digit's counts over the blocks, one digit per block: exclusive scan
// in place and the digit's total (a single block over all digits' counts
// took 35 us a pass for 200k keys)
__global__ __launch_bounds__(RS_THREADS) void k_rs_rows(int* __restrict__ hist, int nblocks, int* __restrict__ tot) {
  __shared__ int part[RS_THREADS / 64];
  int* row = hist + (size_t)blockIdx.x * nblocks;
  int run = 0;
  for (int i0 = 0; i0 < nblocks; i0 += RS_THREADS) {
    const int i = i0 + threadIdx.x;
    const int c = i < nblocks ? row[i] : 0;
    const int incl = block_scan(c, part);
    if (i < nblocks) row[i] = run + incl - c;
    run += part[0] + part[1] + part[2] + part[3];
    __syncthreads();
  }
  if (threadIdx.x == 0) tot[blockIdx.x] = run;
}

__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(const uint64_t* __restrict__ kin,
                                                           const int* __restrict__ vin, int n,
                                                           int shift, int nblocks,
                                                           const int* __restrict__ hist, const int* __restrict__ tot,
                                                           uint64_t* __restrict__ kout,
                                                           int* __restrict__ vout) {
  __shared__ int gbase[256];
  __shared__ int running[256];
  __shared__ int wcount[RS_THREADS / 64][256];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  __shared__ int part[RS_THREADS / 64];
  gbase[t] = hist[(size_t)t * nblocks + blockIdx.x] + block_scan(tot[t], part) - tot[t];
  running[t] = 0;
  for (int w = 0; w < RS_THREADS / 64; ++w) wcount[w][t] = 0;
  __syncthreads();
  int base = blockIdx.x * RS_TILE;
  for (int k = 0; k < RS_ITEMS; ++k) {
    int i = base + k * RS_THREADS + t;
    bool valid = i < n;
    uint64_t key = valid ? kin[i] : 0;
    int val = valid ? vin[i] : 0;
    int d = valid ? (int)((key >> shift) & 255) : 256;
    // lanes of this wave holding the same digit
    uint64_t same = __ballot(valid);
    for (int b = 0; b < 8; ++b) {
      uint64_t bits = __ballot(valid && ((d >> b) & 1));
      same &= ((d >> b) & 1) ? bits : ~bits;
    }
    if (!valid) same = 0;
    uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int rank = __popcll(same & lt);
    int leader = valid && rank == 0;
    if (leader) wcount[wave][d] = __popcll(same);
    __syncthreads();
    if (valid) {
      int off = running[d] + rank;
      for (int w = 0; w < wave; ++w) off += wcount[w][d];
      int dst = gbase[d] + off;
      kout[dst] = key;
      vout[dst] = val;
    }
    __syncthreads();
    int add = 0;
    for (int w = 0; w < RS_THREADS / 64; ++w) {
      add += wcount[w][t];
      wcount[w][t] = 0;
    }
    running[t] += add;
    __syncthreads();
  }
}

// ---- PLOC clustering -----------------------------------------------------------
// cluster codes: >= 0 internal node (build numbering), < 0 ~leaf (Morton position)
__device__ inline float half_area(float4 lo, float4 hi) {
  float dx = hi.x - lo.x, dy = hi.y - lo.y, dz = hi.z - lo.z;
  return dx * dy + dy * dz + dz * dx;
}

// leaf boxes in Morton order, one cluster each
__global__ void k_leaf_clusters(const float* __restrict__ v, const int* __restrict__ order, int n,
                                float* __restrict__ lbox, int* __restrict__ cid, float4* __restrict__ cbox,
                                int2* __restrict__ csz, int2* __restrict__ state) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) state[0] = make_int2(n, n - 2);  // clusters, next internal node
  if (i >= n) return;
  const float* p = v + 9 * (size_t)order[i];
  float b[6];
  for (int a = 0; a < 3; ++a) {
    b[a] = fminf(p[a], fminf(p[3 + a], p[6 + a]));
    b[3 + a] = fmaxf(p[a], fmaxf(p[3 + a], p[6 + a]));
  }
  for (int a = 0; a < 6; ++a) lbox[6 * (size_t)i + a] = b[a];
  cid[i] = ~i;
  cbox[2 * (size_t)i] = make_float4(b[0], b[1], b[2], 0.0f);
  cbox[2 * (size_t)i + 1] = make_float4(b[3], b[4], b[5], 0.0f);
  csz[i] = make_int2(1, 0);  // (triangles, kept internal nodes) of the subtree
}

// the half area of the union of two boxes
__device__ inline float merged_area(float4 lo, float4 hi, float4 l2, float4 h2) {
  return half_area(make_float4(fminf(lo.x, l2.x), fminf(lo.y, l2.y), fminf(lo.z, l2.z), 0.f),
                   make_float4(fmaxf(hi.x, h2.x), fmaxf(hi.y, h2.y), fmaxf(hi.z, h2.z), 0.f));
}

// One clustering round over the state's m clusters, first half: each
// cluster's nearest neighbour within +-PLOC_R positions by merged-box area
// (ties go to the lower index: j runs upwards with a strict comparison), and
// whether the choice is mutual.  A block also finds its neighbours' choices
// within the window, so no other block's result is needed.  mate[i]: the
// mutual neighbour, else -1; count[block]: clusters that survive the round,
// and merges (upper half).  m is read on the device, so the host enqueues
// rounds without waiting for their outcome: with a copy and a wait per round
// and single-block scans the 67 rounds of 200k triangles took 4 ms.
// (five waves, the window's 288 clusters in one pass; the neighbours' areas
// of a group are formed before any is compared, so their LDS reads overlap)
#define PLOC_FIND_THREADS 320
__global__ __launch_bounds__(PLOC_FIND_THREADS) void k_ploc_find(const float4* __restrict__ cbox, const int2* __restrict__ state,
                                                   int* __restrict__ mate, unsigned long long* __restrict__ count) {
  __shared__ float4 blo[256 + 4 * PLOC_R], bhi[256 + 4 * PLOC_R];
  __shared__ int nn[256 + 2 * PLOC_R];
  __shared__ int cs[4], cl[4];
  const int m = state->x;
  const int first = blockIdx.x * 256;
  if (m <= 1 || first >= m) return;
  const int base = first - 2 * PLOC_R, t = threadIdx.x;
  {
    static_assert(256 + 4 * PLOC_R <= PLOC_FIND_THREADS, "one thread per staged cluster");
    const int g = base + t;
    if (t < 256 + 4 * PLOC_R && g >= 0 && g < m) {
      blo[t] = cbox[2 * (size_t)g];
      bhi[t] = cbox[2 * (size_t)g + 1];
    }
  }
  __syncthreads();
  if (t < 256 + 2 * PLOC_R) {
    const int i = first - PLOC_R + t, li = t + PLOC_R;
    int bj = -1;
    if (i >= 0 && i < m) {
      const float4 lo = blo[li], hi = bhi[li];
      float best = INFINITY;
      for (int d0 = -PLOC_R; d0 <= PLOC_R; d0 += 11) {
        float a[11];
#pragma unroll
        for (int k = 0; k < 11; ++k) a[k] = merged_area(lo, hi, blo[li + d0 + k], bhi[li + d0 + k]);
#pragma unroll
        for (int k = 0; k < 11; ++k) {
          const int j = i + d0 + k;
          if (d0 + k != 0 && j >= 0 && j < m && a[k] < best) {
            best = a[k];
            bj = j;
          }
        }
      }
    }
    nn[t] = bj;
  }
  __syncthreads();
  const int i = first + t;
  int j = -1;
  if (t < 256 && i < m) {
    j = nn[t + PLOC_R];
    if (j >= 0 && nn[j - first + PLOC_R] != i) j = -1;
    mate[i] = j;
  }
  const unsigned long long sv = __ballot(t < 256 && i < m && !(j >= 0 && i > j)), ld = __ballot(t < 256 && i < m && j > i);
  if ((t & 63) == 0 && t < 256) {
    cs[t >> 6] = __popcll(sv);
    cl[t >> 6] = __popcll(ld);
  }
  __syncthreads();
  if (t == 0)
    count[blockIdx.x] = (unsigned long long)(unsigned)(cs[0] + cs[1] + cs[2] + cs[3]) |
                        (unsigned long long)(unsigned)(cl[0] + cl[1] + cl[2] + cl[3]) << 32;
}

// exclusive scan of the blocks' counts in place by one block (scenes of many
// blocks: there the merging blocks' own sums would be quadratic)
__global__ __launch_bounds__(1024) void k_ploc_scan(unsigned long long* __restrict__ a,
                                                    const int2* __restrict__ state) {
  __shared__ unsigned long long part[1024];
  const int m = (state->x + 255) / 256;
  const int t = threadIdx.x, chunk = (m + 1023) / 1024;
  const int lo = min(m, t * chunk), hi = min(m, lo + chunk);
  unsigned long long s = 0;
  for (int i = lo; i < hi; ++i) s += a[i];
  part[t] = s;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    unsigned long long v = t >= off ? part[t - off] : 0ull;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  unsigned long long run = part[t] - s;
  for (int i = lo; i < hi; ++i) {
    unsigned long long x = a[i];
    a[i] = run;
    run += x;
  }
}

// what a merge writes about its node; returns the subtree's size
__device__ inline int2 ploc_node(int node, int c1, int c2, float4 lo, float4 hi, int2 s1, int2 s2,
                                 int* __restrict__ bl, int* __restrict__ br, float* __restrict__ bbox,
                                 int2* __restrict__ bsz) {
  const int cnt = s1.x + s2.x;
  const int2 sz = make_int2(cnt, s1.y + s2.y + (cnt > HDOF_BVH_LEAF ? 1 : 0));
  bl[node] = c1;
  br[node] = c2;
  float* bb = bbox + 6 * (size_t)node;
  bb[0] = lo.x;
  bb[1] = lo.y;
  bb[2] = lo.z;
  bb[3] = hi.x;
  bb[4] = hi.y;
  bb[5] = hi.z;
  bsz[node] = sz;
  return sz;
}

// Second half: mutual pairs merge into the lower one's place, the survivors
// are compacted.  Merged clusters take internal node indices counting down
// from `next`, so the last merge (the root) gets index 0.  The block of the
// last cluster writes the next round's state.
__global__ __launch_bounds__(256) void k_ploc_merge(const int* __restrict__ mate,
                                                    const unsigned long long* __restrict__ count, int scanned,
                                                    const int2* __restrict__ state, int2* __restrict__ state_out,
                                                    const int* __restrict__ cid, const float4* __restrict__ cbox,
                                                    const int2* __restrict__ csz, int* __restrict__ oid,
                                                    float4* __restrict__ obox, int2* __restrict__ osz,
                                                    int* __restrict__ bl, int* __restrict__ br,
                                                    float* __restrict__ bbox, int2* __restrict__ bsz) {
  __shared__ int2 red[4], wave_n[4];
  const int m = state->x, next = state->y;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, blk = blockIdx.x;
  const int nblk = (m + 255) / 256;
  if (m <= 1) {
    if (blk == 0 && t == 0) *state_out = make_int2(m, next);
    return;
  }
  if (blk >= nblk) return;
  int2 before = make_int2(0, 0);
  if (scanned) {
    before = make_int2((int)(count[blk] & 0xffffffffull), (int)(count[blk] >> 32));
  } else {
    for (int b = t; b < blk; b += 256) {
      const unsigned long long c = count[b];
      before.x += (int)(c & 0xffffffffull);
      before.y += (int)(c >> 32);
    }
    for (int o = 32; o > 0; o >>= 1) {
      before.x += __shfl_xor(before.x, o);
      before.y += __shfl_xor(before.y, o);
    }
    if (lane == 0) red[wave] = before;
  }
  const int i = blk * 256 + t;
  const int j = i < m ? mate[i] : -1;
  const bool lead = i < m && j > i, keep = i < m && !(j >= 0 && i > j);
  const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const unsigned long long km = __ballot(keep), lm = __ballot(lead);
  if (lane == 0) wave_n[wave] = make_int2(__popcll(km), __popcll(lm));
  __syncthreads();
  if (!scanned)
    before = make_int2(red[0].x + red[1].x + red[2].x + red[3].x, red[0].y + red[1].y + red[2].y + red[3].y);
  if (blk == nblk - 1 && t == 0)
    *state_out = make_int2(before.x + wave_n[0].x + wave_n[1].x + wave_n[2].x + wave_n[3].x,
                           next - (before.y + wave_n[0].y + wave_n[1].y + wave_n[2].y + wave_n[3].y));
  for (int w = 0; w < wave; ++w) {
    before.x += wave_n[w].x;
    before.y += wave_n[w].y;
  }
  if (!keep) return;
  const int pos = before.x + (int)__popcll(km & lt);
  float4 lo = cbox[2 * (size_t)i], hi = cbox[2 * (size_t)i + 1];
  int id = cid[i];
  int2 sz = csz[i];
  if (lead) {
    const int node = next - (before.y + (int)__popcll(lm & lt));
    const float4 l2 = cbox[2 * (size_t)j], h2 = cbox[2 * (size_t)j + 1];
    lo = make_float4(fminf(lo.x, l2.x), fminf(lo.y, l2.y), fminf(lo.z, l2.z), 0.f);
    hi = make_float4(fmaxf(hi.x, h2.x), fmaxf(hi.y, h2.y), fmaxf(hi.z, h2.z), 0.f);
    sz = ploc_node(node, id, cid[j], lo, hi, sz, csz[j], bl, br, bbox, bsz);
    id = node;
  }
  oid[pos] = id;
  obox[2 * (size_t)pos] = lo;
  obox[2 * (size_t)pos + 1] = hi;
  osz[pos] = sz;
}

// a block barrier that orders LDS accesses only: the nodes' stores stay in flight
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The remaining rounds of at most PLOC_TAIL clusters in one block, which
// keeps them in LDS: most rounds of a build have few clusters, and two
// launches each would cost more than their work.  A cluster's search is
// shared by up to eight threads once the clusters leave that many idle; the
// barriers do not wait for the nodes' stores (127 -> 104 us).
// Stops at one cluster, or at a round without a merge; the clusters left by
// its merges are not written back (see ploc_step).
__global__ __launch_bounds__(PLOC_TAIL) void k_ploc_tail(const int* __restrict__ cid, const float4* __restrict__ cbox,
                                                         const int2* __restrict__ csz, int2* __restrict__ state,
                                                         int* __restrict__ bl, int* __restrict__ br,
                                                         float* __restrict__ bbox, int2* __restrict__ bsz) {
  // two buffers of the clusters (a round reads one and writes the other)
  __shared__ float box[2][6][PLOC_TAIL];
  __shared__ int nn[PLOC_TAIL], idb[2][PLOC_TAIL];
  __shared__ int2 szb[2][PLOC_TAIL];
  __shared__ int2 wave_n[PLOC_TAIL / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int m = state->x, next = state->y;
  if (m > PLOC_TAIL) return;
  if (t < m) {
    const float4 lo = cbox[2 * (size_t)t], hi = cbox[2 * (size_t)t + 1];
    box[0][0][t] = lo.x, box[0][1][t] = lo.y, box[0][2][t] = lo.z;
    box[0][3][t] = hi.x, box[0][4][t] = hi.y, box[0][5][t] = hi.z;
    idb[0][t] = cid[t];
    szb[0][t] = csz[t];
  }
  __syncthreads();
  const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int cur = 0; m > 1; cur ^= 1) {
    const float *lox = box[cur][0], *loy = box[cur][1], *loz = box[cur][2];
    const float *hix = box[cur][3], *hiy = box[cur][4], *hiz = box[cur][5];
    const int* ids = idb[cur];
    const int2* szs = szb[cur];
    // nearest neighbours; window position w stands for the neighbour at
    // w - PLOC_R below PLOC_R and w - PLOC_R + 1 above
    const int sh = m <= PLOC_TAIL / 8 ? 3 : (m <= PLOC_TAIL / 4 ? 2 : (m <= PLOC_TAIL / 2 ? 1 : 0));
    {
      const int i = t >> sh, sub = t & ((1 << sh) - 1), per = (2 * PLOC_R) >> sh;
      float best = INFINITY;
      int bj = -1;
      if (i < m) {
        const float4 lo = make_float4(lox[i], loy[i], loz[i], 0.f), hi = make_float4(hix[i], hiy[i], hiz[i], 0.f);
        for (int w = sub * per; w < (sub + 1) * per; ++w) {
          const int j = i + w - PLOC_R + (w >= PLOC_R ? 1 : 0);
          if (j < 0 || j >= m) continue;
          const float a = merged_area(lo, hi, make_float4(lox[j], loy[j], loz[j], 0.f),
                                      make_float4(hix[j], hiy[j], hiz[j], 0.f));
          if (a < best) {
            best = a;
            bj = j;
          }
        }
      }
      for (int o = 1; o < 1 << sh; o <<= 1) {  // ties to the lower index
        const float a = __shfl_xor(best, o);
        const int j = __shfl_xor(bj, o);
        if (j >= 0 && (bj < 0 || a < best || (a == best && j < bj))) {
          best = a;
          bj = j;
        }
      }
      if (i < m && sub == 0) nn[i] = bj;
    }
    lds_barrier();
    int j = -1;
    if (t < m) {
      j = nn[t];
      if (j >= 0 && nn[j] != t) j = -1;
    }
    const bool lead = t < m && j > t, keep = t < m && !(j >= 0 && t > j);
    const unsigned long long km = __ballot(keep), lm = __ballot(lead);
    if (lane == 0) wave_n[wave] = make_int2(__popcll(km), __popcll(lm));
    lds_barrier();
    int2 before = make_int2(0, 0), all = make_int2(0, 0);
    for (int w = 0; w < PLOC_TAIL / 64; ++w) {
      const int2 c = wave_n[w];
      if (w < wave) before.x += c.x, before.y += c.y;
      all.x += c.x, all.y += c.y;
    }
    const int pos = before.x + (int)__popcll(km & lt);
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
    int id = 0;
    int2 sz = make_int2(0, 0);
    if (keep) {
      lo = make_float4(lox[t], loy[t], loz[t], 0.f);
      hi = make_float4(hix[t], hiy[t], hiz[t], 0.f);
      id = ids[t];
      sz = szs[t];
      if (lead) {
        const int node = next - (before.y + (int)__popcll(lm & lt));
        lo = make_float4(fminf(lo.x, lox[j]), fminf(lo.y, loy[j]), fminf(lo.z, loz[j]), 0.f);
        hi = make_float4(fmaxf(hi.x, hix[j]), fmaxf(hi.y, hiy[j]), fmaxf(hi.z, hiz[j]), 0.f);
        sz = ploc_node(node, id, ids[j], lo, hi, sz, szs[j], bl, br, bbox, bsz);
        id = node;
      }
    }
    if (keep) {
      float(*ob)[PLOC_TAIL] = box[cur ^ 1];
      ob[0][pos] = lo.x, ob[1][pos] = lo.y, ob[2][pos] = lo.z;
      ob[3][pos] = hi.x, ob[4][pos] = hi.y, ob[5][pos] = hi.z;
      idb[cur ^ 1][pos] = id;
      szb[cur ^ 1][pos] = sz;
    }
    if (all.y == 0) break;
    m = all.x;
    next -= all.y;
    lds_barrier();
  }
  if (t == 0) *state = make_int2(m, next);
}

// what a step from a node to its parent adds to the placement below: the
// left sibling's triangles, and one node per level plus the left sibling's
// kept ones
__global__ void k_parents(int nint, const int* __restrict__ bl, const int* __restrict__ br,
                          const int2* __restrict__ bsz, int4* __restrict__ up_int, int4* __restrict__ up_leaf) {
  int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= nint) return;
  const int l = bl[a], r = br[a];
  const int2 ls = l < 0 ? make_int2(1, 0) : bsz[l];
  *(l < 0 ? up_leaf + ~l : up_int + l) = make_int4(a, 0, 1, 0);
  *(r < 0 ? up_leaf + ~r : up_int + r) = make_int4(a, ls.x, 1 + ls.y, 0);
  if (a == 0) up_int[0] = make_int4(-1, 0, 0, 0);
}

// depth-first placement by walking to the root, one record per level: the
// first triangle slot of a subtree and a kept internal node's index
__device__ inline void dfs_place(int4 up, int n, const int4* __restrict__ up_int, int& off, int& idx, int& depth) {
  off = 0;
  idx = 0;
  depth = 0;
  for (int guard = 0; up.x >= 0 && guard < n; ++guard) {
    off += up.y;
    idx += up.z;
    ++depth;
    up = up_int[up.x];
  }
}

// Places the kept nodes by their walks to the root; the
// rest takes a step or two from there (walks from every triangle and node:
// 50 us for 200k triangles, bound by their random 16-byte reads).
__global__ void k_place_nodes(int n, int nint, const int4* __restrict__ up_int, const int2* __restrict__ bsz,
                              int* __restrict__ node_off, int* __restrict__ node_idx, int* __restrict__ node_dep) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= nint || (a != 0 && bsz[a].x <= HDOF_BVH_LEAF)) return;
  int off, idx, d;
  dfs_place(up_int[a], n, up_int, off, idx, d);
  node_off[a] = off;
  node_idx[a] = idx;
  node_dep[a] = d;
}

// threads 0..n-1 place the leaves, the others the small internal nodes; a
// wave adds its depth to the tree's only where it is the largest so far (an
// atomic per triangle took 37 us for 200k triangles, one per wave 33)
__global__ void k_place_rest(int n, int nint, const int4* __restrict__ up_int, const int4* __restrict__ up_leaf,
                             const int2* __restrict__ bsz, const int* __restrict__ node_dep,
                             int* __restrict__ leaf_off, int* __restrict__ node_off, int* __restrict__ depth_out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const bool leaf = i < n, small = !leaf && i - n < nint && i != n && bsz[i - n].x <= HDOF_BVH_LEAF;
  int d = 0;
  if (leaf || small) {
    int4 up = leaf ? up_leaf[i] : up_int[i - n];
    int off = up.y;
    for (d = 1; up.x != 0 && bsz[up.x].x <= HDOF_BVH_LEAF; ++d) {  // at most HDOF_BVH_LEAF small ancestors
      up = up_int[up.x];
      off += up.y;
    }
    off += node_off[up.x];
    d += node_dep[up.x];
    if (leaf)
      leaf_off[i] = off;
    else
      node_off[i - n] = off, d = 0;
  }
  for (int o = 32; o > 0; o >>= 1) d = max(d, __shfl_xor(d, o));
  if ((threadIdx.x & 63) == 0 && d + 1 > __hip_atomic_load(depth_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(depth_out, d + 1);
}

__global__ void k_place_tris(const float* __restrict__ v, const int* __restrict__ order,
                             const int* __restrict__ leaf_off, int n, float4* __restrict__ tris) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int t = order[i], o = leaf_off ? leaf_off[i] : i;
  const float* p = v + 9 * (size_t)t;
  tris[3 * (size_t)o + 0] = make_float4(p[0], p[1], p[2], __int_as_float(t));
  tris[3 * (size_t)o + 1] = make_float4(p[3], p[4], p[5], 0.0f);
  tris[3 * (size_t)o + 2] = make_float4(p[6], p[7], p[8], 0.0f);
}

__device__ inline unsigned leaf_code(int first, int count) {
  return HDOF_LEAF_BIT | ((unsigned)(count - 1) << 27) | (unsigned)first;
}

// ---- half-precision nodes -----------------------------------------------------
// The scene's box unit, a power of two.  Box planes relative to their node's
// centre are halves, of 11 bits from 2^-14 to 2^16 units and of fixed steps
// of 2^-24 below.  The root's largest extent is at most 2^14 units, unless
// that would leave triangles of the usual size (the geometric mean of their
// extents, 2^mean) below 2^-10 units, in a scene whose ground or sky is more
// than 2^24 times as wide: then they have that size, and planes beyond 2^16
// units from their node's centre, of the few nodes that hold the far
// geometry, are infinite (every ray passes them).  Node visits and triangle
// tests per ray of a room on a ground of 1e8 / 1e10 / 1e14 units: 59 / 637 /
// 34006 with the root's extent alone, 57 / 48 / 48 so and by fp32 boxes.  At
// most 2^27: a ray's inverse direction, up to 1e30, is multiplied by the unit.
__device__ inline float box_unit(const float* __restrict__ root, int mean) {
  float ext = 0.0f;
  for (int a = 0; a < 3; ++a) ext = fmaxf(ext, root[3 + a] - root[a]);
  int e = 0;
  frexpf(ext, &e);  // ext < 2^e
  e = ext > 0.0f && ext < INFINITY ? e - 14 : 0;
  return ldexpf(1.0f, max(-100, min(27, min(e, mean + 10))));
}

// the box plane d above its node's centre in units, rounded outwards (dir -1 or 1)
__device__ inline unsigned half_plane(float d, float unit, float margin, int dir) {
  const float v = (d + (dir > 0 ? margin : -margin)) / unit;
  _Float16 h = (_Float16)v;
  unsigned short u;
  __builtin_memcpy(&u, &h, 2);
  if (dir > 0 ? (float)h < v : (float)h > v) {  // one step towards dir
    if ((u & 0x7FFF) == 0)
      u = dir > 0 ? 0x0001 : 0x8001;
    else
      u = (unsigned short)(((u & 0x8000) != 0) == (dir < 0) ? u + 1 : u - 1);
  }
  return u;
}

// Half-precision record of a node with child boxes b0, b1 (minimum, maximum):
// (centre, code 1), (x of both children, y of both), (z of both, code 0, -),
// a pair of planes (minimum, maximum) per dword; a node's code is its
// record's position in float4s, three times its index.
// The planes are widened by 2^-21 of the node's own half extent: the
// traversal forms a plane's distance from the centre's and the plane's offset
// from it, whose rounding is relative to those two.  The offset's share the
// margin covers; the centre's share beyond it is relative to the distance
// itself and lies in the walk's comparison (see box_hit_half).  (A margin of
// 2^-21 of the scene's largest coordinate also held, but widened every box
// of a scene far from the origin or with a wide ground: 8.3M rays of a room
// 10^4 / 10^5 units away took 2735 / 100748 us, with a ground of 10^5 units
// 36802.)
__device__ inline void emit_half(float4* __restrict__ o, const float* b0, const float* b1, unsigned c0, unsigned c1,
                                 float s) {
  float c[3];
  unsigned pl[3][2];
  for (int a = 0; a < 3; ++a) {
    const float lo = fminf(b0[a], b1[a]), hi = fmaxf(b0[3 + a], b1[3 + a]);
    c[a] = 0.5f * (lo + hi);
    const float mg = fmaxf(c[a] - lo, hi - c[a]) * 4.76837158e-7f;
    pl[a][0] = half_plane(b0[a] - c[a], s, mg, -1) | half_plane(b0[3 + a] - c[a], s, mg, 1) << 16;
    pl[a][1] = half_plane(b1[a] - c[a], s, mg, -1) | half_plane(b1[3 + a] - c[a], s, mg, 1) << 16;
  }
  o[0] = make_float4(c[0] / s, c[1] / s, c[2] / s, __uint_as_float(c1));
  o[1] = make_float4(__uint_as_float(pl[0][0]), __uint_as_float(pl[0][1]), __uint_as_float(pl[1][0]),
                     __uint_as_float(pl[1][1]));
  o[2] = make_float4(__uint_as_float(pl[2][0]), __uint_as_float(pl[2][1]), __uint_as_float(c0), 0.0f);
}

// kept internal nodes (more than HDOF_BVH_LEAF triangles, or the root) are
// written at their depth-first index; smaller subtrees become leaf ranges
__global__ void k_emit_nodes(int nint, const int* __restrict__ bl, const int* __restrict__ br,
                             const int2* __restrict__ bsz, const float* __restrict__ bbox,
                             const float* __restrict__ lbox, const int* __restrict__ leaf_off,
                             const int* __restrict__ node_off, const int* __restrict__ node_idx,
                             const int* __restrict__ mean, float* __restrict__ unit, float4* __restrict__ nodes,
                             float4* __restrict__ hnodes) {
  int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= nint) return;
  const float u = box_unit(bbox, *mean);  // node 0 is the root
  if (a == 0) *unit = u;
  if (a != 0 && bsz[a].x <= HDOF_BVH_LEAF) return;
  int ch[2] = {bl[a], br[a]};
  float b[2][6];
  unsigned code[2];
  for (int k = 0; k < 2; ++k) {
    int c = ch[k];
    const float* src;
    if (c < 0) {
      src = lbox + 6 * (size_t)(~c);
      code[k] = leaf_code(leaf_off[~c], 1);
    } else {
      src = bbox + 6 * (size_t)c;
      int cnt = bsz[c].x;
      code[k] = cnt <= HDOF_BVH_LEAF ? leaf_code(node_off[c], cnt) : (unsigned)node_idx[c];
    }
    for (int q = 0; q < 6; ++q) b[k][q] = src[q];
  }
  float4* o = nodes + 4 * (size_t)node_idx[a];
  o[0] = make_float4(b[0][0], b[0][3], b[0][1], b[0][4]);
  o[1] = make_float4(b[1][0], b[1][3], b[1][1], b[1][4]);
  o[2] = make_float4(b[0][2], b[0][5], b[1][2], b[1][5]);
  o[3] = make_float4(__uint_as_float(code[0]), __uint_as_float(code[1]), 0.0f, 0.0f);
  for (int k = 0; k < 2; ++k)
    if (!(code[k] & HDOF_LEAF_BIT)) code[k] *= 3u;
  emit_half(hnodes + 3 * (size_t)node_idx[a], b[0], b[1], code[0], code[1], u);
}

// one triangle: a root whose second child box is empty
__global__ void k_single_root(const float* __restrict__ lbox, const int* __restrict__ mean, float* __restrict__ unit,
                              float4* __restrict__ nodes, float4* __restrict__ hnodes) {
  const float u = box_unit(lbox, *mean);
  *unit = u;
  emit_half(hnodes, lbox, lbox, leaf_code(0, 1), leaf_code(0, 1), u);
  float4* o = nodes;
  o[0] = make_float4(lbox[0], lbox[3], lbox[1], lbox[4]);
  o[1] = make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
  o[2] = make_float4(lbox[2], lbox[5], INFINITY, -INFINITY);
  o[3] = make_float4(__uint_as_float(leaf_code(0, 1)), __uint_as_float(leaf_code(0, 1)), 0.0f, 0.0f);
}

__global__ void k_fill_int(int* p, int n, int v) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

}  // namespace

hdof_status launch_bvh_build(hdof_ctx* ctx, const float* verts, const float* albedo, int n,
                             hdof_scene* sc, hipStream_t st) {
  const int nint = n > 1 ? n - 1 : 1;
  const int nb = cdiv(n, RS_TILE);
  const int nbounds = min(BOUNDS_BLOCKS, cdiv(n, RS_THREADS));
  size_t off = 0;
  auto carve = [&](size_t bytes) {
    size_t o = off;
    off += (bytes + 255) & ~(size_t)255;
    return o;
  };
  // permanent storage, one allocation (node slots for every internal node;
  // collapsed subtrees leave the tail unused)
  const size_t p_nodes = carve(sizeof(float4) * 4 * (size_t)nint), p_half = carve(sizeof(float4) * 3 * (size_t)nint);
  const size_t p_tris = carve(sizeof(float4) * 3 * (size_t)n), p_alb = carve(sizeof(float) * 3 * (size_t)n);
  const size_t p_depth = carve(sizeof(int)), p_unit = carve(sizeof(float));
  HDOF_HIP(hipMalloc(&sc->mem, off));
  sc->nodes = (float4*)(sc->mem + p_nodes);
  sc->hnodes = (float4*)(sc->mem + p_half);
  sc->tris = (float4*)(sc->mem + p_tris);
  sc->albedo = (float*)(sc->mem + p_alb);
  sc->depth_out = (int32_t*)(sc->mem + p_depth);
  sc->unit = (float*)(sc->mem + p_unit);
  sc->n_nodes = nint;
  sc->bytes = (int64_t)sizeof(float4) * (7 * (int64_t)nint + 3 * (int64_t)n) + 12 * (int64_t)n;
  // build scratch, one buffer of the context
  off = 0;
  size_t o_bounds = carve(sizeof(float) * 6 * nbounds), o_sizes = carve(sizeof(int2) * nbounds);
  size_t o_mean = carve(sizeof(int));
  size_t o_k0 = carve(sizeof(uint64_t) * n), o_k1 = carve(sizeof(uint64_t) * n);
  size_t o_v0 = carve(sizeof(int) * n), o_v1 = carve(sizeof(int) * n);
  size_t o_hist = carve(sizeof(int) * 256 * (size_t)nb), o_dig = carve(sizeof(int) * 256);
  size_t o_lbox = carve(sizeof(float) * 6 * (size_t)n);
  size_t o_cid0 = carve(sizeof(int) * n), o_cid1 = carve(sizeof(int) * n);
  size_t o_cb0 = carve(sizeof(float4) * 2 * (size_t)n), o_cb1 = carve(sizeof(float4) * 2 * (size_t)n);
  size_t o_cs0 = carve(sizeof(int2) * n), o_cs1 = carve(sizeof(int2) * n);
  size_t o_mate = carve(sizeof(int) * n), o_cnt = carve(sizeof(unsigned long long) * cdiv(n, 256));
  size_t o_state = carve(sizeof(int2) * 2);
  size_t o_bl = carve(sizeof(int) * nint), o_br = carve(sizeof(int) * nint);
  size_t o_bbox = carve(sizeof(float) * 6 * (size_t)nint), o_bsz = carve(sizeof(int2) * nint);
  size_t o_pint = carve(sizeof(int4) * nint), o_pleaf = carve(sizeof(int4) * n);
  size_t o_loff = carve(sizeof(int) * n), o_noff = carve(sizeof(int) * nint), o_nidx = carve(sizeof(int) * nint);
  size_t o_ndep = carve(sizeof(int) * nint);
  hdof_status status = hdof_ensure(ctx->bvh_scratch, off);
  if (status != HDOF_OK) return status;
  char* s = (char*)ctx->bvh_scratch.p;
  float* bounds = (float*)(s + o_bounds);
  int2* sizes = (int2*)(s + o_sizes);
  int* mean = (int*)(s + o_mean);
  uint64_t* k0 = (uint64_t*)(s + o_k0);
  uint64_t* k1 = (uint64_t*)(s + o_k1);
  int* v0 = (int*)(s + o_v0);
  int* v1 = (int*)(s + o_v1);
  int *hist = (int*)(s + o_hist), *dig = (int*)(s + o_dig);
  float* lbox = (float*)(s + o_lbox);
  int* cid[2] = {(int*)(s + o_cid0), (int*)(s + o_cid1)};
  float4* cbox[2] = {(float4*)(s + o_cb0), (float4*)(s + o_cb1)};
  int2* csz[2] = {(int2*)(s + o_cs0), (int2*)(s + o_cs1)};
  int* mate = (int*)(s + o_mate);
  unsigned long long* cnt = (unsigned long long*)(s + o_cnt);
  int2* state = (int2*)(s + o_state);
  int *bl = (int*)(s + o_bl), *br = (int*)(s + o_br);
  float* bbox = (float*)(s + o_bbox);
  int2* bsz = (int2*)(s + o_bsz);
  int4 *up_int = (int4*)(s + o_pint), *up_leaf = (int4*)(s + o_pleaf);
  int *loff = (int*)(s + o_loff), *noff = (int*)(s + o_noff), *nidx = (int*)(s + o_nidx);
  int* ndep = (int*)(s + o_ndep);

  hipLaunchKernelGGL(k_centroid_bounds, dim3(nbounds), dim3(RS_THREADS), 0, st, verts, n, bounds, sizes);
  hipLaunchKernelGGL(k_morton, dim3(cdiv(n, RS_THREADS)), dim3(RS_THREADS), 0, st, verts, n, (const float*)bounds,
                     (const int2*)sizes, nbounds, albedo, k0, v0, sc->albedo, mean);
  for (int pass = 0; pass < 8; ++pass) {
    int shift = 8 * pass;
    hipLaunchKernelGGL(k_rs_hist, dim3(nb), dim3(RS_THREADS), 0, st, k0, n, shift, nb, hist);
    hipLaunchKernelGGL(k_rs_rows, dim3(256), dim3(RS_THREADS), 0, st, hist, nb, dig);
    hipLaunchKernelGGL(k_rs_scatter, dim3(nb), dim3(RS_THREADS), 0, st, k0, v0, n, shift, nb, (const int*)hist,
                       (const int*)dig, k1, v1);
    std::swap(k0, k1);
    std::swap(v0, v1);
  }
  hipLaunchKernelGGL(k_leaf_clusters, dim3(cdiv(n, 256)), dim3(256), 0, st, verts, (const int*)v0, n, lbox, cid[0],
                     cbox[0], csz[0], state);
  hipLaunchKernelGGL(k_fill_int, dim3(1), dim3(64), 0, st, sc->depth_out, 1, n == 1 ? 2 : 1);
  if (n == 1) {
    hipLaunchKernelGGL(k_place_tris, dim3(1), dim3(64), 0, st, verts, (const int*)v0, (const int*)nullptr, n, sc->tris);
    hipLaunchKernelGGL(k_single_root, dim3(1), dim3(1), 0, st, (const float*)lbox, (const int*)mean,
                       sc->unit, sc->nodes, sc->hnodes);
  } else {
    // rounds over grids sized by the last count the host has read, as many
    // at a time as should leave PLOC_TAIL clusters (a round leaves between
    // 0.75 and 0.83 of them on the scenes measured); one block does the rest.
    // A round too many costs 9 us, one too few a wait of the host: counting
    // with 1 / 1.25 a round, 200k triangles built in 700 us and 600k in 1140,
    // with 1 / 1.2 in 660 and 1050
    int m = n, cur = 0;
    while (m > 1) {
      const int nblk = cdiv(m, 256), m0 = m;
      if (m > PLOC_TAIL) {
        const int scanned = nblk > 8192;
        const int rounds = (int)ceil(log((double)m / PLOC_TAIL) / log(1.2));
        for (int r = 0; r < rounds; ++r) {
          hipLaunchKernelGGL(k_ploc_find, dim3(nblk), dim3(PLOC_FIND_THREADS), 0, st, (const float4*)cbox[cur],
                             (const int2*)(state + cur), mate, cnt);
          if (scanned) hipLaunchKernelGGL(k_ploc_scan, dim3(1), dim3(1024), 0, st, cnt, (const int2*)(state + cur));
          hipLaunchKernelGGL(k_ploc_merge, dim3(nblk), dim3(256), 0, st, (const int*)mate,
                             (const unsigned long long*)cnt, scanned, (const int2*)(state + cur), state + (cur ^ 1),
                             (const int*)cid[cur], (const float4*)cbox[cur], (const int2*)csz[cur], cid[cur ^ 1],
                             cbox[cur ^ 1], csz[cur ^ 1], bl, br, bbox, bsz);
          cur ^= 1;
        }
      }
      // (returns at once when more clusters are left than it takes)
      hipLaunchKernelGGL(k_ploc_tail, dim3(1), dim3(PLOC_TAIL), 0, st, (const int*)cid[cur],
                         (const float4*)cbox[cur], (const int2*)csz[cur], state + cur, bl, br, bbox, bsz);
      int2 h = make_int2(0, 0);
      hipError_t e = hipMemcpyAsync(&h, state + cur, sizeof h, hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);
      if (e != hipSuccess) {
        status = hdof_set_error(HDOF_ERR_HIP, "BVH clustering: %s", hipGetErrorString(e));
        break;
      }
      m = h.x;
      if (ploc_step(m0, m, h.y) == PLOC_STALLED) {
        status = hdof_set_error(HDOF_ERR_HIP, "BVH clustering made no progress (%d clusters)", m);
        break;
      }
    }
    if (status == HDOF_OK) {
      hipLaunchKernelGGL(k_parents, dim3(cdiv(nint, 256)), dim3(256), 0, st, nint, (const int*)bl, (const int*)br,
                         (const int2*)bsz, up_int, up_leaf);
      hipLaunchKernelGGL(k_place_nodes, dim3(cdiv(nint, 256)), dim3(256), 0, st, n, nint, (const int4*)up_int,
                         (const int2*)bsz, noff, nidx, ndep);
      hipLaunchKernelGGL(k_place_rest, dim3(cdiv((long)n + nint, 256)), dim3(256), 0, st, n, nint,
                         (const int4*)up_int, (const int4*)up_leaf, (const int2*)bsz, (const int*)ndep, loff, noff,
                         sc->depth_out);
      hipLaunchKernelGGL(k_place_tris, dim3(cdiv(n, 256)), dim3(256), 0, st, verts, (const int*)v0,
                         (const int*)loff, n, sc->tris);
      hipLaunchKernelGGL(k_emit_nodes, dim3(cdiv(nint, 256)), dim3(256), 0, st, nint, (const int*)bl,
                         (const int*)br, (const int2*)bsz, (const float*)bbox, (const float*)lbox,
                         (const int*)loff, (const int*)noff, (const int*)nidx, (const int*)mean, sc->unit, sc->nodes,
                         sc->hnodes);
    }
  }
  hipError_t e = hipGetLastError();
  if (status == HDOF_OK && e != hipSuccess)
    status = hdof_set_error(HDOF_ERR_HIP, "BVH build launch: %s", hipGetErrorString(e));
  // the scene may be used on any stream from here on, the scratch by the
  // context's next build
  e = hipStreamSynchronize(st);
  if (status == HDOF_OK && e != hipSuccess) status = hdof_set_error(HDOF_ERR_HIP, "BVH build: %s", hipGetErrorString(e));
  if (ctx->bvh_scratch.bytes > HDOF_BVH_KEEP_BYTES) {  // a large scene's scratch is not kept for the next
    hipFree(ctx->bvh_scratch.p);
    ctx->bvh_scratch = Buf{};
  }
  return status;
}
