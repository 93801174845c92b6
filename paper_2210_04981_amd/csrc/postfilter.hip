// postfilter.hip -- post-process gather DoF filter and the composite.
//
// k_pp_pack: colour + signed CoC packed into one float4 per pixel (one
//   16-byte load per bilinear texel in the gather) and the per-tile maximum
//   CoC radius.
// k_pp_dilate: gather radius per tile = min(r_cap, max radius over the tiles
//   within ceil(r_cap / tile) tiles).
// k_pp_gather16q / k_pp_gather16 / k_pp_gather_any: golden-angle taps,
//   bilinear float4 texels, weights recomputed per tap, nothing stored but
//   the result.  16-pixel tiles stage each tap's footprint in LDS: one wave
//   per tile gathering 2x2 pixel quads (k_pp_gather16q), or, beside the
//   trace in the overlapped frame, four waves per tile (k_pp_gather16).
// k_composite: focus zone / near / far rules, one pass over the pixels.
#include "hdof_internal.h"

#include <hip/hip_ext.h>

#include <mutex>

namespace {

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__global__ __launch_bounds__(256) void k_pp_pack(const float* __restrict__ color,
                                                 const float* __restrict__ depth, CamK k, LensK l,
                                                 int tile, float4* __restrict__ pack,
                                                 float* __restrict__ tile_r) {
  __shared__ float red[256];
  const int tid = threadIdx.x;
  const int BX = (k.W + 15) >> 4, lb = xcd_block(blockIdx.x, BX * ((k.H + 15) >> 4));
  const int x = (lb % BX) * 16 + (tid & 15), y = (lb / BX) * 16 + (tid >> 4);
  const size_t N = (size_t)k.W * k.H;
  float r = 0.0f;
  if (x < k.W && y < k.H) {
    size_t p = (size_t)y * k.W + x;
    float c = coc_px(l, depth[p]);
    pack[p] = make_float4(color[p], color[N + p], color[2 * N + p], c);
    r = 0.5f * fabsf(c);
  }
  red[tid] = r;
  __syncthreads();
  const int tx = tid & 15, ty = tid >> 4;
  if ((tx % tile) == 0 && (ty % tile) == 0 && x < k.W && y < k.H) {
    float m = 0.0f;
    for (int dy = 0; dy < tile; ++dy)
      for (int dx = 0; dx < tile; ++dx) m = fmaxf(m, red[(ty + dy) * 16 + tx + dx]);
    const int TW = (k.W + tile - 1) / tile;
    tile_r[(y / tile) * TW + x / tile] = m;
  }
}

// golden-angle taps u_k = sqrt((k - 0.5)/n) (cos k g, sin k g), g = pi (3 - sqrt 5),
// evaluated in double and stored as (ux, uy, |u|, omega).  A polygonal
// aperture (blades >= 3, first vertex at rot radians) moves each tap
// radially onto the polygon, u' = u P(angle), P its boundary radius at
// circumradius 1, keeping |u| (the tap's gauge distance in the polygonal
// CoC); omega = max(0, 1 + sa (2 |u'|^2 - 1)) is the tap's aberration weight.
__global__ void k_pp_taps(int n, int blades, double rot, float sa, float4* __restrict__ taps) {
  int k = threadIdx.x + 1;
  if (k > n) {  // the table's unused entries are zero (gathers read whole groups of taps)
    taps[k - 1] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const double pi = 3.14159265358979323846;
  const double g = pi * (3.0 - sqrt(5.0));
  double rr = sqrt((k - 0.5) / n);
  double sc = 1.0;
  if (blades >= 3) {
    const double sector = 2.0 * pi / blades;
    double a = fmod(k * g - rot, sector);
    if (a < 0.0) a += sector;
    sc = cos(pi / blades) / cos(a - pi / blades);
  }
  const double r2 = rr * sc;
  const double om = fmax(0.0, 1.0 + (double)sa * (2.0 * r2 * r2 - 1.0));
  taps[k - 1] = make_float4((float)(r2 * cos(k * g)), (float)(r2 * sin(k * g)), (float)rr, (float)om);
}

// (re)build the context's tap table when the tap count or the aperture changed
void pp_taps_ensure(hdof_ctx* ctx, int n, const LensK& l, hipStream_t st) {
  const int blades = l.blades >= 3 ? l.blades : 0;
  if (ctx->pp_taps_n == n && ctx->pp_taps_blades == blades && ctx->pp_taps_rot == l.rot_ht &&
      ctx->pp_taps_sa == l.sa)
    return;
  hipLaunchKernelGGL(k_pp_taps, dim3(1), dim3(256), 0, st, n, blades, (double)l.rot_ht * 3.14159265358979323846,
                     l.sa, (float4*)ctx->pp_taps.p);
  ctx->pp_taps_n = n;
  ctx->pp_taps_blades = blades;
  ctx->pp_taps_rot = l.rot_ht;
  ctx->pp_taps_sa = l.sa;
}

// The largest radius within K tiles of each tile, capped; ARG: also the pixel
// that sets it (-1 when capped or zero; the lowest of equal ones).  A block
// makes 32x8 tiles: their neighbourhood in LDS, the maximum along the rows,
// then along the columns, 2 (2 K + 1) reads a tile instead of (2 K + 1)^2
// dependent ones from memory (1280x720, 8-pixel tiles, K = 8: 35 -> 5 us;
// 1080p, 16-pixel tiles with their pixels, K = 4: 15 -> 5; the filter of
// 333x187 pixels with 4-pixel tiles, K = 16: 139 -> 32).  More than
// DIL_K tiles (a cap above 64 pixels on 4-pixel tiles) are read one by one.
#define DIL_K 16
#define DIL_W 32
#define DIL_H 8
template <bool ARG>
__global__ __launch_bounds__(256) void k_pp_dilate(const float* __restrict__ tile_r, const int* __restrict__ tile_arg,
                                                   int TW, int TH, int K, float r_cap, float* __restrict__ rad,
                                                   int* __restrict__ rad_arg) {
  __shared__ float in[(DIL_H + 2 * DIL_K) * (DIL_W + 2 * DIL_K)], mid[(DIL_H + 2 * DIL_K) * DIL_W];
  __shared__ int ina[ARG ? (DIL_H + 2 * DIL_K) * (DIL_W + 2 * DIL_K) : 1], mida[ARG ? (DIL_H + 2 * DIL_K) * DIL_W : 1];
  const int tid = threadIdx.x, lx = tid & (DIL_W - 1), ly = tid / DIL_W;
  const int bx = blockIdx.x * DIL_W, by = blockIdx.y * DIL_H, tx = bx + lx, ty = by + ly;
  float m = -1.0f;
  int mi = 0x7fffffff;
  const auto take = [&](float v, int vi) {
    if (v > m || (ARG && v == m && vi < mi)) {
      m = v;
      mi = vi;
    }
  };
  if (K <= DIL_K) {
    const int IW = DIL_W + 2 * K, IH = DIL_H + 2 * K;
    for (int i = tid; i < IW * IH; i += 256) {
      const int r = i / IW, xx = bx - K + i - r * IW, yy = by - K + r;
      const bool in_grid = xx >= 0 && xx < TW && yy >= 0 && yy < TH;
      in[i] = in_grid ? tile_r[yy * TW + xx] : -1.0f;
      if (ARG) ina[i] = in_grid ? tile_arg[yy * TW + xx] : 0x7fffffff;
    }
    __syncthreads();
    for (int r = ly; r < IH; r += DIL_H) {
      m = -1.0f;
      mi = 0x7fffffff;
      for (int d = 0; d <= 2 * K; ++d) take(in[r * IW + lx + d], ARG ? ina[r * IW + lx + d] : 0);
      mid[r * DIL_W + lx] = m;
      if (ARG) mida[r * DIL_W + lx] = mi;
    }
    __syncthreads();
    m = -1.0f;
    mi = 0x7fffffff;
    for (int d = 0; d <= 2 * K; ++d) take(mid[(ly + d) * DIL_W + lx], ARG ? mida[(ly + d) * DIL_W + lx] : 0);
  } else if (tx < TW && ty < TH) {
    for (int yy = max(0, ty - K); yy <= min(TH - 1, ty + K); ++yy)
      for (int xx = max(0, tx - K); xx <= min(TW - 1, tx + K); ++xx)
        take(tile_r[yy * TW + xx], ARG ? tile_arg[yy * TW + xx] : 0);
  }
  if (tx >= TW || ty >= TH) return;
  rad[ty * TW + tx] = fminf(r_cap, ARG ? m : fmaxf(m, 0.0f));
  if (ARG) rad_arg[ty * TW + tx] = (m < r_cap && m > 0.0f) ? mi : -1;
}

// ---------------------------------------------------------------- gather
// Tap weights are carried in CoC-diameter units: for a tap with bilinear CoC
// c_q, the paper's weight (R^2/N) a / max(r_q, 0.5)^2 equals
// 4 (R^2/N) a / max(c_q^2, 1), so every tap uses a / max(c_q^2, 1) and the
// centre weight 1 / max(r_p, 0.5)^2 becomes 1 / ((R^2/N) max(c_p^2, 1)); the
// normalised sum is unchanged.  The effective radius in the same units is
// |c_q| - t max(0, |c_q| - |c_p|) (twice the radius form).
struct GatherAcc {
  float ap, ncpr, inv_ramp;  // |c_p|, -c_p / ramp, 1 / ramp
  float ar, ag, ab, ws;
  // (no implicit contraction of a product into a sum here or in tap(): the
  // gather's forms inline these into different code and must round alike)
  __device__ __forceinline__ void init(const float4& cp4, float R, int n_taps, float inv_ramp_) {
#pragma clang fp contract(off)
    inv_ramp = inv_ramp_;
    ap = fabsf(cp4.w);
    ncpr = -cp4.w * inv_ramp;
    const float q = fmaxf(cp4.w * cp4.w, 1.0f);
    const float w0 = R > 0.0f ? __builtin_amdgcn_rcpf(R * R / (float)n_taps * q) : 1.0f;
    ar = w0 * cp4.x;
    ag = w0 * cp4.y;
    ab = w0 * cp4.z;
    ws = w0;
  }
  // one tap: bilinear (rgb, c) from the four texels with weights
  // (w00, w10, w01, w11), d = 0.5 - R |u|
  // om: the tap's aberration weight (1: the disk's uniform weights)
  __device__ __forceinline__ void tap(float w00, float w10, float w01, float w11, float d, const float4& v00,
                                      const float4& v10, const float4& v01, const float4& v11, float om = 1.0f) {
#pragma clang fp contract(off)
    const float sr = fmaf(w11, v11.x, fmaf(w01, v01.x, fmaf(w10, v10.x, w00 * v00.x)));
    const float sg = fmaf(w11, v11.y, fmaf(w01, v01.y, fmaf(w10, v10.y, w00 * v00.y)));
    const float sb = fmaf(w11, v11.z, fmaf(w01, v01.z, fmaf(w10, v10.z, w00 * v00.z)));
    const float cq = fmaf(w11, v11.w, fmaf(w01, v01.w, fmaf(w10, v10.w, w00 * v00.w)));
    const float aq = fabsf(cq);
    const float tk = clamp01(fmaf(cq, inv_ramp, ncpr));
    const float reff2 = fmaf(-tk, fmaxf(0.0f, aq - ap), aq);
    const float a = clamp01(fmaf(reff2, 0.5f, d)) * om;
    const float wt = a * __builtin_amdgcn_rcpf(fmaxf(cq * cq, 1.0f));
    ar = fmaf(wt, sr, ar);
    ag = fmaf(wt, sg, ag);
    ab = fmaf(wt, sb, ab);
    ws += wt;
  }
  __device__ __forceinline__ void store(float* __restrict__ out, size_t N, size_t p) const {
    const float iw = 1.0f / ws;
    out[p] = ar * iw;
    out[N + p] = ag * iw;
    out[2 * N + p] = ab * iw;
  }
};

// Four clamp-to-edge texels of the bilinear footprint whose corner is (xa, ya).
__device__ __forceinline__ void texels_clamped(const float4* __restrict__ pack, int W, int H, int xa, int ya,
                                               float4& v00, float4& v10, float4& v01, float4& v11) {
  const int xa_ = clampi(xa, 0, W - 1), xb_ = clampi(xa + 1, 0, W - 1);
  const int ya_ = clampi(ya, 0, H - 1), yb_ = clampi(ya + 1, 0, H - 1);
  v00 = pack[(size_t)ya_ * W + xa_];
  v10 = pack[(size_t)ya_ * W + xb_];
  v01 = pack[(size_t)yb_ * W + xa_];
  v11 = pack[(size_t)yb_ * W + xb_];
}

// Tap record of the 16-pixel-tile gather: bilinear weights.
struct TapRec {
  float w00, w10, w01, w11;
};

#define PPG_G 4                 // taps per staged group (one per wave)
#define PPG_SIDE 17             // footprint side: 16 pixels + 1 bilinear neighbour
#define PPG_TEX (PPG_SIDE * PPG_SIDE)
#define PPG_SLOTS 5             // ceil(PPG_TEX / 64) texels staged per lane
#ifndef PPG_STRIDE
#define PPG_STRIDE 17           // LDS row stride of a staged footprint, in texels
#endif
#define PPG_TAPSZ (PPG_SIDE * PPG_STRIDE)
#ifndef PPG_BUFS
#define PPG_BUFS 2              // LDS ring: 2 = double-buffered groups, 1 = one group and a second barrier
#endif

// 16-pixel tiles: one 16x16 block per tile, blocks in XCD-contiguous order;
// the gather radius R and with it every tap's footprint offset and bilinear
// weights are uniform over the block.  For one tap the block's 256 pixels
// read the 17x17 texels at the tap's offset, each four times.  Taps are
// processed in groups of four: wave w stages tap w of the next group (its
// 17x17 clamp-to-edge texels, five 16-byte loads per lane, and the tap
// record) into one half of a double-buffered LDS ring while the block
// gathers the current group from the other half, so the vector-memory
// address unit (16 clocks per 64-lane load) handles 5 loads per wave and
// group instead of 16.
struct Stage {
  float4 v0, v1, v2, v3, v4;  // texels s * 64 + lane of the footprint, s = 0..4
  TapRec tr;
};

// Lane constants of the staging: footprint texel idx = s * 64 + lane lies at
// row idx / 17, column idx % 17 (lanes past the 289th texel repeat texel
// 256 + lane - 64 and do not store it); interior blocks address texels by a
// 32-bit byte offset from the footprint corner.
struct StageLane {
  int sr[PPG_SLOTS], sc[PPG_SLOTS];
  unsigned so[PPG_SLOTS];
  int lo[PPG_SLOTS];  // LDS texel index within the tap's footprint
  bool last;          // slot 4 holds a footprint texel of its own
};

// word 3 of a raw buffer resource on gfx9 (32-bit data format, no swizzle)
#define HDOF_BUFFER_WORD3 0x00020000

__device__ __forceinline__ float4 buffer_texel(__amdgpu_buffer_rsrc_t rs, unsigned voff, int soff) {
  const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, soff, 0);
  float4 f;
  __builtin_memcpy(&f, &v, sizeof f);
  return f;
}

// Texels and record of the tap with table entry u (wave-uniform) for the
// block at (x0, y0).
template <bool INTERIOR>
__device__ __forceinline__ Stage stage_load(const float4* __restrict__ pack, const float4 u, float R, int x0,
                                            int y0, int W, int H, const StageLane& sl) {
#pragma clang fp contract(off)
  Stage st;
  const float ox = R * u.x, oy = R * u.y;
  const float fx = floorf(ox), fy = floorf(oy);
  const float ax = ox - fx, ay = oy - fy, bx = 1.0f - ax, by = 1.0f - ay;
  st.tr.w00 = bx * by;
  st.tr.w10 = ax * by;
  st.tr.w01 = bx * ay;
  st.tr.w11 = ax * ay;
  const int gx0 = x0 + __builtin_amdgcn_readfirstlane((int)fx);
  const int gy0 = y0 + __builtin_amdgcn_readfirstlane((int)fy);
  if (INTERIOR) {
    // buffer loads: the footprint corner's byte offset as the scalar
    // offset, each lane's texel offset as the vector one (no per-lane 64-bit
    // address arithmetic; the resource spans the image, which interior
    // blocks require to be under 2 GiB)
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float4*>(pack), (short)0, W * H * 16, HDOF_BUFFER_WORD3);
    const int corner = __builtin_amdgcn_readfirstlane((gy0 * W + gx0) * 16);
    st.v0 = buffer_texel(rs, sl.so[0], corner);
    st.v1 = buffer_texel(rs, sl.so[1], corner);
    st.v2 = buffer_texel(rs, sl.so[2], corner);
    st.v3 = buffer_texel(rs, sl.so[3], corner);
    st.v4 = buffer_texel(rs, sl.so[4], corner);
  } else {
#define PPG_CLAMPED(s) pack[(size_t)clampi(gy0 + sl.sr[s], 0, H - 1) * W + clampi(gx0 + sl.sc[s], 0, W - 1)]
    st.v0 = PPG_CLAMPED(0);
    st.v1 = PPG_CLAMPED(1);
    st.v2 = PPG_CLAMPED(2);
    st.v3 = PPG_CLAMPED(3);
    st.v4 = PPG_CLAMPED(4);
#undef PPG_CLAMPED
  }
  return st;
}

__device__ __forceinline__ void stage_store_texels(float4* __restrict__ dst, const Stage& st, const StageLane& sl) {
  dst[sl.lo[0]] = st.v0;
  dst[sl.lo[1]] = st.v1;
  dst[sl.lo[2]] = st.v2;
  dst[sl.lo[3]] = st.v3;
  if (sl.last) dst[sl.lo[4]] = st.v4;
}

__device__ __forceinline__ void stage_store(float4* __restrict__ dst, TapRec* __restrict__ rdst, const Stage& st,
                                            const StageLane& sl, int lane) {
  stage_store_texels(dst, st, sl);
  if (lane == 0) *rdst = st.tr;
}

// The tap loop of one block.  Groups are always full: a wave whose tap of
// the group lies past n_taps stages the table's zero entry (the footprint
// at the block's corner), and that slot's distance term is -1e30 so its
// coverage, and with it its weight, is 0.
template <bool INTERIOR, bool SA>
__device__ __forceinline__ void gather_taps(float4 (*stg)[PPG_G * PPG_TAPSZ], TapRec (*rec)[PPG_G],
                                            const float4* __restrict__ pack, const float4* __restrict__ taps,
                                            int n_taps, float R, int x0, int y0, int W, int H, int wave, int lane,
                                            int lofs, bool inside, GatherAcc& g) {
  StageLane sl;
#pragma unroll
  for (int s = 0; s < PPG_SLOTS; ++s) {
    const int idx = s * 64 + lane < PPG_TEX ? s * 64 + lane : s * 64 + lane - 64;
    sl.sr[s] = idx / PPG_SIDE;
    sl.sc[s] = idx - sl.sr[s] * PPG_SIDE;
    sl.so[s] = (unsigned)(sl.sr[s] * W + sl.sc[s]) * 16u;
    sl.lo[s] = sl.sr[s] * PPG_STRIDE + sl.sc[s];
  }
  sl.last = lane < PPG_TEX - 4 * 64;
  const int ng = (n_taps + PPG_G - 1) / PPG_G;
  // The table entries of a group (four taps, 64 contiguous bytes of the
  // 256-entry table whose unused entries are zero) are read together right
  // after the group's barrier: the staging wave takes its own tap's offset
  // from them, the gather the taps' radii |u| and weights.  A scalar load's
  // wait also drains the LDS reads in flight, so no table read is left
  // inside the tap loop.
  // (four named values, and the wave's own entry read by its own scalar
  // load: an indexed array of them would live in scratch memory, and value
  // selects among them cost 14 vector instructions per group)
  float4 c0 = taps[0], c1 = taps[1], c2 = taps[2], c3 = taps[3];
  {
    const Stage st = stage_load<INTERIOR>(pack, taps[wave], R, x0, y0, W, H, sl);
    stage_store(stg[0] + wave * PPG_TAPSZ, &rec[0][wave], st, sl, lane);
  }
  for (int gi = 0; gi < ng; ++gi) {
    __syncthreads();
    const int b = PPG_BUFS == 2 ? gi & 1 : 0;
    const bool more = gi + 1 < ng;
    Stage st;
    float4 n0, n1, n2, n3;
    if (more) {
      const float4* tg = taps + (gi + 1) * PPG_G;
      n0 = tg[0];
      n1 = tg[1];
      n2 = tg[2];
      n3 = tg[3];
      st = stage_load<INTERIOR>(pack, tg[wave], R, x0, y0, W, H, sl);
    }
    if (inside) {
      const float4* src = stg[b] + lofs;
      const float uz[PPG_G] = {c0.z, c1.z, c2.z, c3.z}, uw[PPG_G] = {c0.w, c1.w, c2.w, c3.w};
#pragma unroll
      for (int jj = 0; jj < PPG_G; ++jj) {
        const bool valid = gi * PPG_G + jj < n_taps;
        const float d = valid ? fmaf(-R, uz[jj], 0.5f) : -1e30f;
        const float om = SA && valid ? uw[jj] : 1.0f;
        const float4* a = src + jj * PPG_TAPSZ;
        const TapRec t = rec[b][jj];
        g.tap(t.w00, t.w10, t.w01, t.w11, d, a[0], a[1], a[PPG_STRIDE], a[PPG_STRIDE + 1], om);
      }
    }
    if (more) {
      if (PPG_BUFS == 1) __syncthreads();  // every wave has read the group the next one overwrites
      stage_store(stg[PPG_BUFS == 2 ? b ^ 1 : 0] + wave * PPG_TAPSZ, &rec[PPG_BUFS == 2 ? b ^ 1 : 0][wave], st, sl,
                  lane);
      c0 = n0;
      c1 = n1;
      c2 = n2;
      c3 = n3;
    }
  }
}

// Composite applied in the gather's epilogue (whole frames): the same rules
// as k_composite, with the raster colour and CoC from the packed texel.
struct FuseK {
  const uint8_t* spp;
  const float *cn, *cf, *hr;
  float inv_ht;
  int rt_override;
  float* out;
  const float* pps;  // nullable: post-filtered specular luminance
  float inv_sy;      // 1 / spec_y, 0: no specular bokeh rule
};

// The composite's blend of one channel (paper, Composite): the traced
// colour crt = h C_tn + (1 - h) C_tf, the near rule nu, the focus-zone
// weight phi, the far blend beta and the specular weight sig.  Every
// product that meets a sum is an explicit fmaf, so the fused gather
// epilogue and the separate composite kernel round alike.
__device__ __forceinline__ float traced_mix(float h, float cn, float cf) { return fmaf(h, cn, (1.0f - h) * cf); }

__device__ __forceinline__ float composite_mix(float col, float cpp, float crt, float phi, float nu, float rho,
                                               float beta, float sig) {
  const float cnear = fmaf(sig, cpp - crt, crt);
  const float v_near = fmaf(rho, cnear, (1.0f - rho) * cpp);
  const float v_far = fmaf(beta, crt, (1.0f - beta) * cpp);
  const float oof = fmaf(nu, v_near, (1.0f - nu) * v_far);
  return fmaf(phi, oof, (1.0f - phi) * col);
}

// UNTRACED: every pixel takes the untraced pixels' rule (spp, the traced
// colours and pps are not read).
template <bool UNTRACED>
__device__ __forceinline__ void composite_px(const FuseK& fz, size_t N, size_t p, const float4& cp4, float pr,
                                             float pg, float pb) {
  const float c = cp4.w;
  const float phi = clamp01(fabsf(c) - HDOF_SQRT2);
  const float nu = clamp01(fmaf(-c, 0.35355339059327376f, 0.5f));
  const bool traced = !UNTRACED && fz.spp[p] > 0;
  const float h = traced ? fz.hr[p] : 0.0f;
  const float rho = traced ? 1.0f : 0.0f;
  const float beta = traced ? clamp01(1.0f - h * fz.inv_ht) : 0.0f;
  const float sig = (fz.pps && traced && fz.inv_sy > 0.0f) ? clamp01(fz.pps[p] * fz.inv_sy) : 0.0f;
  const float col[3] = {cp4.x, cp4.y, cp4.z}, cpp[3] = {pr, pg, pb};
  for (int q = 0; q < 3; ++q) {
    const size_t i = (size_t)q * N + p;
    const float crt = traced ? traced_mix(h, fz.cn[i], fz.cf[i]) : 0.0f;
    float o = composite_mix(col[q], cpp[q], crt, phi, nu, rho, beta, sig);
    if (fz.rt_override && traced) o = crt;
    fz.out[i] = o;
  }
}

// the filtered colour of pixel p: to `out` (may be NULL when fused) and,
// FUSE 1, through the composite, or FUSE 2, through the untraced pixels'
// rule of the composite
template <int FUSE>
__device__ __forceinline__ void pp_emit(float* __restrict__ out, const FuseK& fz, size_t N, size_t p,
                                        const float4& cp4, float pr, float pg, float pb) {
  if (out) {
    out[p] = pr;
    out[N + p] = pg;
    out[2 * N + p] = pb;
  }
  if (FUSE == 1) composite_px<false>(fz, N, p, cp4, pr, pg, pb);
  if (FUSE == 2) composite_px<true>(fz, N, p, cp4, pr, pg, pb);
}

// The gather radius of tile (tx, ty): min(r_cap, max tile radius within K
// tiles), reduced by the block (uniform result).
__device__ __forceinline__ float block_dilated_radius(const float* __restrict__ tile_r, int TW, int TH, int tx,
                                                      int ty, int K, float r_cap, float* wred) {
  const int D = 2 * K + 1, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float m = 0.0f;
  for (int i = tid; i < D * D; i += 256) {
    const int yy = ty - K + i / D, xx = tx - K + i % D;
    if (yy >= 0 && yy < TH && xx >= 0 && xx < TW) m = fmaxf(m, tile_r[yy * TW + xx]);
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if (lane == 0) wred[wave] = m;
  __syncthreads();
  return fminf(r_cap, fmaxf(fmaxf(wred[0], wred[1]), fmaxf(wred[2], wred[3])));
}

// 16-pixel tiles.  The block first reduces its tile's dilated radius from
// the per-tile maxima; FUSE 1 applies the composite to the result, FUSE 2
// the composite's rule for untraced pixels (the traced ones are rewritten
// later); SA weights the taps by the lens's spherical aberration (the
// table's fourth entry).
template <int FUSE, bool SA>
__device__ __forceinline__ void gather16_tile(float4 (*stg)[PPG_G * PPG_TAPSZ], TapRec (*rec)[PPG_G], float* wred,
                                              const float4* __restrict__ pack, const float* __restrict__ tile_r,
                                              int K, float r_cap, const float4* __restrict__ taps, int n_taps, int W,
                                              int H, float inv_ramp, float* __restrict__ out, const FuseK& fz,
                                              int tile) {
  const int TW = (W + 15) >> 4, TH = (H + 15) >> 4;
  const int x0 = (tile % TW) * 16, y0 = (tile / TW) * 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lx = lane & 15, ly = wave * 4 + (lane >> 4);
  const int x = x0 + lx, y = y0 + ly;
  const bool inside = x < W && y < H;
  const size_t N = (size_t)W * H, p = (size_t)y * W + x;
  const float R = block_dilated_radius(tile_r, TW, TH, tile % TW, tile / TW, K, r_cap, wred);
  if (!(R > 0.0f)) {
    if (inside) {
      const float4 c = pack[p];
      pp_emit<FUSE>(out, fz, N, p, c, c.x, c.y, c.z);
    }
    return;
  }
  const int E = (int)ceilf(R);
  const bool interior = x0 - E - 1 >= 0 && x0 + 16 + E < W && y0 - E - 1 >= 0 && y0 + 16 + E < H &&
                        (long long)W * H * 16 < (1ll << 31);
  const float4 cp4 = inside ? pack[p] : make_float4(0.f, 0.f, 0.f, 0.f);
  GatherAcc g;
  g.init(cp4, R, n_taps, inv_ramp);
  const int lofs = ly * PPG_STRIDE + lx;
  if (interior)
    gather_taps<true, SA>(stg, rec, pack, taps, n_taps, R, x0, y0, W, H, wave, lane, lofs, inside, g);
  else
    gather_taps<false, SA>(stg, rec, pack, taps, n_taps, R, x0, y0, W, H, wave, lane, lofs, inside, g);
  if (inside) {
    const float iw = 1.0f / g.ws;
    pp_emit<FUSE>(out, fz, N, p, cp4, g.ar * iw, g.ag * iw, g.ab * iw);
  }
}

// The tile at position L of an order that walks the tile grid in eight
// rectangles (4 across, 2 down), each row by row.  An XCD's contiguous
// share of positions (xcd_block) then covers about one rectangle, whose
// footprints (up to R_cap + 1 pixels around it) stay in that XCD's L2,
// instead of a full-width band of tile rows whose footprint rows exceed it
// (the quad form: 77.3 -> 49.2 MB fetched per 1080p launch, 151 -> 147 us).
__device__ __forceinline__ int rect_tile(int L, int TW, int TH) {
  int base = 0;
  for (int ry = 0; ry < 2; ++ry) {
    const int y0 = TH * ry / 2, y1 = TH * (ry + 1) / 2;
    for (int rx = 0; rx < 4; ++rx) {
      const int x0 = TW * rx / 4, x1 = TW * (rx + 1) / 4;
      const int n = (x1 - x0) * (y1 - y0);
      if (L < base + n) {
        const int o = L - base, w = x1 - x0;
        return (y0 + o / w) * TW + x0 + o % w;
      }
      base += n;
    }
  }
  return L;  // not reached for L < TW * TH
}

template <int FUSE, bool SA>
__global__ __launch_bounds__(256) void k_pp_gather16(const float4* __restrict__ pack, const float* __restrict__ tile_r,
                                                     int K, float r_cap, const float4* __restrict__ taps, int n_taps,
                                                     int W, int H, float inv_ramp, float* __restrict__ out, FuseK fz) {
  __shared__ float4 stg[PPG_BUFS][PPG_G * PPG_TAPSZ];
  __shared__ TapRec rec[PPG_BUFS][PPG_G];
  __shared__ float wred[4];
  // band order (an XCD's share is a band of tile rows): the rectangle
  // order cut this form's fetches from 57.9 to 41.4 MB but made the
  // overlapped frame slower (0.3923 against 0.3896 ms)
  const int tile = xcd_block(blockIdx.x, ((W + 15) >> 4) * ((H + 15) >> 4));
  gather16_tile<FUSE, SA>(stg, rec, wred, pack, tile_r, K, r_cap, taps, n_taps, W, H, inv_ramp, out, fz, tile);
}

// The batched form's gathers (the quad form) and traced pixels'
// composites, one launch each over every view: a wave (gather) or block
// (composite) finds its view by a binary search over the views' first
// tiles or first pixel blocks; a view's planes start at its px_base and its
// tile radii at its first tile.  The quad form is the batch's: there the
// gather sets the pace (32 views replayed 10.05 ms against 10.68 with the
// four-wave form).
struct PPBatch {
  int n;
  int tile_base[HDOF_MAX_VIEWS + 1];  // [n]: all tiles
  int blk_base[HDOF_MAX_VIEWS + 1];   // [n]: all blocks of HDOF_BATCH_PX_BLOCK pixels
  float* out[HDOF_MAX_VIEWS];
};

// The gather radius of tile (tx, ty) reduced by one wave (uniform result).
__device__ __forceinline__ float wave_dilated_radius(const float* __restrict__ tile_r, int TW, int TH, int tx,
                                                     int ty, int K, float r_cap) {
  const int D = 2 * K + 1, lane = threadIdx.x & 63;
  float m = 0.0f;
  for (int i = lane; i < D * D; i += 64) {
    const int yy = ty - K + i / D, xx = tx - K + i % D;
    if (yy >= 0 && yy < TH && xx >= 0 && xx < TW) m = fmaxf(m, tile_r[yy * TW + xx]);
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  return fminf(r_cap, m);
}

// Orders a wave's LDS stores before its later LDS loads (and its earlier
// loads before its later stores) across lanes: every LDS access in flight
// completes and the compiler moves none across.  No other wave takes part.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The tap loop of one wave whose lanes gather 2x2 pixel quads of one tile;
// per tap a lane reads the 3x3 staged texels its four bilinear footprints
// cover.  Software-pipelined over a two-buffer LDS ring: iteration t stores
// tap t + 1's texels (loaded during iteration t - 1, so a whole gather has
// covered their latency), issues tap t + 2's loads, and gathers tap t.
// Table entries are read two taps ahead; past the last tap the last one is
// staged again (unused), so nothing is carried on a conditional path.
template <bool INTERIOR, bool SA>
__device__ __forceinline__ void gather_taps_quad(float4 (*stg)[PPG_TAPSZ], const float4* __restrict__ pack,
                                                 const float4* __restrict__ taps, int n_taps, float R, int x0,
                                                 int y0, int W, int H, int lane, int lofs, GatherAcc (&g)[4]) {
  StageLane sl;
#pragma unroll
  for (int s = 0; s < PPG_SLOTS; ++s) {
    const int idx = s * 64 + lane < PPG_TEX ? s * 64 + lane : s * 64 + lane - 64;
    sl.sr[s] = idx / PPG_SIDE;
    sl.sc[s] = idx - sl.sr[s] * PPG_SIDE;
    sl.so[s] = (unsigned)(sl.sr[s] * W + sl.sc[s]) * 16u;
    sl.lo[s] = sl.sr[s] * PPG_STRIDE + sl.sc[s];
  }
  sl.last = lane < PPG_TEX - 4 * 64;
  const int last = n_taps - 1;
  const float4 e0 = taps[0];
  float4 e1 = taps[last < 1 ? last : 1], e2 = taps[last < 2 ? last : 2];
  TapRec tr;
  {
    const Stage s0 = stage_load<INTERIOR>(pack, e0, R, x0, y0, W, H, sl);
    stage_store_texels(stg[0], s0, sl);
    tr = s0.tr;
  }
  float uz = e0.z, uw = e0.w;
  Stage sn = stage_load<INTERIOR>(pack, e1, R, x0, y0, W, H, sl);  // tap 1 (in flight)
  for (int t = 0; t < n_taps; ++t) {
    wave_lds_sync();  // tap t's texels stored; tap t - 1's reads done
    const int b = t & 1;
    stage_store_texels(stg[b ^ 1], sn, sl);  // tap t + 1
    const TapRec trn = sn.tr;
    const float unz = e1.z, unw = e1.w;
    sn = stage_load<INTERIOR>(pack, e2, R, x0, y0, W, H, sl);  // tap t + 2
    e1 = e2;
    e2 = taps[t + 3 < last ? t + 3 : last];
    {
      const float4* a = stg[b] + lofs;
      const float4 v00 = a[0], v10 = a[1], v20 = a[2];
      const float4 v01 = a[PPG_STRIDE], v11 = a[PPG_STRIDE + 1], v21 = a[PPG_STRIDE + 2];
      const float4 v02 = a[2 * PPG_STRIDE], v12 = a[2 * PPG_STRIDE + 1], v22 = a[2 * PPG_STRIDE + 2];
      const float d = fmaf(-R, uz, 0.5f);
      const float om = SA ? uw : 1.0f;
      g[0].tap(tr.w00, tr.w10, tr.w01, tr.w11, d, v00, v10, v01, v11, om);
      g[1].tap(tr.w00, tr.w10, tr.w01, tr.w11, d, v10, v20, v11, v21, om);
      g[2].tap(tr.w00, tr.w10, tr.w01, tr.w11, d, v01, v11, v02, v12, om);
      g[3].tap(tr.w00, tr.w10, tr.w01, tr.w11, d, v11, v21, v12, v22, om);
    }
    tr = trn;
    uz = unz;
    uw = unw;
  }
}

// 16-pixel tiles, one wave per tile (the quad form): lane l gathers the
// 2x2 quad at (2 (l mod 8), 2 (l div 8)) of its tile, so per tap a tile
// reads 2.25 staged texels per pixel from LDS instead of 4, and each wave
// stages its own taps into its own ring (no barrier between waves).  A
// block holds four neighbouring tiles, so it frees as much LDS at a time
// as the four-wave form does (a kernel running beside it, such as the ray
// mask, needs whole blocks' worth).  Same arithmetic, in the same tap
// order, as k_pp_gather16, so the same results bit for bit.
template <int FUSE, bool SA>
__device__ __forceinline__ void gather16q_tile(float4 (*stg)[PPG_TAPSZ], const float4* __restrict__ pack,
                                               const float* __restrict__ tile_r, int K, float r_cap,
                                               const float4* __restrict__ taps, int n_taps, int W, int H,
                                               float inv_ramp, float* __restrict__ out, const FuseK& fz, int tile) {
  const int TW = (W + 15) >> 4, TH = (H + 15) >> 4;
  const int x0 = (tile % TW) * 16, y0 = (tile / TW) * 16;
  const int lane = threadIdx.x & 63;
  const int qx = (lane & 7) * 2, qy = (lane >> 3) * 2;
  const size_t N = (size_t)W * H;
  const float R = wave_dilated_radius(tile_r, TW, TH, tile % TW, tile / TW, K, r_cap);
  if (!(R > 0.0f)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int x = x0 + qx + (q & 1), y = y0 + qy + (q >> 1);
      if (x < W && y < H) {
        const size_t p = (size_t)y * W + x;
        const float4 c = pack[p];
        pp_emit<FUSE>(out, fz, N, p, c, c.x, c.y, c.z);
      }
    }
    return;
  }
  const int E = (int)ceilf(R);
  const bool interior = x0 - E - 1 >= 0 && x0 + 16 + E < W && y0 - E - 1 >= 0 && y0 + 16 + E < H &&
                        (long long)W * H * 16 < (1ll << 31);
  GatherAcc g[4];
  float4 cp[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int x = x0 + qx + (q & 1), y = y0 + qy + (q >> 1);
    cp[q] = x < W && y < H ? pack[(size_t)y * W + x] : make_float4(0.f, 0.f, 0.f, 0.f);
    g[q].init(cp[q], R, n_taps, inv_ramp);
  }
  const int lofs = qy * PPG_STRIDE + qx;
  if (interior)
    gather_taps_quad<true, SA>(stg, pack, taps, n_taps, R, x0, y0, W, H, lane, lofs, g);
  else
    gather_taps_quad<false, SA>(stg, pack, taps, n_taps, R, x0, y0, W, H, lane, lofs, g);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int x = x0 + qx + (q & 1), y = y0 + qy + (q >> 1);
    if (x < W && y < H) {
      const size_t p = (size_t)y * W + x;
      const float iw = 1.0f / g[q].ws;
      pp_emit<FUSE>(out, fz, N, p, cp[q], g[q].ar * iw, g[q].ag * iw, g[q].ab * iw);
    }
  }
}

template <int FUSE, bool SA>
__global__ __launch_bounds__(256) void k_pp_gather16q(const float4* __restrict__ pack,
                                                      const float* __restrict__ tile_r, int K, float r_cap,
                                                      const float4* __restrict__ taps, int n_taps, int W, int H,
                                                      float inv_ramp, float* __restrict__ out, FuseK fz) {
  __shared__ float4 stg[4][2][PPG_TAPSZ];
  const int TW = (W + 15) >> 4, TH = (H + 15) >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pos = xcd_block(blockIdx.x, (TW * TH + 3) >> 2) * 4 + wave;
  if (pos >= TW * TH) return;
  const int tile = rect_tile(pos, TW, TH);
  gather16q_tile<FUSE, SA>(stg[wave], pack, tile_r, K, r_cap, taps, n_taps, W, H, inv_ramp, out, fz, tile);
}

// The batched form's gathers in the quad form: each wave finds the view of
// its own tile (a block's four tiles may straddle two views).
template <bool SA>
__global__ __launch_bounds__(256) void k_pp_gather16q_batch(const float4* __restrict__ pack,
                                                            const float* __restrict__ tile_r, int K, float r_cap,
                                                            const float4* __restrict__ taps, int n_taps,
                                                            float inv_ramp, float* __restrict__ pp_out,
                                                            const BatchView* __restrict__ views, PPBatch b) {
  __shared__ float4 stg[4][2][PPG_TAPSZ];
  const int total = b.tile_base[b.n];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = xcd_block(blockIdx.x, (total + 3) >> 2) * 4 + wave;
  if (g >= total) return;
  const int v = __builtin_amdgcn_readfirstlane(batch_view_of(b.tile_base, b.n, g));
  const int W = views[v].k.W, H = views[v].k.H;
  const size_t pb = (size_t)views[v].px_base;
  FuseK fz{};
  fz.out = b.out[v];
  gather16q_tile<2, SA>(stg[wave], pack + pb, tile_r + b.tile_base[v], K, r_cap, taps, n_taps, W, H, inv_ramp,
                        pp_out + 3 * pb, fz, g - b.tile_base[v]);
}

// Tiles of 4 or 8 pixels: per-lane radius and per-lane tap geometry, every
// texel clamped to the edge.  Bound: the texel loads (a 64-lane load of
// float4s at four rows' places takes a CU about 30 clocks): 48 taps, 1280x720,
// 8-pixel tiles 90 us.  (A wave's texels staged in LDS are as many LDS reads:
// 84, and 5 us slower on small images and 6 % on 4-pixel tiles; four pixels of
// a column per lane, 10 texels for 16: 150, their footprints leave the L1.)
__global__ __launch_bounds__(256) void k_pp_gather_any(const float4* __restrict__ pack, const float* __restrict__ rad,
                                                       const float4* __restrict__ taps, int n_taps, int W, int H,
                                                       int tile, float inv_ramp, float* __restrict__ out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int x = blockIdx.x * 16 + (lane & 15), y = blockIdx.y * 16 + wave * 4 + (lane >> 4);
  if (x >= W || y >= H) return;
  const int TW = (W + tile - 1) / tile;
  const size_t N = (size_t)W * H, p = (size_t)y * W + x;
  const float R = rad[(y / tile) * TW + x / tile];
  const float4 cp4 = pack[p];
  GatherAcc g;
  g.init(cp4, R, n_taps, inv_ramp);
  if (R > 0.0f) {
    for (int k = 0; k < n_taps; ++k) {
      const float4 u = taps[k];
      const float ox = R * u.x, oy = R * u.y;
      const float fx = floorf(ox), fy = floorf(oy);
      const float ax = ox - fx, ay = oy - fy, bx = 1.0f - ax, by = 1.0f - ay;
      float4 v00, v10, v01, v11;
      texels_clamped(pack, W, H, x + (int)fx, y + (int)fy, v00, v10, v01, v11);
      g.tap(bx * by, ax * by, bx * ay, ax * ay, 0.5f - R * u.z, v00, v10, v01, v11, u.w);
    }
  }
  g.store(out, N, p);
}

// One wave's taps (wave, wave + 4, ...) of the specular gather for 8x8 pixels
// of one radius R.  Per tap the pixels read the same 9x9 texels, of which
// only the luminance and the CoC matter: the wave stages them in its own
// two-buffer LDS ring a tap ahead; lane i forms the geometry of its i-th tap.
#define PPS_SIDE 9
#define PPS_TEX (PPS_SIDE * PPS_SIDE)
template <bool INTERIOR>
__device__ __forceinline__ void spec_taps8(float2 (*stg)[PPS_TEX], const float4* __restrict__ pack,
                                           const float* __restrict__ ys, const float4* __restrict__ taps, int n_taps,
                                           int wave, float R, int xw, int yw, int W, int H, int lane, GatherAcc& g) {
  const int n = (n_taps - wave + 3) >> 2;
  if (n <= 0) return;
  // (INTERIOR: the image's bytes were checked to fit an int; the other form reads by pointer)
  const int px = INTERIOR ? W * H : 0;
  const __amdgpu_buffer_rsrc_t rp =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(pack), (short)0, px * 16, HDOF_BUFFER_WORD3);
  const __amdgpu_buffer_rsrc_t ry =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(ys), (short)0, px * 4, HDOF_BUFFER_WORD3);
  int sx[2], sy[2], vo[2];  // the lane's two texels of a tap, relative to its corner
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int i = min(s * 64 + lane, PPS_TEX - 1);
    sy[s] = i / PPS_SIDE;
    sx[s] = i - sy[s] * PPS_SIDE;
    vo[s] = sy[s] * W + sx[s];
  }
  const float4 u = taps[min(wave + 4 * lane, n_taps - 1)];
  const float ox = R * u.x, oy = R * u.y;
  const float fx = floorf(ox), fy = floorf(oy);
  const float ax = ox - fx, ay = oy - fy, bx = 1.0f - ax, by = 1.0f - ay;
  const float w00 = bx * by, w10 = ax * by, w01 = bx * ay, w11 = ax * ay, d = 0.5f - R * u.z;
  const int gx = xw + (int)fx, gy = yw + (int)fy, corner = gy * W + gx;
  const auto rl = [](float v, int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i)); };
  const auto texel = [&](int s, int i) {
    if (INTERIOR) {
      const int c = __builtin_amdgcn_readlane(corner, i);
      return make_float2(__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ry, vo[s] * 4, c * 4, 0)),
                         __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rp, vo[s] * 16 + 12, c * 16, 0)));
    }
    const size_t q = (size_t)clampi(__builtin_amdgcn_readlane(gy, i) + sy[s], 0, H - 1) * W +
                     clampi(__builtin_amdgcn_readlane(gx, i) + sx[s], 0, W - 1);
    return make_float2(ys[q], pack[q].w);
  };
  const int at = (lane >> 3) * PPS_SIDE + (lane & 7);
  stg[0][lane] = texel(0, 0);
  if (lane < PPS_TEX - 64) stg[0][64 + lane] = texel(1, 0);
  for (int k = 0; k < n; ++k) {
    wave_lds_sync();  // tap k's texels stored; tap k - 1's reads done
    const int kn = k + 1 < n ? k + 1 : k;
    const float2 t0 = texel(0, kn), t1 = texel(1, kn);
    const float2* a = stg[k & 1] + at;
    const float2 q00 = a[0], q10 = a[1], q01 = a[PPS_SIDE], q11 = a[PPS_SIDE + 1];
    g.tap(rl(w00, k), rl(w10, k), rl(w01, k), rl(w11, k), rl(d, k), make_float4(q00.x, 0.f, 0.f, q00.y),
          make_float4(q10.x, 0.f, 0.f, q10.y), make_float4(q01.x, 0.f, 0.f, q01.y),
          make_float4(q11.x, 0.f, 0.f, q11.y), rl(u.w, k));
    float2* const o = stg[(k & 1) ^ 1];
    o[lane] = t0;
    if (lane < PPS_TEX - 64) o[64 + lane] = t1;
  }
}

// The post-filtered specular luminance (the specular bokeh rule of the
// composite): the post-filter's gather, radius, taps and weights, applied to
// the G-buffer's specular luminance plane.  With spp given only traced
// pixels gather (the rule reads no other), the rest are 0.  One 8x8 block (a
// ray-mask tile) per 256 threads, a pixel per lane, the four waves splitting
// the taps (tap j on wave j mod 4, sums joined in LDS), so the few traced
// tiles of a frame get four times the parallelism of a lane per pixel; a
// block without a traced pixel writes 0 and leaves.  A block of one radius
// (tiles of 8 or 16 pixels) stages its texels (spec_taps8), else every lane
// reads its own.  Bound: latency.  2560x1440 frame: 259 us with four lanes a
// pixel, eight loads and their addresses per tap, 165 so (16x16 pixels per
// block, the traced quarters one after another: 202).
// Blocks run in launch order, round-robin over the XCDs (the traced pixels
// cluster along a few silhouettes, which XCD-contiguous ranges would give to
// one XCD).
// Radius: tile 16, the dilated radius of the block's 16-pixel tile from
// tile_r; otherwise the pixel's tile entry of the dilated radii.
__global__ __launch_bounds__(256) void k_pp_spec(const float4* __restrict__ pack, const float* __restrict__ ys,
                                                 const uint8_t* __restrict__ spp, const float* __restrict__ tile_r,
                                                 const float* __restrict__ rad, int tile, int K, float r_cap,
                                                 const float4* __restrict__ taps, int n_taps, int W, int H,
                                                 float inv_ramp, float* __restrict__ out) {
  __shared__ float wred[4];
  __shared__ float2 ring[4][2][PPS_TEX], sum[4][64];
  const int BW = (W + 7) >> 3;
  const int bx = blockIdx.x % BW, by = blockIdx.x / BW, xw = bx * 8, yw = by * 8;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int x = xw + (lane & 7), y = yw + (lane >> 3);
  const bool in = x < W && y < H;
  const size_t p = in ? (size_t)y * W + x : 0;
  const bool act = in && (!spp || spp[p] > 0);
  if (__builtin_amdgcn_ballot_w64(act) == 0ull) {  // (the waves have the same pixels)
    if (in && wave == 0) out[p] = 0.0f;
    return;
  }
  float R;
  if (tile == 16) {
    R = block_dilated_radius(tile_r, (W + 15) >> 4, (H + 15) >> 4, bx >> 1, by >> 1, K, r_cap, wred);
  } else {
    const int TW = (W + tile - 1) / tile;
    R = rad[(min(y, H - 1) / tile) * TW + min(x, W - 1) / tile];
  }
  GatherAcc g;
  g.init(make_float4(ys[p], 0.0f, 0.0f, pack[p].w), R, n_taps, inv_ramp);
  if (wave != 0) g.ar = g.ws = 0.0f;  // the centre counts once
  if (tile >= 8) {
    R = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(R)));
    const int E = (int)ceilf(R);
    if (xw - E - 1 >= 0 && xw + 8 + E < W && yw - E - 1 >= 0 && yw + 8 + E < H && (long long)W * H * 16 < (1ll << 31))
      spec_taps8<true>(ring[wave], pack, ys, taps, n_taps, wave, R, xw, yw, W, H, lane, g);
    else
      spec_taps8<false>(ring[wave], pack, ys, taps, n_taps, wave, R, xw, yw, W, H, lane, g);
  } else if (act) {
    for (int j = wave; j < n_taps; j += 4) {
      const float4 u = taps[j];
      const float ox = R * u.x, oy = R * u.y;
      const float fx = floorf(ox), fy = floorf(oy);
      const float ax = ox - fx, ay = oy - fy, bxw = 1.0f - ax, byw = 1.0f - ay;
      const int xa = x + (int)fx, ya = y + (int)fy;
      const int xa_ = clampi(xa, 0, W - 1), xb_ = clampi(xa + 1, 0, W - 1);
      const size_t ra = (size_t)clampi(ya, 0, H - 1) * W, rb = (size_t)clampi(ya + 1, 0, H - 1) * W;
      const auto at = [&](size_t i) { return make_float4(ys[i], 0.0f, 0.0f, pack[i].w); };
      g.tap(bxw * byw, ax * byw, bxw * ay, ax * ay, 0.5f - R * u.z, at(ra + xa_), at(ra + xb_), at(rb + xa_),
            at(rb + xb_), u.w);
    }
  }
  sum[wave][lane] = make_float2(g.ar, g.ws);
  __syncthreads();
  if (wave != 0 || !in) return;
  const float2 a = sum[0][lane], b = sum[1][lane], c = sum[2][lane], d = sum[3][lane];
  out[p] = act ? ((a.x + b.x) + (c.x + d.x)) / ((a.y + b.y) + (c.y + d.y)) : 0.0f;
}

// pps (nullable): the post-filtered specular luminance; inv_sy = 1 / spec_y
// (0: the specular bokeh rule is off)
struct CompK {
  const float *color, *pp, *depth;
  const uint8_t* spp;
  const float *cn, *cf, *hr;
  LensK l;
  int N;
  float inv_ht;
  int rt_override;
  const float* pps;
  float inv_sy;
  float* out;
};

__device__ __forceinline__ void composite_at(const CompK& a, int p) {
  const int N = a.N;
  const float c = coc_px(a.l, a.depth[p]);
  const float phi = clamp01(fabsf(c) - HDOF_SQRT2);
  const float nu = clamp01(fmaf(-c, 0.35355339059327376f, 0.5f));
  // the traced colours enter only where the pixel was traced, the filtered
  // colour only outside the focus zone: other loads are skipped (the mask
  // leaves most 64-pixel rows untraced, so their lines are never fetched)
  const bool traced = a.spp[p] > 0;
  const float h = traced ? a.hr[p] : 0.0f;
  const float rho = traced ? 1.0f : 0.0f;
  const float beta = traced ? clamp01(1.0f - h * a.inv_ht) : 0.0f;
  const float sig = (a.pps && traced && a.inv_sy > 0.0f) ? clamp01(a.pps[p] * a.inv_sy) : 0.0f;
  for (int q = 0; q < 3; ++q) {
    size_t i = (size_t)q * N + p;
    const float crt = traced ? traced_mix(h, a.cn[i], a.cf[i]) : 0.0f;
    const float cpp = phi > 0.0f ? a.pp[i] : 0.0f;
    float o = composite_mix(a.color[i], cpp, crt, phi, nu, rho, beta, sig);
    if (a.rt_override && traced) o = crt;
    a.out[i] = o;
  }
}

__global__ void k_composite(CompK a) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < a.N) composite_at(a, p);
}

// Traced pixels only (the others hold the untraced rule's result).  One
// thread per pixel: with four pixels per thread the traced pixels' loads
// serialise and the pass is slower (12.5 against 9.8 µs at 1080p).
__global__ void k_composite_traced(CompK a) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < a.N && a.spp[p] > 0) composite_at(a, p);
}

// every view's traced pixels in one launch, HDOF_BATCH_PX_BLOCK pixels per
// block; `a` holds the first view's planes (all views' planes are
// concatenated from their px_base)
__global__ void k_composite_traced_batch(CompK a, const BatchView* __restrict__ views, PPBatch b) {
  const int v = batch_view_of(b.blk_base, b.n, blockIdx.x);
  const int N = views[v].k.W * views[v].k.H;
  const size_t pb = (size_t)views[v].px_base;
  CompK c = a;
  c.color += 3 * pb;
  c.pp += 3 * pb;
  c.depth += pb;
  c.spp += pb;
  c.cn += 3 * pb;
  c.cf += 3 * pb;
  c.hr += pb;
  c.l = views[v].l;
  c.N = N;
  c.out = b.out[v];
  const int p0 = (blockIdx.x - b.blk_base[v]) * HDOF_BATCH_PX_BLOCK;
  for (int i = threadIdx.x; i < HDOF_BATCH_PX_BLOCK; i += blockDim.x) {
    const int p = p0 + i;
    if (p >= N) break;
    if (c.spp[p] > 0) composite_at(c, p);
  }
}

// ---------------------------------------------------------------------------
// Adjoint of post-filter + composite (differentiable form).
// Reverse mode for the colour (the gather's transpose: every tap's share goes
// back to its four bilinear texels), forward mode for
// the focus distance S1 and aperture A (each value carries its two
// derivatives through the recomputed gather: no weights are stored).
// ---------------------------------------------------------------------------
struct D3 {
  float v, s, a;  // value, d/dS1, d/dA
};
__device__ inline D3 dk(float v, float s, float a) { return D3{v, s, a}; }
__device__ inline D3 dc(float v) { return D3{v, 0.f, 0.f}; }
__device__ inline D3 operator+(D3 x, D3 y) { return D3{x.v + y.v, x.s + y.s, x.a + y.a}; }
__device__ inline D3 operator-(D3 x, D3 y) { return D3{x.v - y.v, x.s - y.s, x.a - y.a}; }
__device__ inline D3 operator*(D3 x, D3 y) { return D3{x.v * y.v, fmaf(x.s, y.v, x.v * y.s), fmaf(x.a, y.v, x.v * y.a)}; }
__device__ inline D3 operator*(float k, D3 x) { return D3{k * x.v, k * x.s, k * x.a}; }
__device__ inline D3 dquot(D3 x, D3 y) {
  const float iy = __builtin_amdgcn_rcpf(y.v), q = x.v * iy;
  return D3{q, (x.s - q * y.s) * iy, (x.a - q * y.a) * iy};
}
// clamp with zero slope outside the open interval (lo, hi)
__device__ inline D3 dclamp(D3 x, float lo, float hi) { return x.v <= lo ? dc(lo) : (x.v >= hi ? dc(hi) : x); }
__device__ inline D3 dmaxc(D3 x, float c) { return x.v > c ? x : dc(c); }
__device__ inline D3 dabs(D3 x) { return x.v >= 0.f ? x : D3{-x.v, -x.s, -x.a}; }

// pack (rgb, c), the CoCs by themselves, tile max with its pixel
__global__ __launch_bounds__(256) void k_ppb_pack(const float* __restrict__ color, const float* __restrict__ depth,
                                                  CamK k, LensK l, int tile, float4* __restrict__ pack,
                                                  float* __restrict__ coc, float* __restrict__ tile_r,
                                                  int* __restrict__ tile_arg) {
  __shared__ float red[256];
  __shared__ int redi[256];
  const int tid = threadIdx.x;
  const int BX = (k.W + 15) >> 4, lb = xcd_block(blockIdx.x, BX * ((k.H + 15) >> 4));
  const int x = (lb % BX) * 16 + (tid & 15), y = (lb / BX) * 16 + (tid >> 4);
  const size_t N = (size_t)k.W * k.H;
  float r = -1.0f;
  int idx = 0x7fffffff;
  if (x < k.W && y < k.H) {
    size_t p = (size_t)y * k.W + x;
    float c = coc_px(l, depth[p]);
    pack[p] = make_float4(color[p], color[N + p], color[2 * N + p], c);
    coc[p] = c;
    r = 0.5f * fabsf(c);
    idx = (int)p;
  }
  red[tid] = r;
  redi[tid] = idx;
  __syncthreads();
  // the largest radius of each tile and its lowest pixel index: first along
  // each tile row (the row's first thread), then over the tile's rows
  const int tx = tid & 15, ty = tid >> 4;
  __shared__ float rowm[256];
  __shared__ int rowi[256];
  if ((tx % tile) == 0) {
    float m = -1.0f;
    int mi = 0x7fffffff;
    for (int dx = 0; dx < tile; ++dx) {
      const float v = red[ty * 16 + tx + dx];
      const int vi = redi[ty * 16 + tx + dx];
      if (v > m || (v == m && vi < mi)) {
        m = v;
        mi = vi;
      }
    }
    rowm[tid] = m;
    rowi[tid] = mi;
  }
  __syncthreads();
  if ((tx % tile) == 0 && (ty % tile) == 0 && x < k.W && y < k.H) {
    float m = -1.0f;
    int mi = 0x7fffffff;
    for (int dy = 0; dy < tile; ++dy) {
      const float v = rowm[(ty + dy) * 16 + tx];
      const int vi = rowi[(ty + dy) * 16 + tx];
      if (v > m || (v == m && vi < mi)) {
        m = v;
        mi = vi;
      }
    }
    const int TW = (k.W + tile - 1) / tile;
    tile_r[(y / tile) * TW + x / tile] = m;
    tile_arg[(y / tile) * TW + x / tile] = mi;
  }
}

__global__ void k_fill_f(float* __restrict__ p, size_t n, float v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Sample geometry of a tap at radius R relative to a pixel's texel grid: the
// footprint corner offset (floor R u) and the bilinear fractions.
struct TapGeo {
  int ix, iy;
  float ax, ay;
};
__device__ __forceinline__ TapGeo tap_geo(float R, float4 u) {
  const float ox = R * u.x, oy = R * u.y;
  const float fx = floorf(ox), fy = floorf(oy);
  return TapGeo{(int)fx, (int)fy, ox - fx, oy - fy};
}

#ifndef PPB_WIN_E
#define PPB_WIN_E 20                            // largest |offset| accumulated in a block's LDS window
#endif
static_assert(17 + 2 * PPB_WIN_E <= 64, "a window row per wave");
#ifndef PPB_MINW
#define PPB_MINW 1
#endif
#ifndef PPB_G
#define PPB_G 5                                 // taps whose weights are exchanged at a time
#endif
#define PPB_WIN (17 + 2 * PPB_WIN_E)            // the window's side
#define PPB_WS ((PPB_WIN + 3) / 8 * 8 + 4)      // its row stride: the four rows a wave adds to at a time lie in different banks
// that of a smaller window, which leaves a footprint's space behind its channels
#define PPB_FAR_E 19
#define PPB_PLANE (((17 + 2 * PPB_FAR_E) * PPB_WS + PPG_SIDE * PPG_SIDE + 3) / 4 * 4)  // a channel's
static_assert(PPB_WIN * PPB_WS <= PPB_PLANE, "either window");
#define PPB_SUMS 9
enum { S_W, S_C, S_A, S_R, S_GW, S_GC, S_GA, S_GR, S_GM };

// The 5x2 texels whose corner is (x, y), clamped to the edge: packed texels,
// or the CoCs alone.  INTERIOR: none lies outside the image (buffer loads,
// their row in the scalar offset).
template <bool INTERIOR>
struct FootRows {
  int W, H, ya;
  unsigned xa, xb;  // INTERIOR: xa is the corner's index
  __device__ __forceinline__ FootRows(int W_, int H_, int x, int y) : W(W_), H(H_), ya(y) {
    if (INTERIOR) {
      xa = __umul24((unsigned)y, (unsigned)W) + (unsigned)x;
      xb = xa + 1;
    } else {
      xa = (unsigned)clampi(x, 0, W - 1);
      xb = (unsigned)clampi(x + 1, 0, W - 1);
    }
  }
  __device__ __forceinline__ void texels(const float4* __restrict__ pack, int j, float4& v0, float4& v1) const {
    if (INTERIOR) {
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float4*>(pack), (short)0, W * H * 16, HDOF_BUFFER_WORD3);
      v0 = buffer_texel(rs, xa << 4, j * W * 16);
      v1 = buffer_texel(rs, (xa << 4) + 16, j * W * 16);
    } else {
      const unsigned row = __umul24((unsigned)clampi(ya + j, 0, H - 1), (unsigned)W);
      v0 = *(const float4*)((const char*)pack + ((row + xa) << 4));
      v1 = *(const float4*)((const char*)pack + ((row + xb) << 4));
    }
  }
  __device__ __forceinline__ float2 cocs(const float* __restrict__ coc, int j) const {
    if (INTERIOR) {
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(coc), (short)0, W * H * 4, HDOF_BUFFER_WORD3);
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(xa << 2), j * W * 4, 0);
      float2 f;
      __builtin_memcpy(&f, &v, sizeof f);
      return f;
    }
    const unsigned row = __umul24((unsigned)clampi(ya + j, 0, H - 1), (unsigned)W);
    return make_float2(*(const float*)((const char*)coc + ((row + xa) << 2)),
                       *(const float*)((const char*)coc + ((row + xb) << 2)));
  }
};

// What one lane keeps of its four pixels for pass 1.
struct PpbPx {
  float c[4], g[3][4], gc[4];  // CoC, incoming gradient, and the pixel's own colour projected on it
};

// Pass 1: the sums of one lane's four pixels over the wave's taps.  A tap's
// weight w = a / max(c_q^2, 1) (see GatherAcc) depends on the sample's CoC
// c_q, the pixel's CoC c_p and the tile radius R, of which S1 and A move all
// CoCs by dcs and c / A and the radius by R.s and R.a, and the samples along
// u with it.  So four sums of the weight and of its partial derivatives
// (S_C: d/dc_q + d/dc_p; S_A: the same times the CoCs; S_R: by R, area and
// motion along u included but for 2 w / R), the same four times the sample's
// colour projected on the pixel's incoming gradient (S_G*), and the motion of
// that projection (S_GM) give both derivatives of the composite: nine
// scalar sums in place of four values of three channels and their weight.
// MOVES: the tile radius moves (it is not at its cap).
template <bool MOVES>
__device__ __forceinline__ void ppb_sums(const float4 (&v0)[5], const float4 (&v1)[5], const float4& u, float ax,
                                         float ay, float R, float inv_ramp, const PpbPx& px,
                                         float (&S)[PPB_SUMS][4]) {
  const float d = fmaf(-R, u.z, 0.5f), uz2 = 2.f * u.z;
  const float dxb = u.x * (1.f - ay), dxa = u.x * ay;
  // a row's slope along x, and its interpolation
  float4 e0 = make_float4(v1[0].x - v0[0].x, v1[0].y - v0[0].y, v1[0].z - v0[0].z, v1[0].w - v0[0].w);
  const float bx = 1.f - ax, by = 1.f - ay;
  float4 h0 = make_float4(fmaf(ax, v1[0].x, bx * v0[0].x), fmaf(ax, v1[0].y, bx * v0[0].y), fmaf(ax, v1[0].z, bx * v0[0].z),
                          fmaf(ax, v1[0].w, bx * v0[0].w));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 a0 = v0[q + 1], a1 = v1[q + 1];
    const float4 e1 = make_float4(a1.x - a0.x, a1.y - a0.y, a1.z - a0.z, a1.w - a0.w);
    const float4 h1 = make_float4(fmaf(ax, a1.x, bx * a0.x), fmaf(ax, a1.y, bx * a0.y), fmaf(ax, a1.z, bx * a0.z),
                                  fmaf(ax, a1.w, bx * a0.w));
    const float4 f1 = make_float4(h1.x - h0.x, h1.y - h0.y, h1.z - h0.z, h1.w - h0.w);  // slope along y
    const float g0 = px.g[0][q], g1 = px.g[1][q], g2 = px.g[2][q];
    const float cq = fmaf(ay, h1.w, by * h0.w);
    const float gy = fmaf(g2, f1.z, fmaf(g1, f1.y, g0 * f1.x));
    const float sg = fmaf(g2, fmaf(ay, h1.z, by * h0.z), fmaf(g1, fmaf(ay, h1.y, by * h0.y), fmaf(g0, fmaf(ay, h1.x, by * h0.x), -px.gc[q])));
    const float cp = px.c[q];
    const float aq = fabsf(cq), raw = (cq - cp) * inv_ramp;
    const float tk = clamp01(raw), dp = fmaxf(0.f, aq - fabsf(cp));
    const float reff = fmaf(-tk, dp, aq);
    const float araw = fmaf(reff, 0.5f, d);
    const float c2 = cq * cq, irq = __builtin_amdgcn_rcpf(fmaxf(c2, 1.f));
    const float w = clamp01(araw) * irq;
    const float kh = araw > 0.f && araw < 1.f ? 0.5f * irq : 0.f;
    const bool ramp = raw > 0.f && raw < 1.f;
    const float tm = dp > 0.f ? tk : 0.f;
    const float f = copysignf(1.f - tm, cq);
    const float w2 = c2 > 1.f ? 2.f * w : 0.f, T = w2 * (irq * cq);
    const float wc = fmaf(kh, fmaf(copysignf(1.f, cp), tm, f), -T);
    const float wa = fmaf(kh, fmaf(-(ramp ? raw : 0.f), dp, reff), -w2);
    S[S_W][q] += w;
    S[S_C][q] += wc;
    S[S_A][q] += wa;
    S[S_GW][q] = fmaf(w, sg, S[S_GW][q]);
    S[S_GC][q] = fmaf(wc, sg, S[S_GC][q]);
    S[S_GA][q] = fmaf(wa, sg, S[S_GA][q]);
    if (MOVES) {
      // slopes along u: of the CoC, and of the projected colour
      const float mc = fmaf(u.y, f1.w, fmaf(dxa, e1.w, dxb * e0.w));
      const float mx = fmaf(dxa, e1.x, dxb * e0.x), my = fmaf(dxa, e1.y, dxb * e0.y),
                  mz = fmaf(dxa, e1.z, dxb * e0.z);
      const float mg = fmaf(u.y, gy, fmaf(g2, mz, fmaf(g1, my, g0 * mx)));
      const float wq = fmaf(kh, fmaf(ramp ? -inv_ramp : 0.f, dp, f), -T);
      const float wr = fmaf(wq, mc, -kh * uz2);
      S[S_R][q] += wr;
      S[S_GR][q] = fmaf(wr, sg, S[S_GR][q]);
      S[S_GM][q] = fmaf(w, mg, S[S_GM][q]);
      e0 = e1;
    }
    h0 = h1;
  }
}

// Pass 1 over the wave's taps, texels read from the image (tiles of 4 or 8
// pixels: the footprint differs between the lanes).
template <bool INTERIOR>
__device__ __forceinline__ void ppb_pass1(const float4* __restrict__ pack, const float4* __restrict__ taps, int k0,
                                          int n_taps, int W, int H, int x, int yb, float R, float inv_ramp,
                                          const PpbPx& px, float (&S)[PPB_SUMS][4]) {
  for (int k = k0; k < n_taps; k += 4) {
    const float4 u = taps[k];
    const TapGeo tg = tap_geo(R, u);
    const FootRows<INTERIOR> rows(W, H, x + tg.ix, yb + tg.iy);
    float4 v0[5], v1[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) rows.texels(pack, j, v0[j], v1[j]);
    ppb_sums<true>(v0, v1, u, tg.ax, tg.ay, R, inv_ramp, px, S);
  }
}

// The same for 16-pixel tiles: the wave stages each of its taps' 17x17
// texels in its own two-buffer LDS ring (see gather_taps_quad), a tap ahead.
template <bool MOVES, bool INTERIOR>
__device__ __forceinline__ void ppb_pass1_staged(float4* stg, const float4* __restrict__ pack,
                                                 const float4* __restrict__ taps, int k0, int n_taps, int W, int H,
                                                 int x0, int y0, int lane, float R, float inv_ramp, const PpbPx& px,
                                                 float (&S)[PPB_SUMS][4]) {
  if (k0 >= n_taps) return;
  StageLane sl;
#pragma unroll
  for (int s = 0; s < PPG_SLOTS; ++s) {
    const int idx = s * 64 + lane < PPG_TEX ? s * 64 + lane : s * 64 + lane - 64;
    sl.sr[s] = idx / PPG_SIDE;
    sl.sc[s] = idx - sl.sr[s] * PPG_SIDE;
    sl.so[s] = (unsigned)(sl.sr[s] * W + sl.sc[s]) * 16u;
    sl.lo[s] = sl.sr[s] * PPG_STRIDE + sl.sc[s];
  }
  sl.last = lane < PPG_TEX - 4 * 64;
  const int lofs = (lane >> 4) * 4 * PPG_STRIDE + (lane & 15);
  float4 u = taps[k0];
  stage_store_texels(stg, stage_load<INTERIOR>(pack, u, R, x0, y0, W, H, sl), sl);
  for (int k = k0, b = 0; k < n_taps; k += 4, b ^= 1) {
    wave_lds_sync();  // tap k's texels stored; tap k - 4's reads done
    const float4 un = taps[min(k + 4, n_taps - 1)];
    const Stage sn = stage_load<INTERIOR>(pack, un, R, x0, y0, W, H, sl);
    const float4* a = stg + b * PPG_TAPSZ + lofs;
    float4 v0[5], v1[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      v0[j] = a[j * PPG_STRIDE];
      v1[j] = a[j * PPG_STRIDE + 1];
    }
    const TapGeo tg = tap_geo(R, u);
    ppb_sums<MOVES>(v0, v1, u, tg.ax, tg.ay, R, inv_ramp, px, S);
    stage_store_texels(stg + (b ^ 1) * PPG_TAPSZ, sn, sl);
    u = un;
  }
}

// Pass 2's weights of one lane's four pixels for the tap with geometry tg
// and distance term d.
template <bool INTERIOR>
__device__ __forceinline__ float4 ppb_weights(const float* __restrict__ coc, int W, int H, int x, int yb,
                                              const TapGeo& tg, float d, float inv_ramp, const PpbPx& px) {
  const FootRows<INTERIOR> rows(W, H, x + tg.ix, yb + tg.iy);
  float h[5], wv[4];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const float2 c = rows.cocs(coc, j);
    h[j] = fmaf(tg.ax, c.y, (1.f - tg.ax) * c.x);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float cq = fmaf(tg.ay, h[q + 1], (1.f - tg.ay) * h[q]);
    const float aq = fabsf(cq), cp = px.c[q];
    const float tk = clamp01((cq - cp) * inv_ramp);
    const float reff = fmaf(-tk, fmaxf(0.f, aq - fabsf(cp)), aq);
    wv[q] = clamp01(fmaf(reff, 0.5f, d)) * __builtin_amdgcn_rcpf(fmaxf(cq * cq, 1.f));
  }
  return make_float4(wv[0], wv[1], wv[2], wv[3]);
}

// a block barrier that orders LDS accesses only (global loads and atomics
// stay in flight)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// lane i's value of lane i - 1 of its row of 16 lanes, 0 in lane 0
__device__ __forceinline__ float row_left(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, true));
}

// Adds one channel of a tile's footprint to the window (w: the lane's texel
// of it): a lane's rows r[0..3] and, in the tile's last rows, r[4], joined
// with the left neighbour's (one rounded sum per tap and texel), and the
// tile's last column.  Lanes of one tile meet in no texel, and a wave's LDS
// accesses run in order; the `nt` tiles of a block take turns (mine: this
// lane's tile's, none above), UNI: one tile.
template <bool UNI>
__device__ __forceinline__ void win_add(float* w, const float (&r)[5], float ax, bool on, bool firstc, bool lastc,
                                        bool lastr, int mine, int nt) {
  float v[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const float left = row_left(r[j]);
    v[j] = fmaf(ax, firstc ? 0.f : left, (1.f - ax) * r[j]);
  }
  for (int t = 0; t < nt; ++t) {
    if (on && (UNI || mine == t)) {
      float a[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] = w[j * PPB_WS];
      if (lastc)
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j * PPB_WS + 1] = fmaf(ax, r[j], w[j * PPB_WS + 1]);
      if (lastr) {
        w[4 * PPB_WS] += v[4];
        if (lastc) w[4 * PPB_WS + 1] = fmaf(ax, r[4], w[4 * PPB_WS + 1]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j * PPB_WS] = a[j] + v[j];
    }
    // (keeps the compiler from moving the next reads, of other lanes'
    // texels, before these writes)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Adds it to the image instead.
__device__ __forceinline__ void image_add(float* __restrict__ gc, const float (&r)[5], int xt, int yt, int W, int H,
                                          float ax, bool on, bool firstc, bool lastc, bool lastr) {
  const unsigned xa = (unsigned)clampi(xt, 0, W - 1), xb = (unsigned)clampi(xt + 1, 0, W - 1);
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    const float left = row_left(r[q]);
    const float t = fmaf(ax, firstc ? 0.f : left, (1.f - ax) * r[q]);
    float* const row = gc + __umul24((unsigned)clampi(yt + q, 0, H - 1), (unsigned)W);
    if (on && (q < 4 || lastr)) {
      if (t != 0.f) atomicAdd(row + xa, t);
      if (lastc && r[q] != 0.f) atomicAdd(row + xb, ax * r[q]);
    }
  }
}

// The same of a wave's whole footprint, 17x17 texels, whose corner is image
// texel (x0, y0): through LDS (foot: the wave's 289 floats), so its rows are
// added in their order.  What the atomics cost is the 64-byte pieces of rows
// they touch: 35 so, 50 with the last column apart.
__device__ __forceinline__ void image_add_foot(float* __restrict__ gc, float* foot, const float (&r)[5], int x0, int y0,
                                               int W, int H, float ax, bool firstc, bool lastc, bool lastr) {
  const int lane = threadIdx.x & 63;
  float* const s = foot + (lane >> 4) * 4 * PPG_SIDE + (lane & 15);
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    const float left = row_left(r[q]);
    const float t = fmaf(ax, firstc ? 0.f : left, (1.f - ax) * r[q]);
    if (q < 4 || lastr) {
      s[q * PPG_SIDE] = t;
      if (lastc) s[q * PPG_SIDE + 1] = ax * r[q];
    }
  }
  // (other lanes' texels are read next, see win_add)
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int t = i * 64 + lane, row = (t * 241) >> 12, col = t - row * PPG_SIDE;  // (t / 17 for t < 320)
    const float v = t < PPG_SIDE * PPG_SIDE ? foot[t] : 0.f;
    float* const gr = gc + __umul24((unsigned)clampi(y0 + row, 0, H - 1), (unsigned)W);
    if (v != 0.f) atomicAdd(gr + clampi(x0 + col, 0, W - 1), v);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Pass 2 of one channel for n <= PPB_G taps: their weights times the pixels'
// kc (and kup of the pixel above the lane's first), joined along the column.
// T16 false (small tiles): a tap that a pixel does not accept takes nothing
// from it, whatever its gradient (0 times infinity).
template <bool UNI, bool T16, class Geo>
__device__ __forceinline__ void ppb_scatter(const float4* wts, int lane, int n, const float (&kc)[4], float kup, int E,
                                            float* win, float* foot, float* __restrict__ gc, int x0, int y0, int W,
                                            int H, bool firstc, bool lastc, bool lastr, int mine, int nt, Geo geo) {
  const int x = x0 + (lane & 15), yb = y0 + (lane >> 4) * 4;
  float4 w4[PPB_G];
  float wu[PPB_G];
#pragma unroll
  for (int j = 0; j < PPB_G; ++j) {
    w4[j] = wts[j * 64 + lane];
    wu[j] = wts[j * 64 + (lane < 16 ? lane : lane - 16)].w;
  }
#pragma unroll
  for (int j = 0; j < PPB_G; ++j) {
    if (j < n) {
      const TapGeo tg = geo(j);
      const auto part = [](float k, float w) { return T16 || w != 0.f ? k * w : 0.f; };
      const float post[4] = {part(kc[0], w4[j].x), part(kc[1], w4[j].y), part(kc[2], w4[j].z), part(kc[3], w4[j].w)};
      const float ay = tg.ay, by = 1.f - ay;
      const float r[5] = {fmaf(by, post[0], ay * part(kup, wu[j])), fmaf(by, post[1], ay * post[0]),
                          fmaf(by, post[2], ay * post[1]), fmaf(by, post[3], ay * post[2]), ay * post[3]};
      const bool in = tg.ix >= -E && tg.ix <= E && tg.iy >= -E && tg.iy <= E;
      if (!UNI || in) win_add<UNI>(win + tg.iy * PPB_WS + tg.ix, r, tg.ax, in, firstc, lastc, lastr, mine, nt);
      if (UNI && !in)
        image_add_foot(gc, foot, r, x0 + tg.ix, y0 + tg.iy, W, H, tg.ax, firstc, lastc, lastr);
      if (!UNI && __builtin_amdgcn_ballot_w64(!in) != 0ull)
        image_add(gc, r, x + tg.ix, yb + tg.iy, W, H, tg.ax, !in, firstc, lastc, lastr);
    }
  }
}

// Adjoint of post-filter + composite.  One block per 16x16 pixels; each of
// its four waves takes every fourth tap of all 256 pixels, a lane four
// vertically adjacent ones (one tile's: tiles are 4, 8 or 16 pixels), whose
// footprints of a tap share 5x2 texels, so a tap's geometry and texels are
// read once per four pixels.  Pass 1: the gather with the sums of its
// derivatives (ppb_sums), joined over the waves in LDS; then one pixel per
// thread: the composite backward, which gives the focus and aperture
// gradients (block partials) and the colour gradient of the pixel itself.
// Pass 2: the colour gradient flowing through the gather weights (recomputed
// from the CoC plane: 48 weights of 256 pixels would take 48 KB of LDS),
// transposed to the texels of every tap: the lanes' posts are joined to the
// tile's footprint in registers and added to the block's LDS window if the
// tap's offset lies in it (up to PPB_WIN_E, or PPB_FAR_E where some lie
// beyond; flushed once with global atomics; window
// texels are image texels clamped to the edge, as in the gather), or to the
// image.  Of PPB_G taps at a time three waves add a channel each to the
// window, without barriers between the taps, and the fourth forms two of
// the weights, the others one each.  (LDS float atomics would let every wave add to all channels,
// but take 190 clocks each: 4.1 ms for the 1080p image below; four waves'
// channels in turns with a barrier each: 0.74.)
// Bound at 1080p, 48 taps, 16-pixel tiles: vector arithmetic (65 %), the rest
// waiting for LDS and, on the quarter of the tiles with R of 46, for global
// atomics (0.14 ms): 0.92 -> 0.68 ms.  With most tiles beyond the window
// (the 1080p interior) the atomics bound it: 1.35 -> 1.27 ms, 1.51 with the
// footprint's last column apart; all blocks at the same group of taps cost
// 2 % more.  1708x923 with 4-pixel tiles, whose
// radii differ within a block: 5.0 -> 1.8 ms, of it 1.5 the tiles' turns.
// The window's limit: a third block per CU fits up to 20 (24: 0.2 ms slower).
// Groups of 5 taps leave the smaller window 19; of 6, 17: 1 to 3 % slower.
struct PpbArgs {
  const float4* pack;
  const float *coc, *rad;
  const int* rad_arg;
  const float4* taps;
  int n_taps, W, H, tile;
  float inv_ramp;
  LensK l;
  float spx;
  const uint8_t* spp;
  const float *cn, *cf, *hr;
  float inv_ht;
  int rt_override;
  const float* g;
  float* gcol;
  float2* partial;
};

struct PpbLds {
  // the waves' rings of staged texels, then their sums, then the window and
  // behind it two buffers of the weights of a group of taps
  static constexpr int WIN = 3 * PPB_PLANE, WTS = 2 * PPB_G * 256, SUMS = 4 * PPB_SUMS * 256,
                       RING = 4 * 2 * 4 * PPG_TAPSZ;
  static constexpr int MAX1 = SUMS > RING ? SUMS : RING;
  float buf[WIN + WTS > MAX1 ? WIN + WTS : MAX1];
  float2 red[4];
};

// The tile of pixel (x, y), -1 where there is none (tile: a power of two).
__device__ __forceinline__ int ppb_tile(const PpbArgs& A, int x, int y) {
  const int sh = 31 - __clz(A.tile), TW = (A.W + A.tile - 1) >> sh;
  return (x >> sh) < TW && (y >> sh) < (A.H + A.tile - 1) >> sh ? (y >> sh) * TW + (x >> sh) : -1;
}

// One block.  UNI: one radius R for all its pixels (a tile of 16 pixels, or
// smaller tiles of equal radius): the taps' geometry is the wave's, their
// texels are staged and the footprint is one of 16x16 pixels.
template <bool UNI, bool T16>
__device__ __forceinline__ void ppb_block(const PpbArgs& A, PpbLds& lds, int blk, float R) {
  const float4* __restrict__ pack = A.pack;
  const float* __restrict__ coc = A.coc;
  const float4* __restrict__ taps = A.taps;
  const float* __restrict__ g = A.g;
  float* __restrict__ gcol = A.gcol;
  const int n_taps = A.n_taps, W = A.W, H = A.H, tile = A.tile;
  const float inv_ramp = A.inv_ramp;
  const LensK& l = A.l;
  float* const buf = lds.buf;
  float4 (*const wts)[PPB_G * 64] = (float4 (*)[PPB_G * 64])(buf + PpbLds::WIN);
  float2* const red = lds.red;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int TWb = (W + 15) >> 4;
  const int x0 = (blk % TWb) * 16, y0 = (blk / TWb) * 16;
  const int lx = lane & 15, ly = (lane >> 4) * 4;
  const int x = x0 + lx, yb = y0 + ly;
  const size_t N = (size_t)W * H;
  const float dcs = -l.A * A.spx * l.invS1 * l.invS1;    // dc/dS1 (every pixel)
  const float inv_A = l.A > 0.0f ? 1.0f / l.A : 0.0f;  // unit CoC = c / A
  // the radius' derivatives through the pixel that sets it
  const int ti = ppb_tile(A, x, yb), m = ti >= 0 ? A.rad_arg[ti] : -1;
  float Rs = 0.f, Ra = 0.f;
  if (m >= 0) {
    const float cm = pack[m].w, sg = cm >= 0.f ? 0.5f : -0.5f;
    Rs = sg * dcs;
    Ra = sg * cm * inv_A;
  }
  const bool some = __builtin_amdgcn_ballot_w64(R > 0.f) != 0ull;
  float Rm = R;
  if (!UNI)
    for (int o = 32; o > 0; o >>= 1) Rm = fmaxf(Rm, __shfl_xor(Rm, o));
  const int ER = __builtin_amdgcn_readfirstlane((int)ceilf(Rm));
  const bool interior = x0 - ER - 1 >= 0 && x0 + 16 + ER < W && y0 - ER - 1 >= 0 && y0 + 16 + ER < H &&
                        (long long)W * H * 16 < (1ll << 31);
  const bool moves = __builtin_amdgcn_ballot_w64(Rs != 0.f || Ra != 0.f) != 0ull;
  PpbPx px;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bool ok = x < W && yb + q < H;
    const size_t p = ok ? (size_t)(yb + q) * W + x : 0;
    const float4 t = pack[p];
    px.c[q] = ok ? t.w : 0.f;
#pragma unroll
    for (int c = 0; c < 3; ++c) px.g[c][q] = ok ? g[c * N + p] : 0.f;
    px.gc[q] = fmaf(px.g[2][q], t.z, fmaf(px.g[1][q], t.y, px.g[0][q] * t.x));
  }
  float S[PPB_SUMS][4] = {};
  if (some) {
    if (UNI) {
      float4* const stg = (float4*)buf + wave * 2 * PPG_TAPSZ;
      if (moves && interior)
        ppb_pass1_staged<true, true>(stg, pack, taps, wave, n_taps, W, H, x0, y0, lane, R, inv_ramp, px, S);
      else if (moves)
        ppb_pass1_staged<true, false>(stg, pack, taps, wave, n_taps, W, H, x0, y0, lane, R, inv_ramp, px, S);
      else
        ppb_pass1_staged<false, false>(stg, pack, taps, wave, n_taps, W, H, x0, y0, lane, R, inv_ramp, px, S);
      __syncthreads();  // the ring's space takes the sums
    } else if (interior) {
      ppb_pass1<true>(pack, taps, wave, n_taps, W, H, x, yb, R, inv_ramp, px, S);
    } else {
      ppb_pass1<false>(pack, taps, wave, n_taps, W, H, x, yb, R, inv_ramp, px, S);
    }
  }
#pragma unroll
  for (int i = 0; i < PPB_SUMS; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) buf[(wave * PPB_SUMS + i) * 256 + q * 64 + lane] = S[i][q];
  __syncthreads();
  // one pixel per thread: row `wave` of its lane's four
  float gs = 0.f, ga = 0.f, own[3] = {0.f, 0.f, 0.f}, gpp[3] = {0.f, 0.f, 0.f};
  const int y = yb + wave;
  const bool inside = x < W && y < H;
  const size_t p = inside ? (size_t)y * W + x : 0;
  const bool traced = inside && A.spp[p] > 0;
  if (inside && !(A.rt_override && traced)) {
    float s[PPB_SUMS];
#pragma unroll
    for (int i = 0; i < PPB_SUMS; ++i) {
      s[i] = 0.f;
#pragma unroll
      for (int v = 0; v < 4; ++v) s[i] += buf[(v * PPB_SUMS + i) * 256 + tid];
    }
    const float4 cp4 = pack[p];
    const D3 cpv = dk(cp4.w, dcs, cp4.w * inv_A);
    // composite weights
    const D3 phi = dclamp(dabs(cpv) - dc(HDOF_SQRT2), 0.f, 1.f);
    const D3 nu = dclamp(dc(0.5f) - 0.35355339059327376f * cpv, 0.f, 1.f);
    const float h = A.hr[p];
    const float rho = traced ? 1.0f : 0.0f;
    const float beta = traced ? clamp01(1.0f - h * A.inv_ht) : 0.0f;
    const D3 acoef = rho * nu + beta * (dc(1.f) - nu);
    const D3 bcoef = (1.f - rho) * nu + (1.f - beta) * (dc(1.f) - nu);
    // the filtered colour, projected on the incoming gradient
    const float gq[3] = {g[p], g[N + p], g[2 * N + p]};
    const float cr[3] = {cp4.x, cp4.y, cp4.z};
    const float gcr = fmaf(gq[2], cr[2], fmaf(gq[1], cr[1], gq[0] * cr[0]));  // (as px.gc)
    float gct = 0.f;
    for (int c = 0; c < 3; ++c) {
      gct = fmaf(gq[c], h * A.cn[c * N + p] + (1.f - h) * A.cf[c * N + p], gct);
    }
    const D3 cp1 = dmaxc(dabs(cpv), 1.f);
    const D3 w0 = dquot(dc(1.f), cp1 * cp1);
    const float area = R * R / (float)n_taps, i2R = R > 0.f ? 2.f / R : 0.f;
    const float dr = fmaf(i2R, s[S_W], s[S_R]), gr = fmaf(i2R, s[S_GW], s[S_GR] + s[S_GM]);
    const D3 den = w0 + area * dk(s[S_W], fmaf(dcs, s[S_C], Rs * dr), fmaf(inv_A, s[S_A], Ra * dr));
    const D3 num = area * dk(s[S_GW], fmaf(dcs, s[S_GC], Rs * gr), fmaf(inv_A, s[S_GA], Ra * gr));
    const D3 oof = gct * acoef + bcoef * (dc(gcr) + dquot(num, den));
    const D3 out = gcr * (dc(1.f) - phi) + phi * oof;
    gs = out.s;
    ga = out.a;
    const float iden = phi.v * bcoef.v / den.v;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      gpp[c] = gq[c] * iden;
      own[c] = fmaf(gq[c], 1.f - phi.v, gpp[c] * w0.v);
      gpp[c] *= area;
    }
  }
  // the window: texel (r, s) of a channel is image texel (y0 - E + r, x0 - E + s)
  // (UNI: a window of E > PPB_FAR_E has room for every tap, with one texel for
  // the offsets' rounding)
  const bool far = ER >= PPB_WIN_E;
  const int E = UNI && far ? PPB_FAR_E : min(PPB_WIN_E, ER + 1), wd = 17 + 2 * E;
  constexpr int PL = PPB_PLANE;  // a channel's plane
  float* const gp = (float*)wts;
  __syncthreads();  // all sums read
#pragma unroll
  for (int c = 0; c < 3; ++c) gp[c * 256 + tid] = gpp[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c)
    for (int i = tid; i < wd * (PPB_WS / 4); i += 256) ((float4*)(buf + c * PL))[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  // the pixels' gpp of the wave's channel, and of the one above them (0 if
  // that is another footprint's)
  float kc[4];
  const float kup = (ly & ((UNI ? 16 : tile) - 1)) == 0 ? 0.f : gp[(wave < 3 ? wave : 0) * 256 + 3 * 64 + lane - 16];
  bool scat = false;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    kc[q] = gp[(wave < 3 ? wave : 0) * 256 + q * 64 + lane];
    scat |= gp[q * 64 + lane] != 0.f || gp[256 + q * 64 + lane] != 0.f || gp[512 + q * 64 + lane] != 0.f;
  }
  scat = __builtin_amdgcn_ballot_w64(scat) != 0ull;
  lds_barrier();
#pragma unroll
  for (int c = 0; c < 3; ++c) buf[c * PL + (ly + wave + E) * PPB_WS + lx + E] = own[c];
  lds_barrier();
  // pass 2: the weights again (value only) and the transpose of gpp * weight
  if (some && scat) {
    const int tl = UNI ? 16 : tile, all = (16 / tl) * (16 / tl);
    const bool firstc = (lx & (tl - 1)) == 0, lastc = (lx & (tl - 1)) == tl - 1;
    const bool lastr = (ly & (tl - 1)) == tl - 4;
    // turns for the tiles that have a gradient in the wave's channel: of a
    // sparse one few have (one pixel in 1517 of 1280x720, 4-pixel tiles: 456
    // us with a turn for each, 207 so)
    int mine = (ly / tl) * (16 / tl) + lx / tl, nt = 1;
    if (!UNI) {
      const bool any = kc[0] != 0.f || kc[1] != 0.f || kc[2] != 0.f || kc[3] != 0.f;
      unsigned turns = 0;
      for (int t = 0; t < all; ++t) turns |= __builtin_amdgcn_ballot_w64(any && mine == t) != 0ull ? 1u << t : 0u;
      mine = turns >> mine & 1 ? __popc(turns & ((1u << mine) - 1u)) : all;
      nt = __popc(turns);
    }
    float* const win = buf + wave * PL + (ly + E) * PPB_WS + lx + E;
    float* const gc = gcol + wave * N;
    // blocks with taps outside the window start at different groups of taps:
    // their atomics land on different texels at a time
    const int ng = (n_taps + PPB_G - 1) / PPB_G, rot = far ? (blk * 17) % ng : 0;
    float* const foot = buf + wave * PL + (17 + 2 * PPB_FAR_E) * PPB_WS;
    // (UNI) lane i keeps the geometry and distance term of tap kl + i
    TapGeo lg{0, 0, 0.f, 0.f};
    float ld = 0.f;
    for (int i = 0, kl = -64; i < ng; ++i) {
      const int k0 = PPB_G * (i + rot < ng ? i + rot : i + rot - ng), b = i & 1;
      if (UNI && (k0 < kl || k0 + PPB_G > kl + 64)) {
        kl = k0;
        const float4 u = taps[min(k0 + lane, n_taps - 1)];
        lg = tap_geo(R, u);
        ld = fmaf(-R, u.z, 0.5f);
      }
      const auto geo = [&](int j) {
        if (!UNI) return tap_geo(R, taps[k0 + j]);
        const int e = k0 - kl + j;
        return TapGeo{__builtin_amdgcn_readlane(lg.ix, e), __builtin_amdgcn_readlane(lg.iy, e),
                      __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lg.ax), e)),
                      __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lg.ay), e))};
      };
      // the fourth wave, which has no channel, forms the weights that are left
      const int n = min(PPB_G, n_taps - k0), j1 = wave < 3 ? wave + 1 : PPB_G;
      for (int j = wave; j < j1 && j < n; ++j) {
        const float d = UNI ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ld), k0 - kl + j))
                            : fmaf(-R, taps[k0 + j].z, 0.5f);
        const TapGeo tg = geo(j);
        wts[b][j * 64 + lane] = interior ? ppb_weights<true>(coc, W, H, x, yb, tg, d, inv_ramp, px)
                                         : ppb_weights<false>(coc, W, H, x, yb, tg, d, inv_ramp, px);
      }
      lds_barrier();
      if (wave < 3)
        ppb_scatter<UNI, T16>(wts[b], lane, n, kc, kup, E, win, foot, gc, x0, y0, W, H, firstc, lastc, lastr, mine, nt, geo);
    }
  }
  __syncthreads();
  {  // (a window row is no longer than a wave)
    const int gx = clampi(x0 - E + lane, 0, W - 1);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll 4
      for (int r = wave; r < wd; r += 4) {
        const float v = lane < wd ? buf[c * PL + r * PPB_WS + lane] : 0.f;
        if (v != 0.f) atomicAdd(gcol + c * N + (size_t)clampi(y0 - E + r, 0, H - 1) * W + gx, v);
      }
  }
  for (int o = 32; o > 0; o >>= 1) {
    gs += __shfl_xor(gs, o);
    ga += __shfl_xor(ga, o);
  }
  if (lane == 0) red[wave] = make_float2(gs, ga);
  __syncthreads();
  if (tid == 0)
    A.partial[blockIdx.x] = make_float2((red[0].x + red[1].x) + (red[2].x + red[3].x),
                                      (red[0].y + red[1].y) + (red[2].y + red[3].y));
}

template <bool T16>
__global__ __launch_bounds__(256, PPB_MINW) void k_ppc_backward(PpbArgs A) {
  __shared__ __attribute__((aligned(16))) PpbLds lds;
  const int TWb = (A.W + 15) >> 4, blk = xcd_block(blockIdx.x, TWb * ((A.H + 15) >> 4));
  if (T16) {
    ppb_block<true, true>(A, lds, blk, A.rad[blk]);
    return;
  }
  // lanes of a tile that lies partly outside the image have its radius too
  // (they carry the inner ones' last texels in pass 2); those of no tile, the
  // first lane's
  const int lane = threadIdx.x & 63;
  const int ti = ppb_tile(A, (blk % TWb) * 16 + (lane & 15), (blk / TWb) * 16 + (lane >> 4) * 4);
  float R = ti >= 0 ? A.rad[ti] : 0.f;
  const float R0 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(R)));
  if (ti < 0) R = R0;
  if (__builtin_amdgcn_ballot_w64(R != R0) == 0ull)
    ppb_block<true, false>(A, lds, blk, R0);
  else
    ppb_block<false, false>(A, lds, blk, R);
}

// block partials summed in a fixed order (deterministic), in double
__global__ void k_sum_partials(const float2* __restrict__ partial, int n, float* __restrict__ out) {
  __shared__ double sx[256], sy[256];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    a += partial[i].x;
    b += partial[i].y;
  }
  sx[threadIdx.x] = a;
  sy[threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sx[threadIdx.x] += sx[threadIdx.x + o];
      sy[threadIdx.x] += sy[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = (float)sx[0];
    out[1] = (float)sy[0];
  }
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

}  // namespace

hdof_status postfilter_reserve(hdof_ctx* ctx, const CamK& k, const LensK& l, const hdof_pp_params& pp,
                               hipStream_t st) {
  const int t = pp.tile;
  const size_t N = (size_t)k.W * k.H, NT = (size_t)cdiv(k.W, t) * cdiv(k.H, t);
  hdof_status s;
  if ((s = hdof_ensure(ctx->pp_pack, sizeof(float4) * N)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->pp_tile, sizeof(float) * NT)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->pp_rad, sizeof(float) * NT)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->pp_taps, sizeof(float4) * 256)) != HDOF_OK) return s;
  pp_taps_ensure(ctx, pp.n_taps, l, st);
  return HDOF_OK;
}

namespace {

// where one post-filter call keeps its intermediates
struct PPScratch {
  float4* pack;   // packed texels (rgb, signed CoC), one per pixel
  float* tile;    // per-tile maximum CoC radius
  float* rad;     // dilated tile radius (tiles other than 16 px)
  float4* taps;   // tap table, 256 entries
};

hdof_status postfilter_run(hdof_ctx* ctx, const PPScratch& S, const float* color, const float* depth,
                           const CamK& k, const LensK& l, const hdof_pp_params& pp, float* out, hipStream_t st,
                           bool packed, const PostFuse* fuse) {
  const int W = k.W, H = k.H, t = pp.tile;
  const int TW = cdiv(W, t), TH = cdiv(H, t);
  const int K = (int)ceil((double)pp.r_cap / t);
  if (!packed)
    hipLaunchKernelGGL(k_pp_pack, dim3(cdiv(W, 16) * cdiv(H, 16)), dim3(256), 0, st, color, depth, k, l, t,
                       S.pack, S.tile);
  if (t != 16)
    hipLaunchKernelGGL(k_pp_dilate<false>, dim3(cdiv(TW, DIL_W), cdiv(TH, DIL_H)), dim3(256), 0, st,
                       (const float*)S.tile, (const int*)nullptr, TW, TH, K, pp.r_cap, S.rad, (int*)nullptr);
  hdof_prof_mark(ctx, 8, st);
  if (t == 16) {
    // The quad form (a wave per tile, blocks of four) rises in steps of four
    // tiles per CU, the four-wave form evenly: it is the faster one below
    // 11 tiles per CU and on the first half of the next step, 12 to 14
    // (filter alone, quad / four-wave form, us: 333x187, 1 tile per CU,
    // 46 / 21; 853x479, 6.3, 63 / 52; 1120x640, 10.9, 71 / 68; 1024x720, 11.3,
    // 71 / 73; 1024x768, 12.0, 71 / 74; 1040x768, 12.2, 84 / 77; 1136x800,
    // 13.9, 84 / 83; 1280x720, 14.1, 84 / 87; 1024x1024, 16, 84 / 95; 1600x900,
    // 22.3, 130 / 135; 1080p, 31.9, 157 / 178).
    const int nt = TW * TH, cu = ctx->n_cu;
    const bool sa = l.sa != 0.0f, few = nt < 11 * cu || (nt > 12 * cu && nt < 14 * cu);
    FuseK fz{};
    if (fuse && fuse->untraced_only) {
      fz.out = fuse->out;
      // beside the trace (the overlapped frame) the four-wave form: the quad
      // form finishes sooner but takes the trace's issue slots on the way
      auto kern = sa ? k_pp_gather16<2, true> : k_pp_gather16<2, false>;
      if (fuse->done)
        hipExtLaunchKernelGGL(kern, dim3(TW * TH), dim3(256), 0, st, nullptr, fuse->done, 0,
                              (const float4*)S.pack, (const float*)S.tile, K, pp.r_cap, (const float4*)S.taps,
                              pp.n_taps, W, H, 1.0f / pp.bg_ramp_px, out, fz);
      else
        hipLaunchKernelGGL(kern, dim3(TW * TH), dim3(256), 0, st, (const float4*)S.pack,
                           (const float*)S.tile, K, pp.r_cap, (const float4*)S.taps, pp.n_taps, W, H,
                           1.0f / pp.bg_ramp_px, out, fz);
    } else if (fuse) {
      fz = FuseK{fuse->spp, fuse->rt.c_near, fuse->rt.c_far, fuse->rt.hit_ratio, 1.0f / fuse->cp.h_t,
                 fuse->cp.rt_override, fuse->out, fuse->pps,
                 fuse->pps && fuse->cp.spec_y > 0.0f ? 1.0f / fuse->cp.spec_y : 0.0f};
      auto kern = few ? (sa ? k_pp_gather16<1, true> : k_pp_gather16<1, false>)
                      : (sa ? k_pp_gather16q<1, true> : k_pp_gather16q<1, false>);
      hipLaunchKernelGGL(kern, dim3(few ? TW * TH : (TW * TH + 3) / 4), dim3(256), 0, st, (const float4*)S.pack,
                         (const float*)S.tile, K, pp.r_cap, (const float4*)S.taps, pp.n_taps, W, H,
                         1.0f / pp.bg_ramp_px, out, fz);
    } else {
      auto kern = few ? (sa ? k_pp_gather16<0, true> : k_pp_gather16<0, false>)
                      : (sa ? k_pp_gather16q<0, true> : k_pp_gather16q<0, false>);
      hipLaunchKernelGGL(kern, dim3(few ? TW * TH : (TW * TH + 3) / 4), dim3(256), 0, st, (const float4*)S.pack,
                         (const float*)S.tile, K, pp.r_cap, (const float4*)S.taps, pp.n_taps, W, H,
                         1.0f / pp.bg_ramp_px, out, fz);
    }
  } else {
    hipLaunchKernelGGL(k_pp_gather_any, dim3(cdiv(W, 16), cdiv(H, 16)), dim3(256), 0, st, (const float4*)S.pack,
                       (const float*)S.rad, (const float4*)S.taps, pp.n_taps, W, H, t, 1.0f / pp.bg_ramp_px, out);
    if (fuse && !fuse->untraced_only) {
      HDOF_HIP(hipGetLastError());
      return launch_composite(ctx, color, out, depth, fuse->spp, fuse->rt, k, l, fuse->cp, fuse->out, st,
                              fuse->pps);
    }
  }
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

}  // namespace

hdof_status launch_postfilter(hdof_ctx* ctx, const float* color, const float* depth, const CamK& k,
                              const LensK& l, const hdof_pp_params& pp, float* out, hipStream_t st, bool packed,
                              const PostFuse* fuse) {
  hdof_status s;
  if ((s = postfilter_reserve(ctx, k, l, pp, st)) != HDOF_OK) return s;
  const PPScratch S{(float4*)ctx->pp_pack.p, (float*)ctx->pp_tile.p, (float*)ctx->pp_rad.p, (float4*)ctx->pp_taps.p};
  return postfilter_run(ctx, S, color, depth, k, l, pp, out, st, packed, fuse);
}

hdof_status launch_postfilter_batched(hdof_ctx* ctx, const float4* pack, const float* tile_r, int n_views,
                                      const BatchView* hviews, const void* views_dev, float* const* outs,
                                      const hdof_pp_params& pp, float* pp_out, hipStream_t st) {
  if (pp.tile != 16) return hdof_set_error(HDOF_ERR_INVALID_ARG, "batched gather: 16-pixel tiles only");
  PPBatch b{};
  b.n = n_views;
  const bool sa = hviews[0].l.sa != 0.0f;
  for (int v = 0; v < n_views; ++v) {
    if ((hviews[v].l.sa != 0.0f) != sa)
      return hdof_set_error(HDOF_ERR_UNSUPPORTED, "batched gather: one spherical aberration for every view");
    b.tile_base[v + 1] = b.tile_base[v] + cdiv(hviews[v].k.W, 16) * cdiv(hviews[v].k.H, 16);
    b.out[v] = outs[v];
  }
  const int K = (int)ceil((double)pp.r_cap / 16);
  auto kern = sa ? k_pp_gather16q_batch<true> : k_pp_gather16q_batch<false>;
  hipLaunchKernelGGL(kern, dim3((b.tile_base[n_views] + 3) / 4), dim3(256), 0, st, pack, tile_r, K, pp.r_cap,
                     (const float4*)ctx->pp_taps.p, pp.n_taps, 1.0f / pp.bg_ramp_px, pp_out,
                     (const BatchView*)views_dev, b);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

hdof_status launch_composite_traced_batched(hdof_ctx* ctx, const float* color, const float* pp, const float* depth,
                                            const uint8_t* spp, hdof_rt_bufs rt, int n_views,
                                            const BatchView* hviews, const void* views_dev, float* const* outs,
                                            const hdof_composite_params& cp, hipStream_t st) {
  (void)ctx;
  PPBatch b{};
  b.n = n_views;
  for (int v = 0; v < n_views; ++v) {
    b.blk_base[v + 1] = b.blk_base[v] + cdiv(hviews[v].k.W * hviews[v].k.H, HDOF_BATCH_PX_BLOCK);
    b.out[v] = outs[v];
  }
  const CompK a{color, pp, depth, spp, rt.c_near, rt.c_far, rt.hit_ratio, hviews[0].l, 0, 1.0f / cp.h_t,
                cp.rt_override, nullptr, 0.0f, nullptr};
  hipLaunchKernelGGL(k_composite_traced_batch, dim3(b.blk_base[n_views]), dim3(256), 0, st, a,
                     (const BatchView*)views_dev, b);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

// ---------------------------------------------------------------------------
// The post-filter without allocation: its intermediates live in `scratch`,
// one file-scope device array per device (tap table, tile radii, dilated
// tile radii, packed texels), sized for images of up to
// HDOF_POSTFILTER_NOALLOC_MAX_PX pixels.  In host code `scratch` names a
// host-side stand-in, never device memory: kernels get the address that
// hipGetSymbolAddress returns for the current device, looked up once per
// device when the library's first context on it is created.
// ---------------------------------------------------------------------------
namespace {
constexpr size_t NA_TAPS_BYTES = 256 * sizeof(float4);
// tile radii at the smallest tile (4 px) of any W x H <= the maximum with
// W, H <= 16384: ceil(W/4) ceil(H/4) <= N/16 + (W + H)/4 + 1
constexpr size_t NA_TILES = (size_t)HDOF_POSTFILTER_NOALLOC_MAX_PX / 16 + 8193;
constexpr size_t NA_TILE_BYTES = (NA_TILES * sizeof(float) + 255) / 256 * 256;
constexpr size_t NA_BYTES = NA_TAPS_BYTES + 2 * NA_TILE_BYTES + sizeof(float4) * (size_t)HDOF_POSTFILTER_NOALLOC_MAX_PX;
static_assert(NA_BYTES == (size_t)HDOF_POSTFILTER_NOALLOC_BYTES, "header size of the no-alloc scratch");
constexpr int NA_MAX_DEVICES = 64;

std::mutex na_mu;
void* na_ptr[NA_MAX_DEVICES] = {};
}  // namespace

static __device__ __align__(256) unsigned char scratch[NA_BYTES];

hdof_status postfilter_noalloc_init(int device, void** out) {
  *out = nullptr;
  if (device < 0 || device >= NA_MAX_DEVICES)
    return hdof_set_error(HDOF_ERR_UNSUPPORTED, "device %d beyond the %d the library tracks", device, NA_MAX_DEVICES);
  std::lock_guard<std::mutex> lock(na_mu);
  if (!na_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return hdof_set_error(HDOF_ERR_HIP, "no-alloc scratch address on device %d: %s", device, hipGetErrorString(e));
    na_ptr[device] = p;
  }
  *out = na_ptr[device];
  return HDOF_OK;
}

hdof_status launch_postfilter_noalloc(hdof_ctx* ctx, const float* color, const float* depth, const CamK& k,
                                      const LensK& l, const hdof_pp_params& pp, float* out, hipStream_t st) {
  if ((size_t)k.W * (size_t)k.H > (size_t)HDOF_POSTFILTER_NOALLOC_MAX_PX)
    return hdof_set_error(HDOF_ERR_CAPACITY, "%dx%d exceeds the no-alloc post-filter's %d pixels", k.W, k.H,
                          HDOF_POSTFILTER_NOALLOC_MAX_PX);
  unsigned char* base = (unsigned char*)ctx->noalloc_scratch;
  if (!base) return hdof_set_error(HDOF_ERR_UNSUPPORTED, "the context holds no no-alloc scratch");
  const PPScratch S{(float4*)(base + NA_TAPS_BYTES + 2 * NA_TILE_BYTES), (float*)(base + NA_TAPS_BYTES),
                    (float*)(base + NA_TAPS_BYTES + NA_TILE_BYTES), (float4*)base};
  // the tap table is rebuilt every call: the array keeps whatever the last
  // call on this device left in it
  const int blades = l.blades >= 3 ? l.blades : 0;
  hipLaunchKernelGGL(k_pp_taps, dim3(1), dim3(256), 0, st, pp.n_taps, blades,
                     (double)l.rot_ht * 3.14159265358979323846, l.sa, S.taps);
  return postfilter_run(ctx, S, color, depth, k, l, pp, out, st, false, nullptr);
}

hdof_status launch_composite(hdof_ctx* ctx, const float* color, const float* pp, const float* depth,
                             const uint8_t* spp, hdof_rt_bufs rt, const CamK& k, const LensK& l,
                             const hdof_composite_params& cp, float* out, hipStream_t st, const float* pps,
                             bool sparse) {
  (void)ctx;
  const int N = k.W * k.H;
  const float inv_sy = pps && cp.spec_y > 0.0f ? 1.0f / cp.spec_y : 0.0f;
  const CompK a{color, pp, depth, spp, rt.c_near, rt.c_far, rt.hit_ratio, l, N, 1.0f / cp.h_t, cp.rt_override,
                pps, inv_sy, out};
  if (sparse)
    hipLaunchKernelGGL(k_composite_traced, dim3(cdiv(N, 256)), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(k_composite, dim3(cdiv(N, 256)), dim3(256), 0, st, a);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

hdof_status launch_pp_spec(hdof_ctx* ctx, const float* ys, const uint8_t* spp, const CamK& k, const LensK& l,
                           const hdof_pp_params& pp, float* out, hipStream_t st) {
  const int W = k.W, H = k.H, t = pp.tile;
  const int K = (int)ceil((double)pp.r_cap / t);
  if (!ctx->pp_pack.p || !ctx->pp_tile.p || (t != 16 && !ctx->pp_rad.p))
    return hdof_set_error(HDOF_ERR_INVALID_ARG, "specular post-filter before the frame's post-filter preparation");
  hdof_status s;
  if ((s = hdof_ensure(ctx->pp_taps, sizeof(float4) * 256)) != HDOF_OK) return s;
  pp_taps_ensure(ctx, pp.n_taps, l, st);
  hipLaunchKernelGGL(k_pp_spec, dim3(cdiv(W, 8) * cdiv(H, 8)), dim3(256), 0, st, (const float4*)ctx->pp_pack.p, ys,
                     spp, (const float*)ctx->pp_tile.p, (const float*)ctx->pp_rad.p, t, K, pp.r_cap,
                     (const float4*)ctx->pp_taps.p, pp.n_taps, W, H, 1.0f / pp.bg_ramp_px, out);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}

hdof_status launch_ppc_backward(hdof_ctx* ctx, const float* color, const float* depth, const uint8_t* spp,
                                hdof_rt_bufs rt, const CamK& k, const LensK& l, const hdof_pp_params& pp,
                                const hdof_composite_params& cp, const float* grad_out, float* grad_color,
                                float* grad_lens, hipStream_t st) {
  const int W = k.W, H = k.H, t = pp.tile;
  const size_t N = (size_t)W * H;
  const int TW = cdiv(W, t), TH = cdiv(H, t);
  const int K = (int)ceil((double)pp.r_cap / t);
  const dim3 grid(cdiv(W, 16), cdiv(H, 16));
  const int nblk = (int)(grid.x * grid.y);
  hdof_status s;
  if ((s = hdof_ensure(ctx->pp_pack, sizeof(float4) * N)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->pp_tile, sizeof(float) * (size_t)TW * TH)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->pp_rad, sizeof(float) * (size_t)TW * TH)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->pp_taps, sizeof(float4) * 256)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->ppb_coc, sizeof(float) * N)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->ppb_args, sizeof(int) * 2 * (size_t)TW * TH)) != HDOF_OK) return s;
  if ((s = hdof_ensure(ctx->ppb_partial, sizeof(float2) * (size_t)nblk)) != HDOF_OK) return s;
  pp_taps_ensure(ctx, pp.n_taps, l, st);
  int* tile_arg = (int*)ctx->ppb_args.p;
  int* rad_arg = tile_arg + (size_t)TW * TH;
  hipLaunchKernelGGL(k_ppb_pack, dim3(nblk), dim3(256), 0, st, color, depth, k, l, t, (float4*)ctx->pp_pack.p,
                     (float*)ctx->ppb_coc.p, (float*)ctx->pp_tile.p, tile_arg);
  hipLaunchKernelGGL(k_pp_dilate<true>, dim3(cdiv(TW, DIL_W), cdiv(TH, DIL_H)), dim3(256), 0, st,
                     (const float*)ctx->pp_tile.p, (const int*)tile_arg, TW, TH, K, pp.r_cap, (float*)ctx->pp_rad.p, rad_arg);
  hipLaunchKernelGGL(k_fill_f, dim3(cdiv(3 * (long)N, 256)), dim3(256), 0, st, grad_color, 3 * N, 0.0f);
  const PpbArgs A{(const float4*)ctx->pp_pack.p, (const float*)ctx->ppb_coc.p, (const float*)ctx->pp_rad.p, rad_arg,
                  (const float4*)ctx->pp_taps.p, pp.n_taps, W, H, t, 1.0f / pp.bg_ramp_px, l, k.spx, spp, rt.c_near,
                  rt.c_far, rt.hit_ratio, 1.0f / cp.h_t, cp.rt_override, grad_out, grad_color,
                  (float2*)ctx->ppb_partial.p};
  if (t == 16)
    hipLaunchKernelGGL(k_ppc_backward<true>, dim3(nblk), dim3(256), 0, st, A);
  else
    hipLaunchKernelGGL(k_ppc_backward<false>, dim3(nblk), dim3(256), 0, st, A);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, st, (const float2*)ctx->ppb_partial.p, nblk,
                     grad_lens);
  HDOF_HIP(hipGetLastError());
  return HDOF_OK;
}
