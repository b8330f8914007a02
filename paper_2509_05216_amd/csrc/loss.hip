// Training loss: mean over views of (1 - lambda) L1 + lambda (1 - SSIM), and its
// gradient with respect to the rendered image.
//
// SSIM uses an 11 x 11 Gaussian window (sigma 1.5, separable, weights summing
// to one), C1 = 0.01^2, C2 = 0.03^2, zero padding, averaged over pixels and
// channels.  Two LDS-tiled passes per view and channel (32 x 32 output pixels
// at a time, in 42 x 42 windows): the first forms the five local moments by separable filtering and writes, per pixel, the partials
// g1 = dS/dmu_x, g2 = dS/dE[x^2] and g3 = dS/dE[xy]; the second filters those
// maps (the window is symmetric, so the zero-padded correlation is its own
// adjoint) and combines them with the L1 term:
//   dL/dx = s [(1 - lambda) sign(x - y) - lambda (w*g1 + 2 x w*g2 + y w*g3)],
//   s = 1/(3 H W V).
// A horizontal task makes four outputs of one halo row from 14 inputs (read
// 8 bytes at a time, with x^2, y^2 and x y formed once per input), each tap an
// explicit fused multiply-add per moment.  In the vertical pass each thread
// produces four consecutive rows of one column from 14 LDS rows.  Loss sums are reduced per block into
// float64 partials and summed by a final single-block kernel, so the loss
// value is deterministic.
#include <algorithm>
#include <atomic>

#include "internal.h"

namespace isogs {
namespace {

constexpr int kT = 32;           // output tile side
constexpr int kR = 5;            // window radius
constexpr int kN = 2 * kR + 1;   // taps
constexpr int kH = kT + 2 * kR;  // 42: halo tile side (LDS rows of 168 bytes, 8-byte aligned)
constexpr int kC = 2 * kR;       // 10: filtered rows that a tile shares with the one below
constexpr int kRows = 4;         // output rows per thread in the vertical pass
constexpr int kGroups = kT / 4;  // four-wide output groups per row in the horizontal pass
static_assert(kT * kGroups == 256, "one horizontal task per thread and tile");
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

struct Win {
  float w[kN];
};

// Rows are loaded by waves: wave w takes rows w, w + 4, ..., lane l column l (lanes 42-63
// load a valid clamped address and store nothing), so the column clamp is a per-lane
// constant and the row clamp a scalar.
struct HaloCols {
  uint32_t gxc;  // clamped image column of this lane
  bool inx;      // lane < 42 and its column inside the image
};

__device__ inline HaloCols halo_cols(int ox, int W) {
  const int lane = (int)(threadIdx.x % 64);
  const int gx = ox + lane;
  return {(uint32_t)min(max(gx, 0), W - 1), lane < kH && gx >= 0 && gx < W};
}

// This thread's share of 4 K rows of NI image planes from row oy on, into registers; the
// loads are issued together, and waited for where rows_store uses them.
template <int NI, int K>
__device__ inline void rows_load(const float* const (&img)[NI], HaloCols hc, int oy, int W, int H,
                                 float (&v)[NI][K]) {
  // wave-uniform (scalar) row arithmetic; per lane only the column offset
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int gy = min(max(oy + wave + 4 * k, 0), H - 1);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const float* rp = img[i] + (size_t)gy * W;
      v[i][k] = rp[hc.gxc];
    }
  }
}

// ... and from registers into rows of LDS tiles, zero outside the image (of the rows only
// the first R).
template <int NI, int K, int R>
__device__ inline void rows_store(float (*const (&tile)[NI])[kH], int row,
                                  const float (&v)[NI][K], HaloCols hc, int oy, int H) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  const int lane = (int)(threadIdx.x % 64);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int r = wave + 4 * k;
    const bool in = hc.inx && oy + r >= 0 && oy + r < H;
    if (lane < kH && r < R) {
#pragma unroll
      for (int i = 0; i < NI; ++i) tile[i][row + r][lane] = in ? v[i][k] : 0.f;
    }
  }
}

// Columns c0 .. c0 + 13 of row r of an LDS halo tile (c0 a multiple of 4, so
// the seven 8-byte reads are aligned): the inputs of four horizontal outputs.
__device__ inline void row14(const float (*tile)[kH], int r, int c0, float (&v)[14]) {
  const float2* p = reinterpret_cast<const float2*>(&tile[r][c0]);
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const float2 u = p[k];
    v[2 * k] = u.x;
    v[2 * k + 1] = u.y;
  }
}

// Views of one launch: blocks [first[k], first[k + 1]) are the strips of view k, channel by
// channel: a block takes `len` tiles below each other.  The views share a launch as far as
// the workspace holds their partials together.
struct LossViews {
  int n, len;
  uint32_t first[kMaxViews + 1];
  uint32_t tile0[kMaxViews];  // place of the view's first tile in the list of all tiles
  const float* x[kMaxViews];
  const float* y[kMaxViews];
  float* dl[kMaxViews];       // gradient, or null: none
  float* gmap[kMaxViews];     // partials of the view
  float scale[kMaxViews];
  int W[kMaxViews], H[kMaxViews];
};

// The strip of this block: view, channel, tile column bx and tile rows [by0, by1).
// Workgroups are dispatched to the eight XCDs (each with its own L2) in turn, so
// consecutive block indices go to different XCDs; the permutation below gives each XCD a
// contiguous run of strips instead, so that the columns neighbouring strips share are read
// into the same L2.  A bijection (the last total % 8 blocks keep their place), so every
// strip is done once whatever the dispatch order.
struct Strip {
  int v, ch, bx, by0, by1;
  uint32_t tile;     // list place of tile (bx, by0) of the channel; the next row is gx on
  uint32_t gx;
};

__device__ inline Strip strip_of(const LossViews& lv) {
  const uint32_t total = gridDim.x, L = blockIdx.x, n8 = total / 8;
  const uint32_t T = L < 8 * n8 ? (L % 8) * n8 + L / 8 : L;
  Strip st;
  st.v = 0;
  for (int k = 1; k < lv.n; ++k)
    if (T >= lv.first[k]) st.v = k;
  const uint32_t gx = (uint32_t)(lv.W[st.v] + kT - 1) / kT, gy = (uint32_t)(lv.H[st.v] + kT - 1) / kT;
  const uint32_t segs = (gy + lv.len - 1) / lv.len;
  const uint32_t t = T - lv.first[st.v], r = t % (gx * segs);
  st.ch = (int)(t / (gx * segs));
  st.by0 = (int)(r / gx) * lv.len;
  st.by1 = min(st.by0 + lv.len, (int)gy);
  st.bx = (int)(r % gx);
  st.gx = gx;
  st.tile = lv.tile0[st.v] + ((uint32_t)st.ch * gy + st.by0) * gx + st.bx;
  return st;
}

// Thread layout of the vertical pass: column c, rows r0 .. r0 + 3.
__device__ inline void vert_slot(int& c, int& r0) {
  c = threadIdx.x % kT;
  r0 = (threadIdx.x / kT) * kRows;
}

// Vertical filtering of NM moment maps held in LDS (hq[m][row][col]) for the
// four rows of this thread: out[o][m] = sum_i w[i] hq[m][r0 + o + i][c].
template <int NM>
__device__ inline void vert_filter(const float (*hq)[kH][kT], const Win& win, int c, int r0,
                                   float (*out)[NM]) {
#pragma unroll
  for (int o = 0; o < kRows; ++o)
#pragma unroll
    for (int m = 0; m < NM; ++m) out[o][m] = 0.f;
#pragma unroll
  for (int i = 0; i < kN + kRows - 1; ++i) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const float v = hq[m][r0 + i][c];
#pragma unroll
      for (int o = 0; o < kRows; ++o)
        if (i - o >= 0 && i - o < kN) out[o][m] = fmaf(win.w[i - o], v, out[o][m]);
    }
  }
}

// Four horizontally filtered outputs (columns c0 ..) of 14 inputs, into a row of hq.
__device__ inline void filter_row(const float (&in)[14], const Win& win, float* out) {
  float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < kN; ++i)
#pragma unroll
    for (int o = 0; o < 4; ++o) a[o] = fmaf(win.w[i], in[o + i], a[o]);
  *reinterpret_cast<float4*>(out) = make_float4(a[0], a[1], a[2], a[3]);
}

// The five moments of row r of the tiles, filtered, into row q of hq: map by map, with the
// products x^2, y^2, x y formed once per input (five maps at once hold 90 registers).
__device__ inline void moments_row(const float (*sx)[kH], const float (*sy)[kH], int r, int c0,
                                   const Win& win, float (*hq)[kH][kT], int q) {
  float xv[14], yv[14], p[14];
  row14(sx, r, c0, xv);
  row14(sy, r, c0, yv);
  filter_row(xv, win, &hq[0][q][c0]);
  __builtin_amdgcn_sched_barrier(0);
  filter_row(yv, win, &hq[1][q][c0]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 14; ++k) p[k] = xv[k] * xv[k];
  filter_row(p, win, &hq[2][q][c0]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 14; ++k) p[k] = yv[k] * yv[k];
  filter_row(p, win, &hq[3][q][c0]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < 14; ++k) p[k] = xv[k] * yv[k];
  filter_row(p, win, &hq[4][q][c0]);
}

// The last kC rows of NM filtered maps are carried to the top of the next tile's: quad j of
// this thread's share (threads past the end repeat the last quad), read into registers and,
// after a barrier, written.
constexpr int kCarryQuads = kC * kT / 4;  // per map

template <int NM>
__device__ inline int carry_quad(int j) {
  return min((int)threadIdx.x + 256 * j, NM * kCarryQuads - 1);
}

template <int NM>
__device__ inline float4 carry_read(const float (*hq)[kH][kT], int j) {
  const int e = carry_quad<NM>(j);
  return reinterpret_cast<const float4*>(&hq[e / kCarryQuads][kT][0])[e % kCarryQuads];
}

template <int NM>
__device__ inline void carry_write(float (*hq)[kH][kT], int j, float4 q) {
  const int e = carry_quad<NM>(j);
  reinterpret_cast<float4*>(&hq[e / kCarryQuads][0][0])[e % kCarryQuads] = q;
}

// SSIM and its partials of the four outputs of this thread (rows by kT + r0 .., column gx)
// from the five filtered maps; sx, sy at row 0: the tile's first row of centres.  Leaves the
// wave's sums of |x - y| and of SSIM in red.
template <bool GRAD>
__device__ inline void ssim_tile(const float (*hq)[kH][kT], const float (*sx)[kH],
                                 const float (*sy)[kH], const Win& win, int by, int c, int r0,
                                 int gx, int W, int H, float* __restrict__ g1,
                                 float* __restrict__ g2, float* __restrict__ g3,
                                 double (&red)[2][4]) {
  float mom[kRows][5];
  vert_filter<5>(hq, win, c, r0, mom);
  double l1 = 0.0, ss = 0.0;
  uint32_t pix = (uint32_t)(by * kT + r0) * (uint32_t)W + (uint32_t)gx;
#pragma unroll
  for (int o = 0; o < kRows; ++o, pix += (uint32_t)W) {
    const int gy = by * kT + r0 + o;
    if (gx < W && gy < H) {
      const float mx = mom[o][0], my = mom[o][1];
      const float sxx = mom[o][2] - mx * mx, syy = mom[o][3] - my * my;
      const float sxy = mom[o][4] - mx * my;
      const float A1 = 2.f * mx * my + kC1, A2 = 2.f * sxy + kC2;
      const float B1 = mx * mx + my * my + kC1, B2 = sxx + syy + kC2;
      // With P = 1/(B1 B2) and S = A1 A2 P:
      //   dS/dmu_x = 2 P my (A2 - A1) + 2 S mx (1/B2 - 1/B1),
      //   dS/dE[x^2] = -S / B2,  dS/dE[xy] = 2 A1 P,
      // so only B1 >= C1 and B2 >= C2 are inverted (A2 = 2 sigma_xy + C2 may vanish).
      const float iB1 = __builtin_amdgcn_rcpf(B1), iB2 = __builtin_amdgcn_rcpf(B2);
      const float Pb = iB1 * iB2;
      const float S = (A1 * A2) * Pb;
      if constexpr (GRAD) {
        g1[pix] = 2.f * (my * (A2 - A1) * Pb + S * mx * (iB2 - iB1));
        g2[pix] = -S * iB2;
        g3[pix] = 2.f * A1 * Pb;
      }
      l1 += fabs((double)sx[r0 + o][c + kR] - (double)sy[r0 + o][c + kR]);
      ss += (double)S;
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    l1 += __shfl_xor(l1, d, 64);
    ss += __shfl_xor(ss, d, 64);
  }
  if (__lane_id() == 0) {
    red[0][threadIdx.x / 64] = l1;
    red[1][threadIdx.x / 64] = ss;
  }
}

// The block's sums of a tile, by one thread after a barrier.
__device__ inline void write_part(double* part, uint32_t tile, const double (&red)[2][4]) {
  part[2 * (size_t)tile + 0] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
  part[2 * (size_t)tile + 1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
}

// STRIP: one block per strip of 32 x 32 tiles below each other and channel.  The ten
// filtered rows that a tile shares with the one below are carried, so each tile filters its
// 32 new rows only (one task per thread, where 42 rows take one and a third), and the next
// tile's rows are loaded while this one's are filtered.  Bound by VALU issue (about 200
// lane operations per output).  2048^2, three channels: 99 us, with a 42-row window per
// block 119.  Otherwise one tile per block: few blocks are bound by a block's chain of
// steps, which the strip's start lengthens.  GRAD: also write the partials (the metrics
// need none).
constexpr int kFwdBlocks = 4;  // strips resident per CU, by LDS (39.4 KB)
template <bool GRAD, bool STRIP>
__global__ __launch_bounds__(256, STRIP ? kFwdBlocks : 1) void k_ssim_fwd(
    LossViews lv, Win win, double* __restrict__ part) {
  // image rows of a tile's window; of a strip's tiles from the sixth on (centres and below)
  constexpr int kTop = STRIP ? kR : 0, kS = kH - kTop;
  __shared__ alignas(16) float sx[kS][kH];
  __shared__ alignas(16) float sy[kS][kH];
  __shared__ alignas(16) float hq[5][kH][kT];
  __shared__ double red[2][2][4];
  const Strip st = strip_of(lv);
  const int W = lv.W[st.v], H = lv.H[st.v], ch = st.ch;
  const size_t plane = (size_t)W * H;
  // partials of this channel (32-bit pixel offsets: a view has at most 2^28 pixels)
  float* __restrict__ const g1 = lv.gmap[st.v] + (size_t)ch * plane;
  float* __restrict__ const g2 = g1 + 3 * plane;
  float* __restrict__ const g3 = g2 + 3 * plane;
  const float* const src[2] = {lv.x[st.v] + ch * plane, lv.y[st.v] + ch * plane};
  float (*const dst[2])[kH] = {sx, sy};
  const HaloCols hc = halo_cols(st.bx * kT - kR, W);
  const int t = threadIdx.x, hr = t / kGroups, hc0 = (t % kGroups) * 4;
  const int oy = st.by0 * kT - kR;
  int c, r0;
  vert_slot(c, r0);
  const int gx = st.bx * kT + c;
  if constexpr (!STRIP) {
    float u[2][11];
    rows_load<2, 11>(src, hc, oy, W, H, u);
    rows_store<2, 11, kH>(dst, 0, u, hc, oy, H);
    __syncthreads();
    moments_row(sx, sy, hr, hc0, win, hq, hr);
    if (t < kC * kGroups) moments_row(sx, sy, kT + hr, hc0, win, hq, kT + hr);
    __syncthreads();
    ssim_tile<GRAD>(hq, sx + kR, sy + kR, win, st.by0, c, r0, gx, W, H, g1, g2, g3, red[0]);
    __syncthreads();
    if (t == 0) write_part(part, st.tile, red[0]);
    return;
  }
  float v[2][8];
  {
    // the rows above: the last ten of a tile before the first
    float u[2][3];
    rows_load<2, 3>(src, hc, oy, W, H, u);
    rows_load<2, 8>(src, hc, oy + kC, W, H, v);
    rows_store<2, 3, kC>(dst, kS - kC, u, hc, oy, H);
    __syncthreads();
    if (t < kC * kGroups) moments_row(sx, sy, kS - kC + hr, hc0, win, hq, kT + hr);
    __syncthreads();
  }
  uint32_t b = st.tile;
  for (int by = st.by0; by < st.by1; ++by, b += st.gx) {
    const float4 q0 = carry_read<5>(hq, 0), q1 = carry_read<5>(hq, 1);
    constexpr int kPairs = kR * kH / 2;  // and the last five image rows
    float2 cs = make_float2(0.f, 0.f);
    if (t < 2 * kPairs)
      cs = reinterpret_cast<const float2*>(t < kPairs ? &sx[kS - kR][0] : &sy[kS - kR][0])[t % kPairs];
    __syncthreads();
    if (by > st.by0 && t == 0) write_part(part, b - st.gx, red[(by - 1) & 1]);
    carry_write<5>(hq, 0, q0);
    carry_write<5>(hq, 1, q1);
    if (t < 2 * kPairs)
      reinterpret_cast<float2*>(t < kPairs ? &sx[0][0] : &sy[0][0])[t % kPairs] = cs;
    rows_store<2, 8, kT>(dst, kR, v, hc, by * kT + kR, H);
    __syncthreads();
    if (by + 1 < st.by1) rows_load<2, 8>(src, hc, (by + 1) * kT + kR, W, H, v);
    moments_row(sx, sy, kR + hr, hc0, win, hq, kC + hr);
    __syncthreads();
    ssim_tile<GRAD>(hq, sx, sy, win, by, c, r0, gx, W, H, g1, g2, g3, red[by & 1]);
  }
  __syncthreads();
  if (t == 0) write_part(part, b - st.gx, red[(st.by1 - 1) & 1]);
}

// Blocks as in the forward; bound by VALU issue and by the bytes of the partials.
// 2048^2, three channels: 71 us in strips, with a 42-row window per block 96.
constexpr int kBwdBlocks = 5;  // strips resident per CU, by LDS (32.3 KB)
template <bool STRIP>
__global__ __launch_bounds__(256, STRIP ? kBwdBlocks : 1) void k_ssim_bwd(LossViews lv, Win win,
                                                                          float lambda) {
  __shared__ alignas(16) float sg[3][STRIP ? kT : kH][kH];
  __shared__ alignas(16) float hq[3][kH][kT];
  const Strip st = strip_of(lv);
  float* __restrict__ dl = lv.dl[st.v];
  if (dl == nullptr) return;  // no gradient of this view (the whole block)
  const int W = lv.W[st.v], H = lv.H[st.v], ch = st.ch;
  const float* __restrict__ gmap = lv.gmap[st.v];
  const float scale = lv.scale[st.v];
  const size_t plane = (size_t)W * H;
  // this channel's planes (32-bit pixel offsets)
  const float* __restrict__ const x = lv.x[st.v] + ch * plane;
  const float* __restrict__ const y = lv.y[st.v] + ch * plane;
  float* __restrict__ const out = dl + ch * plane;
  const float* const src[3] = {gmap + (size_t)(0 * 3 + ch) * plane,
                               gmap + (size_t)(1 * 3 + ch) * plane,
                               gmap + (size_t)(2 * 3 + ch) * plane};
  float (*const dst[3])[kH] = {sg[0], sg[1], sg[2]};
  const HaloCols hc = halo_cols(st.bx * kT - kR, W);
  const int t = threadIdx.x, hr = t / kGroups, hc0 = (t % kGroups) * 4;
  const int oy = st.by0 * kT - kR;
  int c, r0;
  vert_slot(c, r0);
  const int gx = st.bx * kT + c;
  const uint32_t gxc = (uint32_t)min(gx, W - 1);
  auto maps_row = [&](int r, int q) {
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      float gv[14];
      row14(sg[m], r, hc0, gv);
      filter_row(gv, win, &hq[m][q][hc0]);
    }
  };
  float xv[kRows], yv[kRows];
  auto load_images = [&](int by) {
#pragma unroll
    for (int o = 0; o < kRows; ++o) {
      const uint32_t pix = (uint32_t)min(by * kT + r0 + o, H - 1) * (uint32_t)W + gxc;
      xv[o] = x[pix];
      yv[o] = y[pix];
    }
  };
  auto tile = [&](int by) {
    float f[kRows][3];
    vert_filter<3>(hq, win, c, r0, f);
#pragma unroll
    for (int o = 0; o < kRows; ++o) {
      const int gy = by * kT + r0 + o;
      if (gx >= W || gy >= H) break;
      const uint32_t pix = (uint32_t)gy * (uint32_t)W + (uint32_t)gx;
      const float sgn = (xv[o] > yv[o]) ? 1.f : ((xv[o] < yv[o]) ? -1.f : 0.f);
      out[pix] = scale *
                 ((1.f - lambda) * sgn - lambda * (f[o][0] + 2.f * xv[o] * f[o][1] + yv[o] * f[o][2]));
    }
  };
  if constexpr (!STRIP) {
    float u[3][11];
    rows_load<3, 11>(src, hc, oy, W, H, u);
    load_images(st.by0);
    rows_store<3, 11, kH>(dst, 0, u, hc, oy, H);
    __syncthreads();
    maps_row(hr, hr);
    if (t < kC * kGroups) maps_row(kT + hr, kT + hr);
    __syncthreads();
    tile(st.by0);
    return;
  }
  float v[3][8];
  {
    float u[3][3];
    rows_load<3, 3>(src, hc, oy, W, H, u);
    rows_load<3, 8>(src, hc, oy + kC, W, H, v);
    rows_store<3, 3, kC>(dst, 0, u, hc, oy, H);
    __syncthreads();
    if (t < kC * kGroups) maps_row(hr, kT + hr);
    __syncthreads();
  }
  for (int by = st.by0; by < st.by1; ++by) {
    const float4 q0 = carry_read<3>(hq, 0);
    __syncthreads();
    carry_write<3>(hq, 0, q0);
    rows_store<3, 8, kT>(dst, 0, v, hc, by * kT + kR, H);
    __syncthreads();
    load_images(by);
    if (by + 1 < st.by1) rows_load<3, 8>(src, hc, (by + 1) * kT + kR, W, H, v);
    maps_row(hr, kC + hr);
    __syncthreads();
    tile(by);
  }
}

// Tiles per strip for kernels of which `per_cu` blocks run at once on each of `cus` CUs:
// the length that costs a CU least, a strip's start taken as 0.7 tiles and k < per_cu
// blocks as 1 - (1 - k / per_cu)^2 of a full CU's rate (1024^2, three channels, forward:
// strips of 4 tiles 33 us, of 1 tile 41).
static int strip_len(const int* W, const int* H, int n, int per_cu, int cus) {
  int longest = 1, best = 1;
  double least = 1e30;
  for (int k = 0; k < n; ++k) longest = std::max(longest, (H[k] + kT - 1) / kT);
  for (int len = 1; len <= std::min(longest, 64); ++len) {
    size_t blocks = 0;
    for (int k = 0; k < n; ++k)
      blocks += (size_t)((W[k] + kT - 1) / kT) * 3 * (((H[k] + kT - 1) / kT + len - 1) / len);
    const size_t per = (blocks + cus - 1) / cus, rest = per % per_cu;
    const double idle = 1.0 - (double)rest / per_cu;
    const double cost =
        (len + 0.7) * ((double)(per - rest) + (rest != 0 ? rest / (1.0 - idle * idle) : 0.0));
    if (cost < least) {
      least = cost;
      best = len;
    }
  }
  return best;
}

// Up to this many tiles per CU a launch takes them one per block (256 CUs: loss and gradient
// of 64^2 and of 640 x 480 20 and 33 us, in strips 27 and 35; of 1024^2, 3072 tiles, 62
// and 61).
constexpr uint32_t kSinglePerCu = 4;

inline uint32_t tiles_of(int W, int H) {
  return (uint32_t)((W + kT - 1) / kT) * (uint32_t)((H + kT - 1) / kT) * 3u;
}

// Sets the strips of a launch (len: tiles per strip); returns its grid.
static dim3 set_strips(LossViews& lv, int len) {
  lv.len = len;
  lv.first[0] = 0;
  for (int k = 0; k < lv.n; ++k)
    lv.first[k + 1] = lv.first[k] + (uint32_t)((lv.W[k] + kT - 1) / kT) * 3u *
                                        (uint32_t)(((lv.H[k] + kT - 1) / kT + len - 1) / len);
  return dim3(lv.first[lv.n]);
}

// The passes over the views of lv: moments (and partials), then, with gradients, theirs.
template <bool GRAD>
static gs_status launch_views(LossViews& lv, const Win& win, double* part, float lambda, int cus,
                              hipStream_t s) {
  uint32_t tiles = 0;
  for (int k = 0; k < lv.n; ++k) tiles += tiles_of(lv.W[k], lv.H[k]);
  const bool single = tiles <= kSinglePerCu * (uint32_t)cus;
  dim3 grid = set_strips(lv, single ? 1 : strip_len(lv.W, lv.H, lv.n, kFwdBlocks, cus));
  auto fwd = single ? k_ssim_fwd<GRAD, false> : k_ssim_fwd<GRAD, true>;
  hipLaunchKernelGGL(fwd, grid, dim3(256), 0, s, lv, win, part);
  GS_LAUNCHED("ssim_fwd");
  if constexpr (GRAD) {
    grid = set_strips(lv, single ? 1 : strip_len(lv.W, lv.H, lv.n, kBwdBlocks, cus));
    auto bwd = single ? k_ssim_bwd<false> : k_ssim_bwd<true>;
    hipLaunchKernelGGL(bwd, grid, dim3(256), 0, s, lv, win, lambda);
    GS_LAUNCHED("ssim_bwd");
  }
  return GS_OK;
}

struct LossRed {
  int nv;
  int nblk[kMaxViews];
  long long off[kMaxViews];
  double inv_count[kMaxViews];
};

constexpr int kRedBlocks = 64;

__device__ inline void block_sum2(double& a, double& b) {
  __shared__ double sh[2][256];
  sh[0][threadIdx.x] = a;
  sh[1][threadIdx.x] = b;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      sh[0][threadIdx.x] += sh[0][threadIdx.x + st];
      sh[1][threadIdx.x] += sh[1][threadIdx.x + st];
    }
    __syncthreads();
  }
  a = sh[0][0];
  b = sh[1][0];
  __syncthreads();
}

// Stage 1: block (b, v) sums view v's partials b, b + 64, ... (fixed order).
__global__ __launch_bounds__(256) void k_loss_partial(const double* __restrict__ part, LossRed lr,
                                                      double* __restrict__ part2) {
  const int v = blockIdx.y;
  double a = 0.0, b = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < lr.nblk[v]; i += kRedBlocks * 256) {
    a += part[2 * (lr.off[v] + i) + 0];
    b += part[2 * (lr.off[v] + i) + 1];
  }
  block_sum2(a, b);
  if (threadIdx.x == 0) {
    part2[2 * (v * kRedBlocks + blockIdx.x) + 0] = a;
    part2[2 * (v * kRedBlocks + blockIdx.x) + 1] = b;
  }
}

// Stage 2: one block combines the per-view sums into the loss.
__global__ __launch_bounds__(256) void k_loss_final(const double* __restrict__ part2, LossRed lr,
                                                    float lambda, float* __restrict__ out) {
  double total = 0.0;
  for (int v = 0; v < lr.nv; ++v) {
    double a = 0.0, b = 0.0;
    if (threadIdx.x < kRedBlocks) {
      a = part2[2 * (v * kRedBlocks + threadIdx.x) + 0];
      b = part2[2 * (v * kRedBlocks + threadIdx.x) + 1];
    }
    block_sum2(a, b);
    total += (1.0 - lambda) * a * lr.inv_count[v] + lambda * (1.0 - b * lr.inv_count[v]);
  }
  if (threadIdx.x == 0) *out = (float)(total / lr.nv);
}

// Image-quality metrics: block (b, v) sums (x - y)^2 over view v's values
// b * 256 + t, b * 256 + t + 64 * 256, ... (fixed order) in float64.
struct ImagePtrs {
  const float* x[kMaxViews];
  const float* y[kMaxViews];
};

__global__ __launch_bounds__(256) void k_sq_partial(ImagePtrs im, LossRed lr,
                                                    double* __restrict__ part3) {
  const int v = blockIdx.y;
  const float* x = im.x[v];
  const float* y = im.y[v];
  const long long count = (long long)(0.5 + 1.0 / lr.inv_count[v]);
  double a = 0.0, b = 0.0;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < count;
       i += (long long)kRedBlocks * 256) {
    const double d = (double)x[i] - (double)y[i];
    a += d * d;
  }
  block_sum2(a, b);
  if (threadIdx.x == 0) part3[v * kRedBlocks + blockIdx.x] = a;
}

// Block v: mse, psnr = 10 log10(1 / mse), mean |x - y| and mean SSIM of view v.
__global__ __launch_bounds__(256) void k_metrics_final(const double* __restrict__ part2,
                                                       const double* __restrict__ part3,
                                                       LossRed lr, float* __restrict__ out) {
  const int v = blockIdx.x;
  double a = 0.0, b = 0.0, c = 0.0, d = 0.0;
  if (threadIdx.x < kRedBlocks) {
    a = part2[2 * (v * kRedBlocks + threadIdx.x) + 0];
    b = part2[2 * (v * kRedBlocks + threadIdx.x) + 1];
    c = part3[v * kRedBlocks + threadIdx.x];
  }
  block_sum2(a, b);
  block_sum2(c, d);
  if (threadIdx.x == 0) {
    const double mse = c * lr.inv_count[v];
    out[4 * v + 0] = (float)mse;
    out[4 * v + 1] = (float)(mse > 0.0 ? -10.0 * log10(mse) : INFINITY);
    out[4 * v + 2] = (float)(a * lr.inv_count[v]);
    out[4 * v + 3] = (float)(b * lr.inv_count[v]);
  }
}

}  // namespace

void loss_scratch_bytes(const int* W, const int* H, int nv, size_t* gmap_bytes,
                        size_t* part_bytes) {
  size_t max_plane = 0, total_blocks = 0;
  for (int v = 0; v < nv; ++v) {
    const size_t plane = (size_t)W[v] * H[v];
    if (plane > max_plane) max_plane = plane;
    total_blocks += (size_t)((W[v] + kT - 1) / kT) * ((H[v] + kT - 1) / kT) * 3;
  }
  *gmap_bytes = sizeof(float) * 9 * max_plane;  // the least: one view at a time
  // block partials (2 each), per-view stage-1 sums (2 each), metric sums (1 each)
  *part_bytes = sizeof(double) * (2 * (total_blocks + kRedBlocks * kMaxViews) +
                                  (size_t)kRedBlocks * kMaxViews);
}

gs_status loss_reserve(Ctx* ctx, LossScratch& ls, const int* W, const int* H, int nv,
                       hipStream_t s, bool shared) {
  if (ls.last_use == nullptr)
    GS_HIP(hipEventCreateWithFlags(&ls.last_use, hipEventDisableTiming));
  ls.cus = ctx->cu_count;
  size_t gb = 0, pb = 0;
  loss_scratch_bytes(W, H, nv, &gb, &pb);
  gs_status st = buf_ensure(ctx, ls.part, pb, s, ls.last_use);
  if (st != GS_OK) return st;
  // room for several small views at once (up to 2^22 pixels together), if there is any; a
  // graph's workspace cannot be given back, so under a budget it takes no more than it needs
  size_t pix = 0;
  for (int v = 0; v < nv; ++v) pix += (size_t)W[v] * H[v];
  const size_t want = sizeof(float) * 9 * std::min(pix, (size_t)1 << 22);
  if (want > gb && (shared || ctx->budget == 0) && buf_try(ctx, ls.gmap, want, s, ls.last_use))
    return GS_OK;
  return buf_ensure(ctx, ls.gmap, gb, s, ls.last_use);
}

// Whether two arrays of na and nb floats share memory (null: no array).
static bool meet(const float* a, size_t na, const float* b, size_t nb) {
  return a != nullptr && b != nullptr && a < b + nb && b < a + na;
}

// Launches `go` on runs of consecutive views that fit the workspace together (grad: their
// partials; without gradients all views at once).  Views that share an output, or read
// what another writes, go one after the other.
template <class F>
static gs_status loss_groups(const LossScratch& ls, const float* const* x, const float* const* y,
                             const int* W, const int* H, int nv, float* const* dl, bool grad,
                             F go) {
  const size_t cap = ls.gmap.cap / (sizeof(float) * 9);
  for (int v0 = 0, v1; v0 < nv; v0 = v1) {
    LossViews lv;
    lv.n = 0;
    uint32_t tiles = 0;
    size_t used = 0;
    for (v1 = v0; v1 < nv; ++v1) {
      const size_t plane = (size_t)W[v1] * H[v1];
      if (v1 > v0 && grad && used + plane > cap) break;
      float* d = grad && dl != nullptr ? dl[v1] : nullptr;
      bool apart = false;
      for (int k = 0; k < lv.n; ++k) {
        const size_t ak = 3 * (size_t)lv.W[k] * lv.H[k], a1 = 3 * plane;
        apart |= meet(d, a1, lv.dl[k], ak) || meet(d, a1, lv.x[k], ak) ||
                 meet(d, a1, lv.y[k], ak) || meet(lv.dl[k], ak, x[v1], a1) ||
                 meet(lv.dl[k], ak, y[v1], a1);
      }
      if (apart) break;
      const int k = lv.n++;
      lv.x[k] = x[v1];
      lv.y[k] = y[v1];
      lv.dl[k] = d;
      lv.gmap[k] = (float*)ls.gmap.p + 9 * used;
      lv.scale[k] = (float)(1.0 / (3.0 * (double)W[v1] * H[v1] * nv));
      lv.W[k] = W[v1];
      lv.H[k] = H[v1];
      lv.tile0[k] = tiles;
      tiles += tiles_of(W[v1], H[v1]);
      used += plane;
    }
    const gs_status st = go(lv, v0);
    if (st != GS_OK) return st;
  }
  return GS_OK;
}

gs_status launch_loss(const LossScratch& ls, const float* const* x, const float* const* y,
                      const int* W, const int* H, int nv, float lambda, float* loss_out,
                      float* const* dl, hipStream_t s) {
  Win win;
  {
    double g[kN], sum = 0.0;
    for (int i = 0; i < kN; ++i) {
      const double d = i - kR;
      g[i] = exp(-(d * d) / (2.0 * 1.5 * 1.5));
      sum += g[i];
    }
    for (int i = 0; i < kN; ++i) win.w[i] = (float)(g[i] / sum);
  }
  size_t total_blocks = 0;
  LossRed lr;
  lr.nv = nv;
  for (int v = 0; v < nv; ++v) {
    const size_t plane = (size_t)W[v] * H[v];
    const int nbx = (W[v] + kT - 1) / kT, nby = (H[v] + kT - 1) / kT;
    lr.nblk[v] = nbx * nby * 3;
    lr.off[v] = (long long)total_blocks;
    lr.inv_count[v] = 1.0 / (3.0 * (double)plane);
    total_blocks += (size_t)lr.nblk[v];
  }
  {
    size_t gb = 0, pb = 0;
    loss_scratch_bytes(W, H, nv, &gb, &pb);
    if (ls.gmap.cap < gb || ls.part.cap < pb) {
      set_error("internal: loss workspace of %zu / %zu bytes is smaller than %zu / %zu",
                ls.gmap.cap, ls.part.cap, gb, pb);
      return GS_ERR_CAPACITY;
    }
  }
  double* part2 = (double*)ls.part.p + 2 * total_blocks;
  bool grad = false;
  for (int v = 0; dl != nullptr && v < nv; ++v) grad |= dl[v] != nullptr;
  const gs_status st =
      loss_groups(ls, x, y, W, H, nv, dl, grad, [&](LossViews& lv, int v0) -> gs_status {
        double* part = (double*)ls.part.p + 2 * lr.off[v0];
        return grad ? launch_views<true>(lv, win, part, lambda, ls.cus, s)
                    : launch_views<false>(lv, win, part, lambda, ls.cus, s);
      });
  if (st != GS_OK) return st;
  if (loss_out != nullptr) {
    hipLaunchKernelGGL(k_loss_partial, dim3(kRedBlocks, nv), dim3(256), 0, s,
                       (const double*)ls.part.p, lr, part2);
    GS_LAUNCHED("loss_partial");
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, (const double*)part2, lr, lambda,
                       loss_out);
    GS_LAUNCHED("loss_final");
  }
  return GS_OK;
}

// ---------------------------------------------------------- fixed workspace
// Workspace of gs_loss_grad_noalloc: one file-scope device array per GPU, held
// for the life of the process, so that call allocates nothing.  In host code
// `scratch` names a host-side stand-in, never the device array: its device
// address comes from hipGetSymbolAddress, taken once per device with that
// device current (loss_noalloc_setup, called when a context is created) and
// kept in g_noalloc_ptr.
constexpr size_t kNoAllocGmapBytes = sizeof(float) * 9 * kNoAllocMaxPixels;
// 2048 output tiles cover any view of <= 2^20 pixels whose sides are <= 16384
// (ceil(W/32) ceil(H/32) <= 1536 there)
constexpr size_t kNoAllocPartBytes =
    sizeof(double) * (2 * ((size_t)kMaxViews * 3 * 2048 + (size_t)kRedBlocks * kMaxViews) +
                      (size_t)kRedBlocks * kMaxViews);
constexpr size_t kNoAllocBytes = kNoAllocGmapBytes + kNoAllocPartBytes;
static_assert(kNoAllocGmapBytes % 256 == 0, "partials start 256-byte aligned");

static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

constexpr int kNoAllocDevices = 64;
static std::atomic<void*> g_noalloc_ptr[kNoAllocDevices];

gs_status loss_noalloc_setup(int device) {
  if (device < 0 || device >= kNoAllocDevices) {
    set_error("device %d: the fixed loss workspace supports devices 0..%d", device,
              kNoAllocDevices - 1);
    return GS_ERR_UNSUPPORTED;
  }
  if (g_noalloc_ptr[device].load(std::memory_order_acquire) != nullptr) return GS_OK;
  static std::mutex mu;
  std::lock_guard<std::mutex> lk(mu);
  if (g_noalloc_ptr[device].load(std::memory_order_relaxed) != nullptr) return GS_OK;
  int cur = -1;
  GS_HIP(hipGetDevice(&cur));
  if (cur != device) {
    set_error("internal: loss_noalloc_setup(%d) with device %d current", device, cur);
    return GS_ERR_INVALID;
  }
  void* ptr = nullptr;
  GS_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
  if (ptr == nullptr) {
    set_error("hipGetSymbolAddress returned no address for the loss workspace");
    return GS_ERR_HIP;
  }
  g_noalloc_ptr[device].store(ptr, std::memory_order_release);
  return GS_OK;
}

gs_status loss_noalloc_workspace(const Ctx* ctx, const int* W, const int* H, int nv,
                                 LossScratch* out) {
  const int device = ctx->device;
  size_t gb = 0, pb = 0;
  loss_scratch_bytes(W, H, nv, &gb, &pb);
  if (gb > kNoAllocGmapBytes || pb > kNoAllocPartBytes) {
    set_error("gs_loss_grad_noalloc: views need a %zu + %zu byte workspace; the fixed one "
              "holds %zu + %zu bytes (at most %zu pixels per view)", gb, pb,
              kNoAllocGmapBytes, kNoAllocPartBytes, kNoAllocMaxPixels);
    return GS_ERR_CAPACITY;
  }
  void* base = (device >= 0 && device < kNoAllocDevices)
                   ? g_noalloc_ptr[device].load(std::memory_order_acquire)
                   : nullptr;
  if (base == nullptr) {
    set_error("gs_loss_grad_noalloc: the fixed workspace of device %d was not set up", device);
    return GS_ERR_INVALID;
  }
  out->gmap.p = base;
  out->gmap.cap = kNoAllocGmapBytes;
  out->part.p = (unsigned char*)base + kNoAllocGmapBytes;
  out->part.cap = kNoAllocPartBytes;
  out->last_use = nullptr;
  out->cus = ctx->cu_count;
  return GS_OK;
}

gs_status launch_metrics(const LossScratch& ls, const float* const* x, const float* const* y,
                         const int* W, const int* H, int nv, float* out, hipStream_t s) {
  Win win;
  {
    double g[kN], sum = 0.0;
    for (int i = 0; i < kN; ++i) {
      const double d = i - kR;
      g[i] = exp(-(d * d) / (2.0 * 1.5 * 1.5));
      sum += g[i];
    }
    for (int i = 0; i < kN; ++i) win.w[i] = (float)(g[i] / sum);
  }
  size_t total_blocks = 0;
  LossRed lr;
  lr.nv = nv;
  for (int v = 0; v < nv; ++v) {
    const size_t plane = (size_t)W[v] * H[v];
    lr.nblk[v] = ((W[v] + kT - 1) / kT) * ((H[v] + kT - 1) / kT) * 3;
    lr.off[v] = (long long)total_blocks;
    lr.inv_count[v] = 1.0 / (3.0 * (double)plane);
    total_blocks += (size_t)lr.nblk[v];
  }
  size_t gb = 0, pb = 0;
  loss_scratch_bytes(W, H, nv, &gb, &pb);
  if (ls.gmap.cap < gb || ls.part.cap < pb) {
    set_error("internal: metrics workspace too small");
    return GS_ERR_CAPACITY;
  }
  double* part = (double*)ls.part.p;
  double* part2 = part + 2 * total_blocks;
  double* part3 = part2 + 2 * (size_t)kRedBlocks * kMaxViews;
  const gs_status st = loss_groups(
      ls, x, y, W, H, nv, nullptr, false, [&](LossViews& lv, int v0) -> gs_status {
        return launch_views<false>(lv, win, part + 2 * lr.off[v0], 0.f, ls.cus, s);
      });
  if (st != GS_OK) return st;
  hipLaunchKernelGGL(k_loss_partial, dim3(kRedBlocks, nv), dim3(256), 0, s, (const double*)part,
                     lr, part2);
  GS_LAUNCHED("loss_partial");
  ImagePtrs im;
  for (int v = 0; v < nv; ++v) {
    im.x[v] = x[v];
    im.y[v] = y[v];
  }
  hipLaunchKernelGGL(k_sq_partial, dim3(kRedBlocks, nv), dim3(256), 0, s, im, lr, part3);
  GS_LAUNCHED("sq_partial");
  hipLaunchKernelGGL(k_metrics_final, dim3(nv), dim3(256), 0, s, (const double*)part2,
                     (const double*)part3, lr, out);
  GS_LAUNCHED("metrics_final");
  return GS_OK;
}

void loss_scratch_free(Ctx* ctx, LossScratch& ls) {
  buf_free(ctx, ls.gmap);
  buf_free(ctx, ls.part);
  if (ls.last_use != nullptr) (void)hipEventDestroy(ls.last_use);
  ls.last_use = nullptr;
}

}  // namespace isogs
