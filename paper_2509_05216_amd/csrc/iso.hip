// Isosurface points and ray-cast target views of a device-resident volume: the
// extraction and rendering that Sec. III does with ParaView, done on the GPU so
// a volume already in HBM (the in-situ setting of Sec. V) never leaves it.
//
// Extraction: edge crossings of the iso level (the vertex rule of marching
// cubes) in a canonical order: vertices row-major (k, j, i), per vertex its
// +x, +y, +z edges.  Three launches over blocks of 4096 vertices (16 per
// thread, four consecutive ones per 16-byte load; the +y and +z neighbours come
// through L1 and L2): count per block (comparison ballots), scan (two launches),
// emit (the blocks that hold crossings: the same predicates, ranked inside the
// block by ballot prefix counts, points written in order).  A crossing on edge e
// is kept when the Philox4x32-10 uniform of counter (e lo, e hi, 3, 0) is
// below keep_prob, so a subsample needs no sort and is the same however the
// grid is blocked.  Positions and the interpolation parameter in float64.
//
// Ray-cast: one thread per pixel: slab clipping to the box, samples at t_near + k step of
// the trilinear interpolant, the first rise through iso, ten bisections, headlight shading
// with the interpolant's gradient.  Every decision is that of the float64 interpolant:
// blocks of cells that lie on one side of the level are passed without samples, and a
// sample is evaluated in float32 first and in float64 where that cannot decide.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace isogs {
namespace {

constexpr int kIB = 256;          // threads per block
constexpr int kIV = 16;           // vertices per thread
constexpr int kIG = kIB * kIV;    // vertices per block
constexpr int kIW = kIB / 64;

struct VolDev {
  const float* v;
  long long nx, ny, nz;
  double lo[3], h[3];
  float iso;
};

struct KeepRule {
  uint32_t k0, k1;
  float prob;  // >= 1: keep all
};

__device__ inline bool kept(const KeepRule& r, unsigned long long e) {
  if (r.prob >= 1.0f) return true;
  uint32_t c[4] = {(uint32_t)e, (uint32_t)(e >> 32), 3u, 0u};
  philox4x32_10(c, r.k0, r.k1);
  return (float)(c[0] >> 8) * (1.0f / 16777216.0f) < r.prob;
}

// Chunk of this block: workgroups go to the eight XCDs in turn, so this bijection
// gives each XCD a contiguous run of chunks; the next plane's values, read for the z
// edges, are then still in that XCD's L2 when its own vertices are reached.
__device__ inline long long iso_chunk() {
  const uint32_t n8 = gridDim.x / 8;
  return blockIdx.x < 8 * n8 ? (blockIdx.x % 8) * n8 + blockIdx.x / 8 : blockIdx.x;
}

// Four values from p + o (any 4-byte alignment).
__device__ inline void load4(const float* p, uint32_t o, float* v) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  const f4u q = *reinterpret_cast<const f4u*>(p + o);
#pragma unroll
  for (int s = 0; s < 4; ++s) v[s] = q[s];
}

// What a block of kIG consecutive vertices needs: its first vertex, the vertices of
// the volume from it on, from its +y and from its +z neighbour on (clamped to 32 bits).
struct IsoBlock {
  const float* p[3];
  long long base;
  uint32_t left[3];
  uint32_t i, j, k;  // position of the first vertex
  float rnx, rny;
};

__device__ inline IsoBlock iso_block(const VolDev& V, long long nvert, long long chunk) {
  IsoBlock b;
  b.base = chunk * kIG;
  const long long row = b.base / V.nx;
  b.i = (uint32_t)(b.base - row * V.nx);
  b.k = (uint32_t)(row / V.ny);
  b.j = (uint32_t)(row - (long long)b.k * V.ny);
  b.rnx = 1.0f / (float)V.nx;
  b.rny = 1.0f / (float)V.ny;
  const long long st[3] = {0, V.nx, V.nx * V.ny};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const long long l = nvert - b.base - st[a];
    b.left[a] = l <= 0 ? 0u : (uint32_t)min(l, (long long)(2 * kIG));
    b.p[a] = V.v + (l > 0 ? b.base + st[a] : 0);
  }
  return b;
}

// n / d and its remainder for n < 2^22, d < 2^21, from d's float reciprocal: the estimate is
// off by at most one.
__device__ inline uint32_t div_small(uint32_t n, uint32_t d, float rd, uint32_t& rem) {
  uint32_t q = (uint32_t)((float)n * rd);
  int32_t r = (int32_t)(n - q * d);
  q = r < 0 ? q - 1 : (r >= (int32_t)d ? q + 1 : q);
  rem = n - q * d;
  return q;
}

// Position of vertex o of the block on the grid (sides up to 2^20, o < 2 kIG).
__device__ inline void vertex_ijk(const VolDev& V, const IsoBlock& B, uint32_t o, uint32_t& i,
                                  uint32_t& j, uint32_t& k) {
  const uint32_t dj = div_small(B.i + o, (uint32_t)V.nx, B.rnx, i);
  k = B.k + div_small(B.j + dj, (uint32_t)V.ny, B.rny, j);
}

// The values that the edges of this lane's four consecutive vertices o .. o + 3 of the
// block need: a (and in a[4] the vertex after the last), b (+y) and c (+z).
struct EdgeValues {
  float a[5], b[4], c[4];
};

__device__ inline void edge_load(const IsoBlock& B, uint32_t o, EdgeValues& v) {
  if (B.left[2] >= kIG) {  // the whole block and its neighbours are in the volume
    load4(B.p[0], o, v.a);
    v.a[4] = B.p[0][o + 4];
    load4(B.p[1], o, v.b);
    load4(B.p[2], o, v.c);
  } else {  // clamped addresses; what lies past the end is masked in edge_flags
#pragma unroll
    for (int s = 0; s < 5; ++s) v.a[s] = B.p[0][min(o + s, B.left[0] - 1)];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      v.b[s] = B.p[1][min(o + s, max(B.left[1], 1u) - 1)];
      v.c[s] = B.p[2][min(o + s, max(B.left[2], 1u) - 1)];
    }
  }
}

// Of the crossings f (see edge_flags), those that the subsample keeps.
__device__ inline uint32_t kept_flags(const KeepRule& r, const IsoBlock& B, uint32_t o, uint32_t f) {
  if (r.prob < 1.0f) {
    const unsigned long long e0 = 3ull * (unsigned long long)(B.base + o);
    for (uint32_t left = f; left != 0; left &= left - 1) {
      const int e = __builtin_ctz(left);
      if (!kept(r, e0 + e)) f &= ~(1u << e);
    }
  }
  return f;
}

// The kept crossings among those edges: bit 3 s + x for the edge of vertex o + s along axis
// x (the canonical order).  Returns 0 for the whole wave, without looking at positions,
// when no edge of its 256 vertices crosses (most waves: a surface meets few of them).  The
// sign tests compare the float32 values with iso directly, strictly (exact; NaN never
// crosses); every test is one comparison whose result is a wave mask, and the rest is
// scalar mask arithmetic.
__device__ inline uint32_t edge_flags(const VolDev& V, const KeepRule& r, const IsoBlock& B,
                                      uint32_t o, const EdgeValues& v) {
  const float(&a)[5] = v.a;
  const float(&b)[4] = v.b;
  const float(&c)[4] = v.c;
  unsigned long long lt[5], gt[5], m[4][3], any = 0;
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    lt[s] = __builtin_amdgcn_ballot_w64(a[s] < V.iso);
    gt[s] = __builtin_amdgcn_ballot_w64(a[s] > V.iso);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    m[s][0] = (lt[s] & gt[s + 1]) | (gt[s] & lt[s + 1]);
    m[s][1] = (lt[s] & __builtin_amdgcn_ballot_w64(b[s] > V.iso)) |
              (gt[s] & __builtin_amdgcn_ballot_w64(b[s] < V.iso));
    m[s][2] = (lt[s] & __builtin_amdgcn_ballot_w64(c[s] > V.iso)) |
              (gt[s] & __builtin_amdgcn_ballot_w64(c[s] < V.iso));
    any |= m[s][0] | m[s][1] | m[s][2];
  }
  if (any == 0) return 0u;
  uint32_t f = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int x = 0; x < 3; ++x)
      f |= __builtin_amdgcn_inverse_ballot_w64(m[s][x]) ? 1u << (3 * s + x) : 0u;
  // edges of the grid only: not past the last vertex of a row, column or the volume; a wave
  // inside one row knows its position as a whole
  const uint32_t o0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
  uint32_t i0, j0, k0;
  vertex_ijk(V, B, o0, i0, j0, k0);
  i0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)i0);
  j0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)j0);
  if (i0 + 256 <= (uint32_t)V.nx && B.left[2] >= kIG) {
    if (j0 + 1 == (uint32_t)V.ny) f &= ~0x492u;                          // the y edges
    if (i0 + 256 == (uint32_t)V.nx && __lane_id() == 63) f &= ~0x200u;  // the last x edge
    return kept_flags(r, B, o, f);
  }
  const uint32_t nx = (uint32_t)V.nx, ny = (uint32_t)V.ny;
  uint32_t i, j, k;
  vertex_ijk(V, B, o, i, j, k);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    uint32_t out = i + 1 == nx ? 1u : 0u;
    out |= j + 1 == ny ? 2u : 0u;
    out |= o + s >= B.left[2] ? 4u : 0u;
    out |= o + s >= B.left[0] ? 7u : 0u;
    f &= ~(out << (3 * s));
    const bool wrap = i + 1 == nx;
    j = wrap ? (j + 1 == ny ? 0u : j + 1) : j;
    i = wrap ? 0u : i + 1;
  }
  return kept_flags(r, B, o, f);
}

constexpr int kIS = kIV / 4;  // steps of four vertices per thread

// Bound by the read of the volume (4 B per vertex; the neighbours come from L1 and L2):
// 118 us for 512^3 vertices (4.6 TB/s; with every lane dividing for its position 139, with
// the loads step by step as well 144, with one vertex per lane, 64-bit positions and blocks
// in dispatch order 435).  Also writes which of the block's sixteen 256-vertex waves hold crossings (bit 4 q + w).
__global__ __launch_bounds__(kIB) void k_iso_count(VolDev V, KeepRule r, long long nvert,
                                                    uint32_t* __restrict__ tot,
                                                    uint16_t* __restrict__ held) {
  __shared__ uint32_t sh[kIW], sm[kIW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long long chunk = iso_chunk();
  const IsoBlock B = iso_block(V, nvert, chunk);
  EdgeValues v[kIS];
#pragma unroll
  for (int q = 0; q < kIS; ++q) edge_load(B, 4u * (q * kIB + threadIdx.x), v[q]);
  uint32_t n = 0, mine = 0;
#pragma unroll
  for (int q = 0; q < kIS; ++q) {
    const uint32_t f = edge_flags(V, r, B, 4u * (q * kIB + threadIdx.x), v[q]);
    n += (uint32_t)__popc(f);
    mine |= __builtin_amdgcn_ballot_w64(f != 0) != 0 ? 1u << (4 * q + w) : 0u;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d, 64);
  if (lane == 0) {
    sh[w] = n;
    sm[w] = mine;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0, m = 0;
    for (int q = 0; q < kIW; ++q) {
      t += sh[q];
      m |= sm[q];
    }
    tot[chunk] = t;
    held[chunk] = (uint16_t)m;
  }
}

// Offsets of the block totals in two launches: exclusive offsets within tiles of 4096
// totals (in place) and the tiles' totals, then the tiles' offsets and the grand total
// by one block.  (One block walking 32768 totals, a run per thread, took 60 us.)
constexpr int kTile = 4096;

__device__ inline uint32_t block_scan1024(uint32_t x, uint32_t* wsum, uint32_t& all) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)inc, d, 64);
    if (lane >= d) inc += y;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t before = 0;
  all = 0;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const uint32_t v = wsum[q];
    if (q < w) before += v;
    all += v;
  }
  return before + inc - x;
}

__global__ __launch_bounds__(1024) void k_iso_scan_tile(uint32_t* __restrict__ tot, long long nb,
                                                        uint32_t* __restrict__ tile_tot) {
  __shared__ uint32_t wsum[16];
  const long long i = (long long)blockIdx.x * kTile + 4 * threadIdx.x;
  uint32_t v[4], s = 0, all;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = i + j < nb ? tot[i + j] : 0u;
    s += v[j];  // a tile holds at most 3 x 2^24 edges
  }
  uint32_t run = block_scan1024(s, wsum, all);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (i + j < nb) tot[i + j] = run;
    run += v[j];
  }
  if (threadIdx.x == 0) tile_tot[blockIdx.x] = all;
}

__global__ __launch_bounds__(1024) void k_iso_scan_top(const uint32_t* __restrict__ tile_tot,
                                                       int tiles,
                                                       unsigned long long* __restrict__ tile_off) {
  __shared__ uint32_t wsum[16];
  unsigned long long carry = 0;
  for (int base = 0; base < tiles; base += 1024) {
    const int i = base + (int)threadIdx.x;
    const uint32_t v = i < tiles ? tile_tot[i] : 0u;
    // 16 bits at a time: 1024 totals of up to 3 x 2^24 do not fit 32 bits
    uint32_t all_lo, all_hi;
    const uint32_t lo = block_scan1024(v & 0xffffu, wsum, all_lo);
    __syncthreads();
    const uint32_t hi = block_scan1024(v >> 16, wsum, all_hi);
    __syncthreads();
    if (i < tiles) tile_off[i] = carry + lo + ((unsigned long long)hi << 16);
    carry += all_lo + ((unsigned long long)all_hi << 16);
  }
  if (threadIdx.x == 0) tile_off[tiles] = carry;
}

// Inclusive sums over the wave: shifts inside the 16-lane rows, then the rows' last lanes
// broadcast to the rows after them.
__device__ inline uint32_t wave_scan(uint32_t x) {
  auto add = [&](uint32_t y) { x += y; };
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true));   // row_shr:1
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true));   // row_shr:2
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true));   // row_shr:4
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true));   // row_shr:8
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false));  // row_bcast:15
  add((uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false));  // row_bcast:31
  return x;
}

// Blocks without a crossing leave at once; of the others only the waves' steps that hold
// crossings are loaded.  The block lists its crossings (vertex and axis) in LDS in the
// canonical order and takes them 256 at a time, so that the float64 divisions run with full
// waves and the points are stored coalesced: 135 us on a 512^3 volume with 1M crossings (a
// list per wave, every step loaded: 195 us; each lane writing the points of its own
// vertices, axis by axis: 312; walking every block as well: 765).
__global__ __launch_bounds__(kIB) void k_iso_emit(VolDev V, KeepRule r, long long nvert,
                                                   const uint32_t* __restrict__ off,
                                                   const unsigned long long* __restrict__ tile_off,
                                                   const uint16_t* __restrict__ held,
                                                   float* __restrict__ xyz, long long cap) {
  __shared__ uint32_t sh[kIS][kIW];
  __shared__ uint16_t list[kIG * 3];  // 4 x vertex in the block + axis
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long long chunk = iso_chunk();
  const uint32_t steps = held[chunk];
  if (steps == 0) return;
  const unsigned long long base = tile_off[chunk / kTile] + off[chunk];
  const IsoBlock B = iso_block(V, nvert, chunk);
  const uint32_t mine = (uint32_t)__builtin_amdgcn_readfirstlane((int)(steps >> w));
  EdgeValues v[kIS];
#pragma unroll
  for (int q = 0; q < kIS; ++q)
    if ((mine >> (4 * q)) & 1u) edge_load(B, 4u * (q * kIB + threadIdx.x), v[q]);
  uint32_t f[kIS], at[kIS];  // this lane's crossings, and the wave's before them
#pragma unroll
  for (int q = 0; q < kIS; ++q) {
    f[q] = at[q] = 0;
    uint32_t n = 0;
    if ((mine >> (4 * q)) & 1u) {
      f[q] = edge_flags(V, r, B, 4u * (q * kIB + threadIdx.x), v[q]);
      const uint32_t own = (uint32_t)__popc(f[q]);
      const uint32_t inc = wave_scan(own);
      n = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
      at[q] = inc - own;
    }
    if (lane == 0) sh[q][w] = n;
  }
  __syncthreads();
  // crossings of step q precede those of step q + 1; inside a step the waves are in order
  uint32_t total = 0;
#pragma unroll
  for (int q = 0; q < kIS; ++q) {
    uint32_t to = total + at[q];
#pragma unroll
    for (int x = 0; x < kIW; ++x) {
      const uint32_t n = sh[q][x];
      to += x < w ? n : 0u;
      total += n;
    }
    const uint32_t ov = 4u * (q * kIB + threadIdx.x);
    for (uint32_t left = f[q]; left != 0; left &= left - 1) {
      const uint32_t e = (uint32_t)__builtin_ctz(left), s = e / 3;
      list[to++] = (uint16_t)(4 * (ov + s) + (e - 3 * s));
    }
  }
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < total; t += kIB) {
    const uint32_t code = list[t];
    const int x = (int)(code & 3u);
    const long long vid = B.base + (code >> 2);
    const float v0 = V.v[vid];
    const float v1 = V.v[vid + (x == 0 ? 1 : (x == 1 ? V.nx : V.nx * V.ny))];
    uint32_t i, j, k;
    vertex_ijk(V, B, code >> 2, i, j, k);
    // t = a / (a - b), a = v0 - iso, b = v1 - iso (both exact in float64)
    const double u = ((double)v0 - (double)V.iso) / ((double)v0 - (double)v1);
    const double px = V.lo[0] + (double)i * V.h[0], py = V.lo[1] + (double)j * V.h[1],
                 pz = V.lo[2] + (double)k * V.h[2];
    const long long o = (long long)(base + t);
    if (o < cap) {
      xyz[o] = (float)(x == 0 ? px + u * V.h[0] : px);
      xyz[cap + o] = (float)(x == 1 ? py + u * V.h[1] : py);
      xyz[2 * cap + o] = (float)(x == 2 ? pz + u * V.h[2] : pz);
    }
  }
}

// ------------------------------------------------------------------ ray-cast
struct RayView {
  double R[9], o[3];
  double fx, fy, cx, cy;
  int W, H;
  int side;  // blocks per side of a chunk (see ray_block)
  float* img;
};

struct RayViews {
  RayView v[kMaxViews];
  int n;
};

// a / h rounded to nearest from r = 1 / h (itself so rounded): the residual of each
// estimate, exact in a fused multiply-add, corrects the next one (Markstein, "Computation
// of elementary functions on the IBM RISC System/6000 processor", 1990; it needs an h whose
// mantissa is not all ones, which the host checks).  Five operations against the
// division's dozen with a quarter-rate reciprocal among them.
__device__ inline double div_by(double a, double h, double r) {
  const double q0 = a * r;
  const double q1 = fma(fma(-h, q0, a), r, q0);
  return fma(fma(-h, q1, a), r, q1);
}

// The two corners of an x edge in one load (any 4-byte alignment).
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
__device__ inline f2u load2(const float* q) { return *reinterpret_cast<const f2u*>(q); }

// Trilinear value (and optionally gradient) of the volume at p.  RECIP: the cell
// coordinates by div_by (the same values).
template <bool RECIP>
__device__ inline double trilerp(const VolDev& V, const double* rh, const double* p, double* g) {
  double u[3];
  long long i0[3];
  double fr[3];
  const long long n[3] = {V.nx, V.ny, V.nz};
  for (int a = 0; a < 3; ++a) {
    u[a] = RECIP ? div_by(p[a] - V.lo[a], V.h[a], rh[a]) : (p[a] - V.lo[a]) / V.h[a];
    long long i = (long long)floor(u[a]);
    i = i < 0 ? 0 : (i > n[a] - 2 ? n[a] - 2 : i);
    i0[a] = i;
    fr[a] = u[a] - (double)i;
  }
  const float* b = V.v + (i0[2] * V.ny + i0[1]) * V.nx + i0[0];
  const long long sy = V.nx, sz = V.nx * V.ny;
  const f2u e00 = load2(b), e10 = load2(b + sy), e01 = load2(b + sz), e11 = load2(b + sz + sy);
  const double c000 = e00[0], c100 = e00[1], c010 = e10[0], c110 = e10[1];
  const double c001 = e01[0], c101 = e01[1], c011 = e11[0], c111 = e11[1];
  const double fx = fr[0], fy = fr[1], fz = fr[2];
  const double c00 = c000 + fx * (c100 - c000);
  const double c10 = c010 + fx * (c110 - c010);
  const double c01 = c001 + fx * (c101 - c001);
  const double c11 = c011 + fx * (c111 - c011);
  const double c0 = c00 + fy * (c10 - c00);
  const double c1 = c01 + fy * (c11 - c01);
  if (g != nullptr) {
    const double dx0 = (c100 - c000) * (1 - fy) + (c110 - c010) * fy;
    const double dx1 = (c101 - c001) * (1 - fy) + (c111 - c011) * fy;
    g[0] = (dx0 * (1 - fz) + dx1 * fz) / V.h[0];
    g[1] = ((c10 - c00) * (1 - fz) + (c11 - c01) * fz) / V.h[1];
    g[2] = (c1 - c0) / V.h[2];
  }
  return c0 + fz * (c1 - c0);
}

// ---- cells whose samples all lie on one side of the level
//
// The march only asks of a sample whether it lies below the level, and a ray spends most
// of its samples in cells whose corners all lie on one side.  A class per block of M^3
// cells (fine) and per 4^3 of those (coarse) lets it pass such blocks in one step each
// and evaluate the interpolant only near the surface, at the same samples t_near + k step
// with the same results.  A block is classed from the values of its cells and of at
// least one cell around it, so that the position's rounding (far below a cell: the host
// checks) cannot take a sample out of them, and with a margin of 1e-6 of the largest
// magnitude, far above the interpolant's rounding.
enum CellClass : uint8_t { kMixed = 0, kBelow = 1, kAbove = 2 };

struct CellGrid {
  const uint8_t *fine, *coarse;
  int shift;           // log2 M
  int b[3], c[3];      // fine and coarse blocks per axis
  int last[3];         // the last cell per axis
  uint32_t plane;      // vertices of an (x, y) plane
  double rh[3];        // 1 / h
};

// Least and largest value of every block of M^3 vertices (unbounded when one is not
// finite).  Bound by reading the volume once (16 bytes per load, a wave 1 KB of a row).
template <int M>
__global__ __launch_bounds__(256) void k_cell_minmax(VolDev V, int bx, int by, float2* mm) {
  constexpr int L = M / 4;  // lanes per block row
  const int x0 = (blockIdx.x * 256 + threadIdx.x) * 4;
  const int j = blockIdx.y, k = blockIdx.z;
  float lo = INFINITY, hi = -INFINITY;
  bool odd = false;
  const int ye = min((long long)M, V.ny - (long long)j * M), ze = min((long long)M, V.nz - (long long)k * M);
  auto take = [&](float v) {
    lo = fminf(lo, v);
    hi = fmaxf(hi, v);
    odd |= !(fabsf(v) < INFINITY);
  };
  if (x0 + 3 < V.nx) {
    typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
    for (int z = 0; z < ze; ++z) {
      const float* row = V.v + (((long long)k * M + z) * V.ny + (long long)j * M) * V.nx + x0;
      f4u q[M];
#pragma unroll
      for (int y = 0; y < M; ++y)  // rows past the last repeat it
        q[y] = *reinterpret_cast<const f4u*>(row + min(y, ye - 1) * V.nx);
#pragma unroll
      for (int y = 0; y < M; ++y)
#pragma unroll
        for (int c = 0; c < 4; ++c) take(q[y][c]);
    }
  } else {
    for (int z = 0; z < ze; ++z)
      for (int y = 0; y < ye; ++y)
        for (int x = x0; x < V.nx; ++x)
          take(V.v[(((long long)k * M + z) * V.ny + (long long)j * M + y) * V.nx + x]);
  }
  if (odd) {
    lo = -INFINITY;
    hi = INFINITY;
  }
#pragma unroll
  for (int d = 1; d < L; d <<= 1) {
    lo = fminf(lo, __shfl_xor(lo, d, 64));
    hi = fmaxf(hi, __shfl_xor(hi, d, 64));
  }
  const int i = x0 / M;
  if (i < bx && (x0 / 4) % L == 0) mm[((size_t)k * by + j) * bx + i] = make_float2(lo, hi);
}

// Classes from the values of a block and its 26 neighbours; one wave per coarse block.
__global__ __launch_bounds__(64) void k_cell_class(const float2* __restrict__ mm, int bx, int by,
                                                   int bz, float iso, uint8_t* __restrict__ fine,
                                                   uint8_t* __restrict__ coarse) {
  __shared__ float2 t[216];
  const int ox = blockIdx.x * 4 - 1, oy = blockIdx.y * 4 - 1, oz = blockIdx.z * 4 - 1;
  for (int q = threadIdx.x; q < 216; q += 64) {
    const int x = ox + q % 6, y = oy + (q / 6) % 6, z = oz + q / 36;
    const bool in = x >= 0 && y >= 0 && z >= 0 && x < bx && y < by && z < bz;
    t[q] = in ? mm[((size_t)z * by + y) * bx + x] : make_float2(INFINITY, -INFINITY);
  }
  __syncthreads();
  const int lx = threadIdx.x % 4, ly = (threadIdx.x / 4) % 4, lz = threadIdx.x / 16;
  float lo = INFINITY, hi = -INFINITY;
  for (int dz = 0; dz < 3; ++dz)
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const float2 v = t[((lz + dz) * 6 + ly + dy) * 6 + lx + dx];
        lo = fminf(lo, v.x);
        hi = fmaxf(hi, v.y);
      }
  const double margin = 1e-6 * (double)fmaxf(fabsf(lo), fabsf(hi));
  const int cls = (double)hi - (double)iso < -margin  ? kBelow
                  : (double)lo - (double)iso > margin ? kAbove
                                                      : kMixed;
  const int x = ox + 1 + lx, y = oy + 1 + ly, z = oz + 1 + lz;
  const bool in = x < bx && y < by && z < bz;
  if (in) fine[((size_t)z * by + y) * bx + x] = (uint8_t)cls;
  const uint64_t all = __ballot(in);
  const uint64_t below = __ballot(in && cls == kBelow), above = __ballot(in && cls == kAbove);
  if (threadIdx.x == 0)
    coarse[((size_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] =
        below == all ? kBelow : (above == all ? kAbove : kMixed);
}

// The cell (and the place in it) at coordinates m s + b.
__device__ inline void cell_of(const CellGrid& G, double m, const double* s, const double* b,
                               int* i, float* fr) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double u = fma(m, s[a], b[a]);
    i[a] = min(max((int)u, 0), G.last[a]);
    if (fr != nullptr) fr[a] = (float)(u - (double)i[a]);
  }
}

// Index of the block of 2^s cells that holds cell i (the host checks that rows of blocks
// fit 24 bits and blocks 32).
__device__ inline uint32_t block_at(const int* i, int s, const int* n) {
  return __umul24(__umul24(i[2] >> s, n[1]) + (i[1] >> s), n[0]) + (i[0] >> s);
}

// Within 1e-6 of a cell's face a sample may belong to another cell than cell_of says (the
// coordinates round by less than 1e-7, as the host checks).  Between finite cells that
// changes nothing, but the cell that the sample belongs to may have corners that are not.
constexpr float kFace = 0.499999f;
__device__ inline float off_centre(const float* fr) {
  return fmaxf(fmaxf(fabsf(fr[0] - 0.5f), fabsf(fr[1] - 0.5f)), fabsf(fr[2] - 0.5f));
}

// The side of the level on which the interpolant at coordinates m s + b lies, from its
// float32 evaluation, whose error is below 1e-5 of the cell's values and of the level;
// kMixed where that cannot tell, and outside the range in which it holds (two terms of the
// bound): differences of corners overflow from about 1.7e38 on, and near 1e-38 the rounding
// stops shrinking with the values.  FACE: also kMixed beside a cell's face.
template <bool FACE>
__device__ inline int quick_side(const VolDev& V, const CellGrid& G, double m, const double* s,
                                 const double* b) {
  int i[3];
  float fr[3];
  cell_of(G, m, s, b, i, fr);
  const uint32_t row = __umul24(i[2], (int)V.ny) + i[1];
  const float* p = V.v + ((unsigned long long)row * (uint32_t)V.nx + i[0]);
  const uint32_t sy = (uint32_t)V.nx, sz = G.plane;
  const f2u e00 = load2(p), e10 = load2(p + sy), e01 = load2(p + sz), e11 = load2(p + sz + sy);
  const float c00 = fmaf(fr[0], e00[1] - e00[0], e00[0]);
  const float c10 = fmaf(fr[0], e10[1] - e10[0], e10[0]);
  const float c01 = fmaf(fr[0], e01[1] - e01[0], e01[0]);
  const float c11 = fmaf(fr[0], e11[1] - e11[0], e11[0]);
  const float c0 = fmaf(fr[1], c10 - c00, c00), c1 = fmaf(fr[1], c11 - c01, c01);
  const float f = fmaf(fr[2], c1 - c0, c0) - V.iso;
  const float big =
      fmaxf(fmaxf(fmaxf(fabsf(e00[0]), fabsf(e00[1])), fmaxf(fabsf(e10[0]), fabsf(e10[1]))),
            fmaxf(fmaxf(fabsf(e01[0]), fabsf(e01[1])), fmaxf(fabsf(e11[0]), fabsf(e11[1]))));
  // infinite from 3.4e36 on, at least 1e-35
  const float bound = fmaf((big + fabsf(V.iso)) * 100.f, 1e-7f, 1e-35f);
  if (FACE && off_centre(fr) > kFace) return kMixed;
  return fabsf(f) > bound ? (f < 0.f ? kBelow : kAbove) : kMixed;
}

// Whether the sample at coordinates m s + b is beside a face of its cell.
__device__ inline bool beside_face(const CellGrid& G, double m, const double* s, const double* b) {
  int i[3];
  float fr[3];
  cell_of(G, m, s, b, i, fr);
  return off_centre(fr) > kFace;
}

// Place (in blocks of 16 x 16 pixels) of block L of a view.  Workgroups go to the eight XCDs
// in turn; each XCD takes whole chunks of side x side blocks, so that neighbouring rays'
// values meet in one L2, and chunks go round the XCDs, so that each has a share of the
// expensive parts of the image.
__device__ inline void ray_block(const RayView& c, uint32_t L, int& bx, int& by) {
  const uint32_t per = (uint32_t)(c.side * c.side), s = L / 8;
  const uint32_t chunk = (s / per) * 8 + L % 8, in = s % per;
  const uint32_t cx = (uint32_t)((c.W + 16 * c.side - 1) / (16 * c.side));
  bx = (int)(chunk % cx) * c.side + (int)(in % c.side);
  by = (int)(chunk / cx) * c.side + (int)(in / c.side);
}

// One thread per pixel, a wave an 8 x 8 block of them: neighbouring rays read the same
// cells and leave the march together (64 x 1 pixels: 4258 us for two 1024^2 views of a
// 512^3 volume at one sample a cell, 8 x 8: 2640).  QUICK: samples are decided by
// quick_side, and by the cell classes where they were built (same views: 2190 us without,
// 568 with them, of which the classes 125); else all in float64.  Without classes bound by
// the gathers' cache lines, with them by the latency of a ray's steps (23 blocks and 20
// samples a wave on average, 116 and 161 in the longest) and float64 issue.  Five waves per
// SIMD: left to itself the compiler takes registers for four (572 us instead of 546 for
// those views, averages of two runs each).
template <bool QUICK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_raycast(
    VolDev V, RayViews rv, CellGrid G, double step, double hi0, double hi1, double hi2) {
  const RayView& c = rv.v[blockIdx.y];
  int bx, by;
  ray_block(c, blockIdx.x, bx, by);
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int x = bx * 16 + (wave % 2) * 8 + lane % 8;
  const int y = by * 16 + (wave / 2) * 8 + lane / 8;
  if (x >= c.W || y >= c.H) return;
  const double dc[3] = {((double)x + 0.5 - c.cx) / c.fx, ((double)y + 0.5 - c.cy) / c.fy, 1.0};
  double d[3];
  for (int a = 0; a < 3; ++a) d[a] = dc[0] * c.R[0 * 3 + a] + dc[1] * c.R[1 * 3 + a] + dc[2] * c.R[2 * 3 + a];
  const double dn = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  for (int a = 0; a < 3; ++a) d[a] /= dn;
  const double hi[3] = {hi0, hi1, hi2};
  double tn = 0.0, tf = INFINITY;
  bool box = true;
  for (int a = 0; a < 3; ++a) {
    if (d[a] == 0.0) {
      if (c.o[a] < V.lo[a] || c.o[a] > hi[a]) box = false;
      continue;
    }
    const double t0 = (V.lo[a] - c.o[a]) / d[a], t1 = (hi[a] - c.o[a]) / d[a];
    tn = fmax(tn, fmin(t0, t1));
    tf = fmin(tf, fmax(t0, t1));
  }
  float rgb[3] = {0.f, 0.f, 0.f};
  if (box && tf > tn && tf < INFINITY) {  // a camera that is not finite sees nothing
    double p[3];
    auto value = [&](double t) {
      for (int a = 0; a < 3; ++a) p[a] = c.o[a] + t * d[a];
      return trilerp<QUICK>(V, G.rh, p, nullptr) - (double)V.iso;
    };
    double lo_t = 0.0, hi_t = -1.0;
    double uo[3], ut[3];
    if constexpr (QUICK) {
      // cell coordinates at t: uo + t ut; at sample k: u0 + k us; the k that reaches a
      // coordinate: plane iu + pu (never along an axis that the ray does not move on)
      double u0[3], us[3], iu[3], pu[3];
      for (int a = 0; a < 3; ++a) {
        uo[a] = (c.o[a] - V.lo[a]) * G.rh[a];
        ut[a] = d[a] * G.rh[a];
        u0[a] = fma(tn, ut[a], uo[a]);
        us[a] = step * ut[a];
        iu[a] = us[a] != 0.0 ? 1.0 / us[a] : 0.0;
        pu[a] = us[a] != 0.0 ? -u0[a] * iu[a] : 1e300;
      }
      // the last sample in the box
      int kl = (int)((tf - tn) / step);
      while (tn + (double)(kl + 1) * step <= tf) ++kl;
      while (tn + (double)kl * step > tf) --kl;
      bool below = false;  // the previous sample lies below the level
      bool risen = false;
      int k = 0;
      while (k <= kl) {
        int i[3];
        int cls = kMixed, ke = kl;
        if (G.fine != nullptr) {
          cell_of(G, (double)k, us, u0, i, nullptr);
          const int sf = G.shift, sc = G.shift + 2;
          const int far = G.coarse[block_at(i, sc, G.c)], near = G.fine[block_at(i, sf, G.b)];
          const int s = far != kMixed ? sc : sf;
          cls = far != kMixed ? far : near;
          // the last sample before the ray leaves the block
          double kx = (double)kl;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const int in = (1 << s) - 1, plane = us[a] > 0.0 ? (i[a] | in) + 1 : i[a] & ~in;
            kx = fmin(kx, fma((double)plane, iu[a], pu[a]));
          }
          ke = max(k, (int)kx);
        }
        if (cls == kMixed) {
          for (; k <= ke; ++k) {
            int at = quick_side<false>(V, G, (double)k, us, u0);
            if (at == kMixed) {
              const double f = value(tn + (double)k * step);
              at = f < 0.0 ? kBelow : (f >= 0.0 ? kAbove : kMixed);
            }
            risen = below && at == kAbove;
            if (risen) break;
            below = at == kBelow;
          }
        } else if (cls == kAbove && below) {
          risen = true;
        } else {
          below = cls == kBelow;
          k = ke + 1;
        }
        if (risen) {
          // the two samples whose sides make the rise, where a neighbouring cell's values
          // may have stood for theirs
          if (beside_face(G, (double)(k - 1), us, u0) || beside_face(G, (double)k, us, u0)) {
            const double f = value(tn + (double)k * step);
            risen = f >= 0.0 && value(tn + (double)(k - 1) * step) < 0.0;
            if (!risen) {
              below = f < 0.0;
              ++k;
              continue;
            }
          }
          lo_t = tn + (double)(k - 1) * step;
          hi_t = tn + (double)k * step;
          break;
        }
      }
    } else {
      double f_prev = value(tn);
      for (long long k = 1;; ++k) {
        const double tk = tn + (double)k * step;
        if (tk > tf) break;
        const double f = value(tk);
        if (f_prev < 0.0 && f >= 0.0) {
          lo_t = tn + (double)(k - 1) * step;
          hi_t = tk;
          break;
        }
        f_prev = f;
      }
    }
    if (hi_t >= 0.0) {
      for (int it = 0; it < 10; ++it) {
        const double mid = 0.5 * (lo_t + hi_t);
        int at = kMixed;
        if constexpr (QUICK) at = quick_side<true>(V, G, mid, ut, uo);
        if (at == kBelow || (at == kMixed && value(mid) < 0.0))
          lo_t = mid;
        else
          hi_t = mid;
      }
      const double th = 0.5 * (lo_t + hi_t);
      for (int a = 0; a < 3; ++a) p[a] = c.o[a] + th * d[a];
      double g[3];
      (void)trilerp<QUICK>(V, G.rh, p, g);
      const double gn = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
      const double lam = gn > 0.0 ? fabs((g[0] * d[0] + g[1] * d[1] + g[2] * d[2]) / gn) : 0.0;
      const double sh = 0.2 + 0.8 * lam;
      rgb[0] = (float)(0.85 * sh);
      rgb[1] = (float)((0.45 + 0.25 * p[2]) * sh);
      rgb[2] = (float)((0.30 + 0.25 * (p[0] + 1.0)) * sh);
    }
  }
  const size_t plane = (size_t)c.W * c.H, pix = (size_t)y * c.W + x;
  for (int ch = 0; ch < 3; ++ch) c.img[ch * plane + pix] = rgb[ch];
}

VolDev vol_dev(const gs_volume& vol, float iso) {
  VolDev V;
  V.v = vol.values;
  V.nx = vol.nx;
  V.ny = vol.ny;
  V.nz = vol.nz;
  const long long n[3] = {vol.nx, vol.ny, vol.nz};
  for (int a = 0; a < 3; ++a) {
    V.lo[a] = (double)vol.lo[a];
    V.h[a] = ((double)vol.hi[a] - (double)vol.lo[a]) / (double)(n[a] - 1);
  }
  V.iso = iso;
  return V;
}

// What the quick march needs of the volume and the rays: cells whose size div_by takes,
// rays whose positions round far inside a cell (1e-16 of the distance from the origin),
// and 32-bit rows and planes.  False: the plain march.
bool quick_suits(const gs_volume& vol, const VolDev& V, const RayViews& rv, CellGrid& G) {
  const long long n[3] = {vol.nx, vol.ny, vol.nz};
  double size = 0.0, cam = 0.0;
  for (int a = 0; a < 3; ++a) size += std::fabs(V.lo[a]) + (double)n[a] * V.h[a];
  for (int k = 0; k < rv.n; ++k)
    cam = std::fmax(cam, std::fabs(rv.v[k].o[0]) + std::fabs(rv.v[k].o[1]) +
                             std::fabs(rv.v[k].o[2]));
  for (int a = 0; a < 3; ++a) {
    int e = 0;
    const double h = V.h[a], m = std::frexp(h, &e);
    if (!(h > 1e-30 && h < 1e30) || m == 1.0 - 0x1p-53) return false;
    if (!((size + cam) * 1e-15 < 1e-7 * h)) return false;
    G.rh[a] = 1.0 / h;
    G.last[a] = (int)n[a] - 2;
  }
  G.plane = (uint32_t)(V.nx * V.ny);
  return V.nx * V.ny < (1LL << 31) && V.ny * V.nz < (1LL << 32);
}

// Whether classing the cells pays, for rays of at most `samples` samples through `cells`
// cells (the box diagonal).  Measured on one MI355X, step = one cell, us without and with
// classes: 64^3 two 1024^2 views 196, 225; 128^3 512^2 100, 108, two 1024^2 368, 279;
// 256^3 128^2 256, 179, two 1024^2 800, 331; 512^3 32^2 430, 318, two 1024^2 2190, 568;
// 100^3 at a fiftieth of a cell 804, 856.  Classing reads the volume (1.4e6 vertices
// per us), a march without it takes about 0.9 us a sample or 0.85e6 samples per us.
bool classes_pay(double vertices, double pixels, double samples, double cells) {
  const double reach = std::min(samples, cells);
  return (reach >= 384.0 || (reach >= 192.0 && pixels >= 1048576.0)) &&
         vertices / 1.4e6 < 0.5 * samples * std::max(0.9, pixels / 0.85e6);
}

// The class grid of the volume in the context's scratch, built on stream s; false when
// there is no room for it.  The caller holds ray_mutex.
bool build_grid(Ctx* ctx, const VolDev& V, CellGrid& G, hipStream_t s) {
  // blocks of 4^3 cells, of 8^3 for volumes of more than 2^28 vertices, whose block
  // values would take more than 36 MB
  const int M = V.nx * V.ny * V.nz > (1LL << 28) ? 8 : 4;
  G.shift = M == 8 ? 3 : 2;
  const long long n[3] = {V.nx, V.ny, V.nz};
  size_t nb = 1, nc = 1;
  for (int a = 0; a < 3; ++a) {
    G.b[a] = (int)((n[a] + M - 1) / M);
    G.c[a] = (G.b[a] + 3) / 4;
    nb *= (size_t)G.b[a];
    nc *= (size_t)G.c[a];
  }
  // block_at's 24- and 32-bit products, and the grid limits of the two launches
  if (nb >= ((size_t)1 << 32) || (long long)G.b[1] * G.b[2] >= (1 << 24) || G.b[1] > 65535 ||
      G.b[2] > 65535)
    return false;
  if (ctx->ray_use == nullptr &&
      hipEventCreateWithFlags(&ctx->ray_use, hipEventDisableTiming) != hipSuccess) {
    ctx->ray_use = nullptr;
    return false;
  }
  const size_t bytes = nb * sizeof(float2) + nb + nc;
  // growing waits for the earlier rays that read the old buffer; other calls' rays on
  // other streams are waited for on the device
  if (!buf_try(ctx, ctx->ray_blk, bytes, s, ctx->ray_use) ||
      hipStreamWaitEvent(s, ctx->ray_use, 0) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  float2* mm = (float2*)ctx->ray_blk.p;
  uint8_t* fine = (uint8_t*)(mm + nb);
  uint8_t* coarse = fine + nb;
  const dim3 gm((unsigned)((V.nx + 1023) / 1024), (unsigned)G.b[1], (unsigned)G.b[2]);
  if (M == 8)
    hipLaunchKernelGGL(k_cell_minmax<8>, gm, dim3(256), 0, s, V, G.b[0], G.b[1], mm);
  else
    hipLaunchKernelGGL(k_cell_minmax<4>, gm, dim3(256), 0, s, V, G.b[0], G.b[1], mm);
  hipLaunchKernelGGL(k_cell_class, dim3(G.c[0], G.c[1], G.c[2]), dim3(64), 0, s,
                     (const float2*)mm, G.b[0], G.b[1], G.b[2], V.iso, fine, coarse);
  G.fine = fine;
  G.coarse = coarse;
  return true;
}

}  // namespace

// The extraction's scratch: tile offsets and the grand total (64-bit), block offsets, tile
// totals, the waves that hold crossings.
struct IsoScratch {
  long long nvert, nb, tiles;
  size_t bytes;
  unsigned long long* tile_off;
  uint32_t *off, *tile_tot;
  uint16_t* held;
  IsoScratch(Ctx* ctx, const gs_volume& vol) {
    nvert = (long long)vol.nx * vol.ny * vol.nz;
    nb = (nvert + kIG - 1) / kIG;
    tiles = (nb + kTile - 1) / kTile;
    bytes = sizeof(unsigned long long) * (size_t)(tiles + 1) +
            sizeof(uint32_t) * (size_t)(nb + tiles) + sizeof(uint16_t) * (size_t)nb;
    place(ctx);
  }
  void place(Ctx* ctx) {
    tile_off = (unsigned long long*)ctx->iso_blk.p;
    off = (uint32_t*)(tile_off + tiles + 1);
    tile_tot = off + nb;
    held = (uint16_t*)(tile_tot + tiles);
  }
};

gs_status iso_count(Ctx* ctx, const gs_volume& vol, float iso, float keep_prob, uint64_t seed,
                    int64_t* n_kept, hipStream_t s) {
  const VolDev V = vol_dev(vol, iso);
  const KeepRule r{(uint32_t)seed, (uint32_t)(seed >> 32), keep_prob};
  IsoScratch w(ctx, vol);
  gs_status st = buf_ensure(ctx, ctx->iso_blk, w.bytes, s);
  if (st != GS_OK) return st;
  w.place(ctx);
  if (ctx->iso_host == nullptr)
    GS_HIP(hipHostMalloc((void**)&ctx->iso_host, sizeof(unsigned long long),
                         hipHostMallocDefault));
  hipLaunchKernelGGL(k_iso_count, dim3((unsigned)w.nb), dim3(kIB), 0, s, V, r, w.nvert, w.off,
                     w.held);
  GS_LAUNCHED("iso_count");
  hipLaunchKernelGGL(k_iso_scan_tile, dim3((unsigned)w.tiles), dim3(1024), 0, s, w.off, w.nb,
                     w.tile_tot);
  GS_LAUNCHED("iso_scan_tile");
  hipLaunchKernelGGL(k_iso_scan_top, dim3(1), dim3(1024), 0, s, (const uint32_t*)w.tile_tot,
                     (int)w.tiles, w.tile_off);
  GS_LAUNCHED("iso_scan_top");
  GS_HIP(hipMemcpyAsync(ctx->iso_host, w.tile_off + w.tiles, sizeof(unsigned long long),
                        hipMemcpyDeviceToHost, s));
  GS_HIP(hipStreamSynchronize(s));
  *n_kept = (int64_t)*ctx->iso_host;
  return GS_OK;
}

gs_status iso_emit(Ctx* ctx, const gs_volume& vol, float iso, float keep_prob, uint64_t seed,
                   float* xyz, int64_t cap, int64_t n_kept, hipStream_t s) {
  if (n_kept > cap) {
    set_error("gs_iso_extract: %lld points do not fit the capacity of %lld", (long long)n_kept,
              (long long)cap);
    return GS_ERR_CAPACITY;
  }
  const VolDev V = vol_dev(vol, iso);
  const KeepRule r{(uint32_t)seed, (uint32_t)(seed >> 32), keep_prob};
  const IsoScratch w(ctx, vol);
  hipLaunchKernelGGL(k_iso_emit, dim3((unsigned)w.nb), dim3(kIB), 0, s, V, r, w.nvert,
                     (const uint32_t*)w.off, (const unsigned long long*)w.tile_off,
                     (const uint16_t*)w.held, xyz,
                     (long long)cap);
  GS_LAUNCHED("iso_emit");
  return GS_OK;
}

gs_status launch_raycast(Ctx* ctx, const gs_volume& vol, float iso, const gs_camera* cams, int nv,
                         float* const* images, double step, hipStream_t s) {
  const VolDev V = vol_dev(vol, iso);
  RayViews rv;
  rv.n = nv;
  int blocks = 0;
  long long pix = 0;
  for (int k = 0; k < nv; ++k) {
    RayView& r = rv.v[k];
    const gs_camera& c = cams[k];
    for (int i = 0; i < 9; ++i) r.R[i] = (double)c.R[i];
    // camera centre -R^T t
    for (int a = 0; a < 3; ++a)
      r.o[a] = -((double)c.R[0 * 3 + a] * c.t[0] + (double)c.R[1 * 3 + a] * c.t[1] +
                 (double)c.R[2 * 3 + a] * c.t[2]);
    r.fx = c.fx;
    r.fy = c.fy;
    r.cx = c.cx;
    r.cy = c.cy;
    r.W = c.width;
    r.H = c.height;
    r.img = images[k];
    // chunks of up to 8 x 8 blocks, at least 1024 of them (or single blocks): fewer leave the
    // XCDs unequal (two 1024^2 views: 2 x 2 blocks 508 us, 4 x 4 526, 8 x 8 625, single
    // blocks 578)
    r.side = 8;
    auto chunks = [&] {
      return ((c.width + 16 * r.side - 1) / (16 * r.side)) *
             ((c.height + 16 * r.side - 1) / (16 * r.side));
    };
    while (r.side > 1 && chunks() < 1024) r.side /= 2;
    blocks = std::max(blocks, (chunks() + 7) / 8 * 8 * r.side * r.side);
    pix += (long long)c.width * c.height;
  }
  const dim3 grid((unsigned)blocks, (unsigned)nv);
  const double hi[3] = {(double)vol.hi[0], (double)vol.hi[1], (double)vol.hi[2]};
  CellGrid G{};
  if (!quick_suits(vol, V, rv, G)) {
    hipLaunchKernelGGL(k_raycast<false>, grid, dim3(256), 0, s, V, rv, G, step, hi[0], hi[1],
                       hi[2]);
    GS_LAUNCHED("raycast");
    return GS_OK;
  }
  double diag = 0.0, cells = 0.0;
  for (int a = 0; a < 3; ++a) {
    diag += (hi[a] - V.lo[a]) * (hi[a] - V.lo[a]);
    cells += (double)(G.last[a] + 1) * (G.last[a] + 1);
  }
  // a stream that is being captured goes without the classes (their scratch is shared)
  const bool capturing = ctx->capturing || stream_captured(s);
  std::unique_lock<std::mutex> lk(ctx->ray_mutex, std::defer_lock);
  if (!capturing && classes_pay((double)V.nx * V.ny * V.nz, (double)pix, std::sqrt(diag) / step,
                                std::sqrt(cells))) {
    lk.lock();
    if (build_grid(ctx, V, G, s))
      GS_LAUNCHED("cell_class");
    else
      lk.unlock();
  }
  hipLaunchKernelGGL(k_raycast<true>, grid, dim3(256), 0, s, V, rv, G, step, hi[0], hi[1], hi[2]);
  GS_LAUNCHED("raycast");
  if (G.fine != nullptr) GS_HIP(hipEventRecord(ctx->ray_use, s));
  return GS_OK;
}

}  // namespace isogs
