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
// Ray-cast: one thread per pixel, all arithmetic in float64 (the FP64 vector
// rate equals the non-packed FP32 rate here, and float64 keeps the marching
// and bisection decisions those of any float64 evaluation): slab clipping to
// the box, samples at t_near + k step of the trilinear interpolant, the first
// rise through iso, ten bisections, headlight shading with the interpolant's
// gradient.
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
};

__device__ inline IsoBlock iso_block(const VolDev& V, long long nvert, long long chunk) {
  IsoBlock b;
  b.base = chunk * kIG;
  const long long st[3] = {0, V.nx, V.nx * V.ny};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const long long l = nvert - b.base - st[a];
    b.left[a] = l <= 0 ? 0u : (uint32_t)min(l, (long long)(2 * kIG));
    b.p[a] = V.v + (l > 0 ? b.base + st[a] : 0);
  }
  return b;
}

// Position of vertex vid on the grid (sides up to 2^20).
__device__ inline void vertex_ijk(const VolDev& V, long long vid, uint32_t& i, uint32_t& j,
                                  uint32_t& k) {
  const uint32_t nx = (uint32_t)V.nx, ny = (uint32_t)V.ny;
  if (V.nx * V.ny * V.nz <= 0xffffffffll) {
    const uint32_t u = (uint32_t)vid, jk = u / nx;
    i = u - jk * nx;
    k = jk / ny;
    j = jk - k * ny;
  } else {
    const long long jk = vid / V.nx;
    i = (uint32_t)(vid - jk * V.nx);
    k = (uint32_t)(jk / V.ny);
    j = (uint32_t)(jk - (long long)k * V.ny);
  }
}

// The kept crossings among the edges of this lane's four consecutive vertices o .. o + 3
// of the block: bit 3 s + x for the edge of vertex o + s along axis x (the canonical
// order); the values they need in a (vertex), b (+y) and c (+z), a[4] the vertex after
// the last.  Returns 0 for the whole wave, without looking at positions, when no edge of
// its 256 vertices crosses (nearly all waves: a surface meets few of them).  The sign
// tests compare the float32 values with iso directly, strictly (exact; NaN never
// crosses); every test is one comparison whose result is a wave mask, and the rest is
// scalar mask arithmetic.
__device__ inline uint32_t edge_flags(const VolDev& V, const KeepRule& r, const IsoBlock& B,
                                      uint32_t o, float (&a)[5], float (&b)[4], float (&c)[4]) {
  if (B.left[2] >= kIG) {  // the whole block and its neighbours are in the volume
    load4(B.p[0], o, a);
    a[4] = B.p[0][o + 4];
    load4(B.p[1], o, b);
    load4(B.p[2], o, c);
  } else {  // clamped addresses; what lies past the end is masked below
#pragma unroll
    for (int s = 0; s < 5; ++s) a[s] = B.p[0][min(o + s, B.left[0] - 1)];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      b[s] = B.p[1][min(o + s, max(B.left[1], 1u) - 1)];
      c[s] = B.p[2][min(o + s, max(B.left[2], 1u) - 1)];
    }
  }
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
  // edges of the grid only: not past the last vertex of a row, column or the volume
  const uint32_t nx = (uint32_t)V.nx, ny = (uint32_t)V.ny;
  uint32_t i, j, k;
  vertex_ijk(V, B.base + o, i, j, k);
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
  if (r.prob < 1.0f) {
    const unsigned long long e0 = 3ull * (unsigned long long)(B.base + o);
    for (uint32_t left = f; left != 0; left &= left - 1) {
      const int e = __builtin_ctz(left);
      if (!kept(r, e0 + e)) f &= ~(1u << e);
    }
  }
  return f;
}

constexpr int kIS = kIV / 4;  // steps of four vertices per thread

// Bound by the read of the volume (4 B per vertex; the neighbours come from L1 and L2):
// 144 us for 512^3 vertices (3.7 TB/s), where one vertex per lane with 64-bit positions
// for every vertex and blocks in dispatch order took 435 us.
__global__ __launch_bounds__(kIB) void k_iso_count(VolDev V, KeepRule r, long long nvert,
                                                    uint32_t* __restrict__ tot) {
  __shared__ uint32_t sh[kIW];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long long chunk = iso_chunk();
  const IsoBlock B = iso_block(V, nvert, chunk);
  uint32_t n = 0;
#pragma unroll
  for (int q = 0; q < kIS; ++q) {
    float a[5], b[4], c[4];
    n += (uint32_t)__popc(edge_flags(V, r, B, 4u * (q * kIB + threadIdx.x), a, b, c));
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d, 64);
  if (lane == 0) sh[w] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int q = 0; q < kIW; ++q) t += sh[q];
    tot[chunk] = t;
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

// Blocks without a crossing leave at once.  The others form the same flags again; every
// wave lists its crossings (vertex and axis) in LDS in order and then takes them 64 at a
// time, so that the float64 divisions run with full waves and the points are stored
// coalesced: 195 us on a 512^3 volume with 1M crossings (each lane writing the points of
// its own vertices, axis by axis: 312 us; walking every block as well: 765 us).
__global__ __launch_bounds__(kIB) void k_iso_emit(VolDev V, KeepRule r, long long nvert,
                                                   const uint32_t* __restrict__ off,
                                                   const unsigned long long* __restrict__ tile_off,
                                                   float* __restrict__ xyz, long long cap) {
  __shared__ uint32_t sh[kIS][kIW];
  __shared__ uint16_t list[kIW][kIS * 64 * 12];  // 4 x vertex in the block + axis
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const long long chunk = iso_chunk(), next = chunk + 1;
  const unsigned long long base = tile_off[chunk / kTile] + off[chunk];
  const unsigned long long end =
      next < (long long)gridDim.x && next % kTile != 0 ? tile_off[chunk / kTile] + off[next]
                                                       : tile_off[chunk / kTile + 1];
  if (base == end) return;
  const IsoBlock B = iso_block(V, nvert, chunk);
  uint32_t first[kIS + 1];  // this wave's list: start of every step's crossings
  first[0] = 0;
#pragma unroll
  for (int q = 0; q < kIS; ++q) {
    const uint32_t ov = 4u * (q * kIB + threadIdx.x);
    float a[5], b[4], c[4];
    const uint32_t f = edge_flags(V, r, B, ov, a, b, c);
    uint32_t n = 0;
    if (__builtin_amdgcn_ballot_w64(f != 0) != 0) {
      const uint32_t own = (uint32_t)__popc(f);
      uint32_t inc = own;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)inc, d, 64);
        if (lane >= d) inc += y;
      }
      n = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
      uint32_t at = first[q] + inc - own;
      for (uint32_t left = f; left != 0; left &= left - 1) {
        const uint32_t e = (uint32_t)__builtin_ctz(left), s = e / 3;
        list[w][at++] = (uint16_t)(4 * (ov + s) + (e - 3 * s));
      }
    }
    first[q + 1] = first[q] + n;
    if (lane == 0) sh[q][w] = n;
  }
  __syncthreads();
  // points of step q precede those of step q + 1; inside a step the waves are in order:
  // shift[q] takes a position in this wave's list to its place among the block's points
  uint32_t shift[kIS], before = 0;
#pragma unroll
  for (int q = 0; q < kIS; ++q) {
    uint32_t pre = 0, all = 0;
#pragma unroll
    for (int x = 0; x < kIW; ++x) {
      if (x < w) pre += sh[q][x];
      all += sh[q][x];
    }
    shift[q] = before + pre - first[q];
    before += all;
  }
  for (uint32_t t = lane; t < first[kIS]; t += 64) {
    const uint32_t code = list[w][t];
    const int x = (int)(code & 3u);
    const long long vid = B.base + (code >> 2);
    const float v0 = V.v[vid];
    const float v1 = V.v[vid + (x == 0 ? 1 : (x == 1 ? V.nx : V.nx * V.ny))];
    uint32_t place = shift[0];
#pragma unroll
    for (int q = 1; q < kIS; ++q) place = t >= first[q] ? shift[q] : place;
    uint32_t i, j, k;
    vertex_ijk(V, vid, i, j, k);
    // t = a / (a - b), a = v0 - iso, b = v1 - iso (both exact in float64)
    const double u = ((double)v0 - (double)V.iso) / ((double)v0 - (double)v1);
    const double px = V.lo[0] + (double)i * V.h[0], py = V.lo[1] + (double)j * V.h[1],
                 pz = V.lo[2] + (double)k * V.h[2];
    const long long o = (long long)(base + (uint32_t)(place + t));
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
  float* img;
};

struct RayViews {
  RayView v[kMaxViews];
  int n;
};

// Trilinear value (and optionally gradient) of the volume at p.
__device__ inline double trilerp(const VolDev& V, const double* p, double* g) {
  double u[3];
  long long i0[3];
  double fr[3];
  const long long n[3] = {V.nx, V.ny, V.nz};
  for (int a = 0; a < 3; ++a) {
    u[a] = (p[a] - V.lo[a]) / V.h[a];
    long long i = (long long)floor(u[a]);
    i = i < 0 ? 0 : (i > n[a] - 2 ? n[a] - 2 : i);
    i0[a] = i;
    fr[a] = u[a] - (double)i;
  }
  const float* b = V.v + (i0[2] * V.ny + i0[1]) * V.nx + i0[0];
  const long long sy = V.nx, sz = V.nx * V.ny;
  const double c000 = b[0], c100 = b[1], c010 = b[sy], c110 = b[sy + 1];
  const double c001 = b[sz], c101 = b[sz + 1], c011 = b[sz + sy], c111 = b[sz + sy + 1];
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

__global__ __launch_bounds__(256) void k_raycast(VolDev V, RayViews rv, double step,
                                                 double hi0, double hi1, double hi2) {
  const RayView& c = rv.v[blockIdx.y];
  const int pix = blockIdx.x * blockDim.x + threadIdx.x;
  if (pix >= c.W * c.H) return;
  const int x = pix % c.W, y = pix / c.W;
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
  if (box && tf > tn) {
    double p[3];
    for (int a = 0; a < 3; ++a) p[a] = c.o[a] + tn * d[a];
    double f_prev = trilerp(V, p, nullptr) - (double)V.iso;
    double lo_t = 0.0, hi_t = -1.0;
    for (long long k = 1;; ++k) {
      const double tk = tn + (double)k * step;
      if (tk > tf) break;
      for (int a = 0; a < 3; ++a) p[a] = c.o[a] + tk * d[a];
      const double f = trilerp(V, p, nullptr) - (double)V.iso;
      if (f_prev < 0.0 && f >= 0.0) {
        lo_t = tn + (double)(k - 1) * step;
        hi_t = tk;
        break;
      }
      f_prev = f;
    }
    if (hi_t >= 0.0) {
      for (int it = 0; it < 10; ++it) {
        const double mid = 0.5 * (lo_t + hi_t);
        for (int a = 0; a < 3; ++a) p[a] = c.o[a] + mid * d[a];
        if (trilerp(V, p, nullptr) - (double)V.iso < 0.0)
          lo_t = mid;
        else
          hi_t = mid;
      }
      const double th = 0.5 * (lo_t + hi_t);
      for (int a = 0; a < 3; ++a) p[a] = c.o[a] + th * d[a];
      double g[3];
      (void)trilerp(V, p, g);
      const double gn = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
      const double lam = gn > 0.0 ? fabs((g[0] * d[0] + g[1] * d[1] + g[2] * d[2]) / gn) : 0.0;
      const double sh = 0.2 + 0.8 * lam;
      rgb[0] = (float)(0.85 * sh);
      rgb[1] = (float)((0.45 + 0.25 * p[2]) * sh);
      rgb[2] = (float)((0.30 + 0.25 * (p[0] + 1.0)) * sh);
    }
  }
  const size_t plane = (size_t)c.W * c.H;
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

}  // namespace

gs_status iso_extract_run(Ctx* ctx, const gs_volume& vol, float iso, float keep_prob,
                          uint64_t seed, float* xyz, int64_t cap, int64_t* n_kept,
                          hipStream_t s) {
  const VolDev V = vol_dev(vol, iso);
  const long long nvert = (long long)vol.nx * vol.ny * vol.nz;
  const long long nb = (nvert + kIG - 1) / kIG;
  KeepRule r{(uint32_t)seed, (uint32_t)(seed >> 32), keep_prob};
  // tile offsets and the grand total (64-bit), block offsets, tile totals
  const long long tiles = (nb + kTile - 1) / kTile;
  const size_t bytes = sizeof(unsigned long long) * (size_t)(tiles + 1) +
                       sizeof(uint32_t) * (size_t)(nb + tiles);
  gs_status st = buf_ensure(ctx, ctx->iso_blk, bytes, s);
  if (st != GS_OK) return st;
  if (ctx->iso_host == nullptr)
    GS_HIP(hipHostMalloc((void**)&ctx->iso_host, sizeof(unsigned long long),
                         hipHostMallocDefault));
  auto* tile_off = (unsigned long long*)ctx->iso_blk.p;
  auto* off = (uint32_t*)(tile_off + tiles + 1);
  auto* tile_tot = off + nb;
  hipLaunchKernelGGL(k_iso_count, dim3((unsigned)nb), dim3(kIB), 0, s, V, r, nvert, off);
  GS_LAUNCHED("iso_count");
  hipLaunchKernelGGL(k_iso_scan_tile, dim3((unsigned)tiles), dim3(1024), 0, s, off, nb, tile_tot);
  GS_LAUNCHED("iso_scan_tile");
  hipLaunchKernelGGL(k_iso_scan_top, dim3(1), dim3(1024), 0, s, (const uint32_t*)tile_tot,
                     (int)tiles, tile_off);
  GS_LAUNCHED("iso_scan_top");
  GS_HIP(hipMemcpyAsync(ctx->iso_host, tile_off + tiles, sizeof(unsigned long long),
                        hipMemcpyDeviceToHost, s));
  GS_HIP(hipStreamSynchronize(s));
  *n_kept = (int64_t)*ctx->iso_host;
  if (xyz == nullptr) return GS_OK;
  if (*n_kept > cap) {
    set_error("gs_iso_extract: %lld points do not fit the capacity of %lld",
              (long long)*n_kept, (long long)cap);
    return GS_ERR_CAPACITY;
  }
  hipLaunchKernelGGL(k_iso_emit, dim3((unsigned)nb), dim3(kIB), 0, s, V, r, nvert,
                     (const uint32_t*)off, (const unsigned long long*)tile_off, xyz,
                     (long long)cap);
  GS_LAUNCHED("iso_emit");
  return GS_OK;
}

gs_status launch_raycast(const gs_volume& vol, float iso, const gs_camera* cams, int nv,
                         float* const* images, double step, hipStream_t s) {
  const VolDev V = vol_dev(vol, iso);
  RayViews rv;
  rv.n = nv;
  int max_pix = 0;
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
    if (c.width * c.height > max_pix) max_pix = c.width * c.height;
  }
  const dim3 grid((unsigned)((max_pix + 255) / 256), (unsigned)nv);
  hipLaunchKernelGGL(k_raycast, grid, dim3(256), 0, s, V, rv, step, (double)vol.hi[0],
                     (double)vol.hi[1], (double)vol.hi[2]);
  GS_LAUNCHED("raycast");
  return GS_OK;
}

}  // namespace isogs
