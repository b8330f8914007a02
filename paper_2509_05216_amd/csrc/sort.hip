// Tile binning: exclusive scan of per-Gaussian tile counts, record emission,
// a stable LSD radix sort of (u32 key, u32 value) pairs, and per-tile ranges.
//
// Order contract: records sorted by the 64-bit key (tile << 32) | depth bits,
// ties by (view * N + Gaussian index).  The LSD sort of that key is split in
// two: the 32 low (depth) digits are sorted once per (view, Gaussian) — every
// record of a Gaussian shares its depth — and records are then emitted in that
// order, so only the tile digits are sorted over the K records.  The result is
// the same permutation an LSD sort of the full 64-bit key over the emitted
// records gives, at a fraction of the traffic.
//
// Radix passes use 8-bit digits, 256 threads (4 waves of 64) and 16 keys per
// thread per block (4 in small sorts); 9 or 10 bits and 512 threads where that saves a
// pass.  Stable ranking inside a block uses wave ballots: for each item slot the lanes
// holding the same digit are found with a ballot per bit, all of them read the wave's LDS
// counter of the digit, the last adds their number, and lanes take their rank from the
// count of lower peer lanes.
#include <algorithm>

#include "internal.h"

namespace isogs {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kItems = 16;
constexpr int kChunk = kThreads * kItems;  // 4096 elements per block
constexpr int kRadix = 256;

__device__ inline uint32_t load_n(uint32_t n_max, const uint32_t* d_n) {
  if (d_n == nullptr) return n_max;
  const uint32_t c = *d_n;
  return c < n_max ? c : n_max;
}

__device__ inline uint64_t lanemask_lt() {
  const int lane = __lane_id();
  return (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
}

// Orders this wave's LDS accesses before and after it among its lanes.  LDS serves a wave's
// accesses in order, so this costs no instruction; it keeps the compiler from answering a
// lane's read from what that lane itself wrote last.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- block scan
// Exclusive scan of one u64 value per thread over a block of WAVES waves.
template <int WAVES = kWaves>
__device__ inline uint64_t block_exclusive_scan(uint64_t x, uint64_t* sh_waves, uint64_t& total) {
  const int lane = __lane_id();
  const int wave = threadIdx.x / 64;
  uint64_t inc = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(inc, d, 64);
    if (lane >= d) inc += y;
  }
  if (lane == 63) sh_waves[wave] = inc;
  __syncthreads();
  uint64_t before = 0;
  total = 0;
  for (int w = 0; w < WAVES; ++w) {
    const uint64_t s = sh_waves[w];
    if (w < wave) before += s;
    total += s;
  }
  __syncthreads();
  return before + inc - x;
}


struct ArrayIn {
  const uint32_t* a;
  __device__ uint32_t operator()(uint32_t i) const { return a[i]; }
};

template <class F>
__global__ __launch_bounds__(kThreads) void k_scan_reduce(F f, uint32_t n, uint64_t* partial) {
  __shared__ uint64_t sw[kWaves];
  const uint32_t base = blockIdx.x * (uint32_t)kChunk;
  uint64_t s = 0;
#pragma unroll 4
  for (int j = 0; j < kItems; ++j) {
    const uint32_t i = base + j * kThreads + threadIdx.x;
    if (i < n) s += f(i);
  }
  uint64_t total;
  block_exclusive_scan(s, sw, total);
  if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// Exclusive scan, in place, of the nb block totals by one block (each thread a
// contiguous run); the grand total goes to d_total when given.  Used when there
// are too many blocks for the down-sweep to sum its predecessors itself.
__global__ __launch_bounds__(kThreads) void k_scan_partials(uint64_t* partial, uint32_t nb,
                                                            uint64_t* d_total) {
  __shared__ uint64_t sw[kWaves];
  const uint32_t per = (nb + kThreads - 1) / kThreads;
  const uint32_t lo = min(nb, threadIdx.x * per), hi = min(nb, lo + per);
  uint64_t s = 0;
  for (uint32_t j = lo; j < hi; ++j) s += partial[j];
  uint64_t total;
  uint64_t run = block_exclusive_scan(s, sw, total);
  for (uint32_t j = lo; j < hi; ++j) {
    const uint64_t v = partial[j];
    partial[j] = run;
    run += v;
  }
  if (d_total != nullptr && threadIdx.x == 0) *d_total = total;
}

// Down-sweep.  With few blocks each forms its carry-in by summing the totals of
// the blocks before it (read from L2), so no separate scan of the totals is
// launched, and the last block writes the grand total when d_total is given
// (`per` totals stand for one block's elements); with many (prescanned), k_scan_partials
// has already turned the totals into the carries and written the grand total.
template <class F>
__global__ __launch_bounds__(kThreads) void k_scan_down(F f, uint32_t n, const uint64_t* partial,
                                                        uint32_t* out, uint64_t* d_total,
                                                        int prescanned, uint32_t per) {
  __shared__ uint64_t sw[kWaves];
  // striped (coalesced) loads and stores, transposed through LDS so that each
  // thread scans kItems consecutive elements; one pad word per 32 avoids bank conflicts
  __shared__ uint32_t buf[kChunk + kChunk / 32];
  const uint32_t base = blockIdx.x * (uint32_t)kChunk;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    const uint32_t i = base + p;
    buf[p + (p >> 5)] = (i < n) ? f(i) : 0u;
  }
  __syncthreads();
  uint32_t v[kItems];
  uint64_t s = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t p = threadIdx.x * kItems + j;
    v[j] = buf[p + (p >> 5)];
    s += v[j];
  }
  uint64_t ctot;
  if (prescanned) {
    ctot = partial[blockIdx.x];
  } else {
    uint64_t carry = 0;
    for (uint32_t b = threadIdx.x; b < blockIdx.x * per; b += kThreads) carry += partial[b];
    block_exclusive_scan(carry, sw, ctot);  // ctot: the sum over all threads
  }
  uint64_t total;
  uint64_t run = block_exclusive_scan(s, sw, total) + ctot;
  if (!prescanned && d_total != nullptr && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
    *d_total = ctot + total;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t p = threadIdx.x * kItems + j;
    buf[p + (p >> 5)] = (uint32_t)run;
    run += v[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint32_t p = j * kThreads + threadIdx.x;
    const uint32_t i = base + p;
    if (i < n) out[i] = buf[p + (p >> 5)];
  }
}

// Chunk of this block, of nchunks that hold keys (blocks from nchunks on have none).
// Workgroups go to the eight XCDs in turn, so consecutive block indices land in
// different L2s; this bijection gives each XCD a contiguous run of chunks instead (the
// last nchunks % 8 keep their place).  nchunks follows the number of keys there are, which
// may be on the device, and not the capacity that the grid is launched for: with runs cut
// from the capacity, 216M records in a capacity of 270M were sorted by 6.4 of the
// XCDs (scatter passes 429 -> 405 us on average).
__device__ inline uint32_t xcd_chunk(uint32_t nchunks) {
  const uint32_t n8 = nchunks / 8;
  return blockIdx.x < 8 * n8 ? (blockIdx.x % 8) * n8 + blockIdx.x / 8 : blockIdx.x;
}

// The one random gather of the rectangles: the tile count of every (view,
// Gaussian) entry in depth order, and the rectangles themselves in that order
// for the emission.  Neighbours in memory are often thousands of entries apart in depth,
// not millions: with a contiguous run of entries per XCD their line is still in its L2
// (4M entries 57 -> 39 us, 16M 238 -> 182, 36M 436 -> 426).
__global__ __launch_bounds__(256) void k_counts(const uint32_t* __restrict__ sidx,
                                                const uint2* __restrict__ rect, uint32_t n,
                                                uint32_t* __restrict__ counts,
                                                uint32_t* __restrict__ srx,
                                                uint32_t* __restrict__ sry,
                                                uint64_t* __restrict__ partial) {
  const uint32_t block = xcd_chunk(gridDim.x);
  const uint32_t i = block * blockDim.x + threadIdx.x;
  uint32_t m = 0;
  if (i < n) {
    const uint2 r = rect[sidx[i]];
    srx[i] = r.x;
    sry[i] = r.y;
    const int x0 = (int)(r.x & 0xffffu), y0 = (int)(r.x >> 16);
    const int x1 = (int)(r.y & 0xffffu), y1 = (int)(r.y >> 16);
    m = (x1 < x0 || y1 < y0) ? 0u : (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1));
    counts[i] = m;
  }
  if (partial == nullptr) return;
  __shared__ uint64_t sw[kWaves];
  uint64_t total;
  block_exclusive_scan(m, sw, total);
  if (threadIdx.x == 0) partial[block] = total;
}

// ---------------------------------------------------------------- radix sort
// Shape of a pass: BITS per digit, blocks of THREADS threads with ITEMS keys each.
template <int BITS_, int THREADS_, int ITEMS_>
struct Pass {
  static constexpr int BITS = BITS_, THREADS = THREADS_, ITEMS = ITEMS_;
  static constexpr int RADIX = 1 << BITS, WAVES = THREADS / 64, CHUNK = THREADS * ITEMS;
  static constexpr int PER = RADIX / THREADS;  // digits of a thread in the offset scan
  static_assert(RADIX % THREADS == 0, "whole digits per thread");
  static_assert(CHUNK < 65536, "local places fit 16 bits");
  __host__ __device__ static uint32_t chunks(uint32_t n) {
    return n / CHUNK + (n % CHUNK != 0 ? 1u : 0u);
  }
};
using PassSmall = Pass<8, kThreads, 4>;
using PassLarge = Pass<8, kThreads, kItems>;
using PassWide9 = Pass<9, 512, kItems>;
using PassWide10 = Pass<10, 512, kItems>;

// Uint4 words of a digit's row that hold nchunks counts (zeros follow the last count).
__host__ __device__ inline uint32_t row_quads(uint32_t nchunks) { return (nchunks + 3) / 4; }

// Four keys from a multiple of four on.
__device__ inline uint4 load4(const uint32_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ inline uint4 load4(const uint16_t* p) {
  const uint2 q = *reinterpret_cast<const uint2*>(p);
  return make_uint4(q.x & 0xffffu, q.x >> 16, q.y & 0xffffu, q.y >> 16);
}

template <class P, class K>
__global__ __launch_bounds__(P::THREADS) void k_radix_hist(const K* __restrict__ keys,
                                                           uint32_t n_max, const uint32_t* d_n,
                                                           int shift, uint32_t stride,
                                                           uint32_t* __restrict__ hist) {
  constexpr int ITEMS = P::ITEMS;
  constexpr int COPIES = P::BITS == 8 ? P::WAVES : 2;  // of the counts, against collisions
  __shared__ uint32_t h[COPIES][P::RADIX];
  const int wave = threadIdx.x / 64, lane = __lane_id();
  uint32_t* const hw = h[wave % COPIES];
  for (int d = threadIdx.x; d < COPIES * P::RADIX; d += P::THREADS) (&h[0][0])[d] = 0;
  __syncthreads();
  const uint32_t n = load_n(n_max, d_n);
  // chunk of this block: XCD-contiguous as in k_radix_scatter, so that the
  // counts of neighbouring chunks, adjacent in every digit's row of the table,
  // are written through the same L2
  const uint32_t nchunks = P::chunks(n);
  const uint32_t chunk = xcd_chunk(nchunks);
  if (chunk >= nchunks) return;  // no keys (uniform)
  // the wave's keys four at a time, all issued before the
  // counting (the order of counting does not matter)
  const uint32_t base = chunk * (uint32_t)P::CHUNK + wave * 64 * ITEMS;
  uint4 q[ITEMS / 4];
#pragma unroll
  for (int j = 0; j < ITEMS / 4; ++j) {
    const uint32_t i = base + 4u * (j * 64 + lane);
    if (i + 4 <= n) {
      q[j] = load4(keys + i);
    } else {  // tail: absent keys marked ~0 and skipped below
      q[j].x = i < n ? keys[i] : ~0u;
      q[j].y = i + 1 < n ? keys[i + 1] : ~0u;
      q[j].z = i + 2 < n ? keys[i + 2] : ~0u;
      q[j].w = ~0u;
    }
  }
  // A digit shared by many lanes of the wave (the high bytes of depths, the
  // tile rows of neighbouring records) would serialise their LDS atomics on one
  // word: the lanes holding lane 0's digit, and those holding the digit of the
  // first lane left, are counted by one atomic each; the rest add one apiece.
#pragma unroll
  for (int j = 0; j < ITEMS / 4; ++j) {
    const uint32_t i = base + 4u * (j * 64 + lane);
    const uint32_t kk[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = i + u < n;
      const uint32_t d = __builtin_amdgcn_ubfe(kk[u], shift, P::BITS);
      const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
      const uint64_t m0 = __builtin_amdgcn_ballot_w64(ok && d == d0);
      const uint64_t r0 = __builtin_amdgcn_ballot_w64(ok && d != d0);
      uint32_t d1 = P::RADIX;  // no digit
      uint64_t m1 = 0;
      if (r0 != 0) {
        d1 = (uint32_t)__builtin_amdgcn_readlane((int)d, __builtin_ctzll(r0));
        m1 = __builtin_amdgcn_ballot_w64(ok && d == d1);
      }
      if (lane == 0) {
        if (m0 != 0) atomicAdd(&hw[d0], (uint32_t)__popcll(m0));
        if (m1 != 0) atomicAdd(&hw[d1], (uint32_t)__popcll(m1));
      }
      if (ok && d != d0 && d != d1) atomicAdd(&hw[d], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < P::RADIX; d += P::THREADS) {
    uint32_t s = 0;
#pragma unroll
    for (int w = 0; w < COPIES; ++w) s += h[w][d];
    uint32_t* row = hist + (size_t)d * stride;
    row[chunk] = s;
    if (chunk == nchunks - 1)
      for (uint32_t c = nchunks; c < row_quads(nchunks) * 4; ++c) row[c] = 0u;
  }
}

// Rows of the digit table: row d (stride words, a multiple of four) holds digit d's count
// in every chunk that has keys, and the totals of the rows follow the table.  One block per
// digit turns its row into the exclusive prefix over the chunks and writes the total; the
// scatter itself scans the totals.  One launch instead of the two of a scan over the whole
// table (passes over 16M and 42M keys: 7 us on average instead of 18).
template <class P>
__global__ __launch_bounds__(kThreads) void k_digit_rows(uint32_t* __restrict__ hist,
                                                         uint32_t stride, uint32_t n_max,
                                                         const uint32_t* d_n) {
  __shared__ uint32_t sw[2][kWaves];
  uint4* row = reinterpret_cast<uint4*>(hist + (size_t)blockIdx.x * stride);
  const uint32_t quads = row_quads(P::chunks(load_n(n_max, d_n)));
  const int lane = __lane_id(), wave = threadIdx.x / 64;
  uint32_t carry = 0;
  int buf = 0;
  for (uint32_t q0 = 0; q0 < quads; q0 += kThreads * 4, buf ^= 1) {  // 4096 counts a round
    uint4 v[4];
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t q = q0 + threadIdx.x * 4 + j;
      v[j] = q < quads ? row[q] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) sum += v[j].x + v[j].y + v[j].z + v[j].w;
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)inc, d, 64);
      if (lane >= d) inc += y;
    }
    if (lane == 63) sw[buf][wave] = inc;
    __syncthreads();  // one barrier a round: the next round's sums go to the other buffer
    uint32_t run = carry + inc - sum;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t t = sw[buf][w];
      if (w < wave) run += t;
      carry += t;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint4 o;
      o.x = run;
      o.y = o.x + v[j].x;
      o.z = o.y + v[j].y;
      o.w = o.z + v[j].z;
      run = o.w + v[j].w;
      const uint32_t q = q0 + threadIdx.x * 4 + j;
      if (q < quads) row[q] = o;
    }
  }
  if (threadIdx.x == 0) hist[(size_t)P::RADIX * stride + blockIdx.x] = carry;
}

// This chunk's prefix in row d, and the row's total: from the scanned table and its
// totals, or (RAW, small tables) summed here from the counts.
template <bool RAW, int RADIX>
__device__ inline void digit_row(const uint32_t* __restrict__ hist, uint32_t stride,
                                 uint32_t nchunks, uint32_t chunk, int d, uint32_t& before, uint32_t& total) {
  if constexpr (!RAW) {
    before = hist[(size_t)d * stride + chunk];
    total = hist[(size_t)RADIX * stride + d];
    return;
  }
  const uint4* row = reinterpret_cast<const uint4*>(hist + (size_t)d * stride);
  before = total = 0;
  for (uint32_t q = 0; q < row_quads(nchunks); ++q) {
    const uint4 v = row[q];
    const uint32_t c = 4 * q;
    total += v.x + v.y + v.z + v.w;
    before += (c < chunk ? v.x : 0u) + (c + 1 < chunk ? v.y : 0u) + (c + 2 < chunk ? v.z : 0u) +
              (c + 3 < chunk ? v.w : 0u);
  }
}

// One pass of the stable LSD sort.  Each block ranks its elements by
// digit (wave ballots, stable), places them in LDS in block-local digit order,
// and writes them out so that consecutive threads store consecutive addresses
// of one digit's run: the global writes are coalesced.  Large passes are bound by memory
// (16 bytes a pair): 216M records of two 4096^2 views move at 4.5 TB/s (8 bits) and 4.0
// (10 bits).  Ranking took more issue slots than that before it was cut from about 150 to
// 75 instructions a key (one three-operand instruction per bit and half, no leader
// election or shuffle, no test whether a key is there): 8-bit passes over 4M to 22M
// pairs 29.3 -> 23.4 us on average, over 16M to 42M 112 -> 92.
constexpr uint32_t kAndXnor = 0xF0 & ~(0xCC ^ 0xAA);  // bitop3 table of a & ~(b ^ c)

// Ranks of a wave's keys among its keys of the same digit, in index order, on top of the
// wave's counts cnt, which they join.  Lanes with the same digit: for every bit, the ballot
// of the bit where the lane's bit is set, its complement where it is clear, on the two
// 32-bit halves (sbit: the bit sign-extended, 0 or all ones; p & ~(ballot ^ sbit) is one
// three-operand instruction).  All of them read the wave's count of the digit, and the
// last adds theirs.
template <int BITS, int ITEMS>
__device__ inline void rank_keys(const uint32_t (&key)[ITEMS], int shift, uint16_t* cnt,
                                 uint32_t (&rank)[ITEMS]) {
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const uint32_t d = __builtin_amdgcn_ubfe(key[j], shift, BITS);
    uint32_t plo = ~0u, phi = ~0u;
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const uint32_t sbit = (uint32_t)__builtin_amdgcn_sbfe((int)key[j], shift + b, 1);
      const uint64_t bb = __builtin_amdgcn_ballot_w64(sbit != 0);
      plo = __builtin_amdgcn_bitop3_b32(plo, (uint32_t)bb, sbit, kAndXnor);
      phi = __builtin_amdgcn_bitop3_b32(phi, (uint32_t)(bb >> 32), sbit, kAndXnor);
    }
    const uint32_t old = cnt[d];
    rank[j] = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, old));
    const uint32_t now = old + __popc(plo) + __popc(phi);
    wave_sync();  // every lane has read before the last one writes
    if (rank[j] + 1 == now) cnt[d] = (uint16_t)now;
    wave_sync();
  }
}

template <bool RAW, class P, class K>
__global__ __launch_bounds__(P::THREADS) void k_radix_scatter(
    const K* __restrict__ kin, const uint32_t* __restrict__ vin, K* __restrict__ kout,
    uint32_t* __restrict__ vout, uint32_t n_max, const uint32_t* d_n, int shift, uint32_t stride,
    const uint32_t* __restrict__ hist) {
  constexpr int ITEMS = P::ITEMS, CHUNK = P::CHUNK;
  __shared__ uint16_t cnt[P::WAVES][P::RADIX];
  __shared__ uint32_t gofs[P::RADIX];  // global position of local index 0 of digit d's run
  __shared__ uint64_t scan_tmp[P::WAVES];
  __shared__ uint32_t stage[CHUNK];
  const int wave = threadIdx.x / 64, lane = __lane_id();
  for (int d = threadIdx.x; d < P::WAVES * P::RADIX; d += P::THREADS) (&cnt[0][0])[d] = 0;
  const uint32_t n = load_n(n_max, d_n);
  // the runs that neighbouring chunks write for one digit, adjacent in the
  // output, meet in the same L2, and the cache lines they share are written
  // back whole
  const uint32_t nchunks = P::chunks(n);
  const uint32_t chunk = xcd_chunk(nchunks);
  if (chunk >= nchunks) return;  // no keys (uniform)
  const uint32_t nloc = min((uint32_t)CHUNK, n - chunk * (uint32_t)CHUNK);
  // this thread's digits: their keys in earlier chunks, and in all
  uint32_t before[P::PER], total_d[P::PER];
#pragma unroll
  for (int u = 0; u < P::PER; ++u)
    digit_row<RAW, P::RADIX>(hist, stride, nchunks, chunk, threadIdx.x * P::PER + u, before[u],
                             total_d[u]);
  // Absent keys of the last chunk are all ones: the last digit, and last of their block (their
  // indices are its highest), so they take local places from nloc on, which are not
  // written out, and nothing below asks whether a key is there.
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
  const uint32_t first = chunk * (uint32_t)CHUNK + wave * 64 * ITEMS + lane;
  if (nloc == (uint32_t)CHUNK) {
    const K* kp = kin + first;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) key[j] = kp[j * 64];
    if (vin != nullptr) {
      const uint32_t* vp = vin + first;
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) val[j] = vp[j * 64];
    } else {
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) val[j] = first + j * 64;
    }
  } else {
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const uint32_t i = first + j * 64;
      key[j] = i < n ? kin[i] : ~0u;
      val[j] = i < n ? (vin != nullptr ? vin[i] : i) : 0u;
    }
  }
  __syncthreads();
  rank_keys<P::BITS, ITEMS>(key, shift, cnt[wave], rank);
  __syncthreads();
  {
    // the block-local start of this thread's digits in every wave, and their global
    // position (unsigned wrap-around is intended in gofs - start)
    const int d0 = threadIdx.x * P::PER;
    uint32_t run[P::PER], sum = 0;
    uint64_t all = 0;
#pragma unroll
    for (int u = 0; u < P::PER; ++u) {
      run[u] = 0;
#pragma unroll
      for (int w = 0; w < P::WAVES; ++w) run[u] += cnt[w][d0 + u];
      sum += run[u];
      all += total_d[u];
    }
    // one scan for both: this block's keys of lower digits (at most CHUNK) in the low
    // 16 bits, all chunks' keys of lower digits above them
    uint64_t total;
    const uint64_t low = block_exclusive_scan<P::WAVES>((all << 16) | sum, scan_tmp, total);
    uint32_t start = (uint32_t)low & 0xffffu, g = (uint32_t)(low >> 16);
#pragma unroll
    for (int u = 0; u < P::PER; ++u) {
      gofs[d0 + u] = g + before[u] - start;
      g += total_d[u];
#pragma unroll
      for (int w = 0; w < P::WAVES; ++w) {
        const uint32_t c = cnt[w][d0 + u];
        cnt[w][d0 + u] = (uint16_t)start;
        start += c;
      }
    }
  }
  __syncthreads();
  // keys, then values, through the one staging array (half the memory of both at once:
  // more blocks resident)
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    rank[j] += cnt[wave][__builtin_amdgcn_ubfe(key[j], shift, P::BITS)];
    stage[rank[j]] = key[j];
  }
  __syncthreads();
  uint32_t pos[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const uint32_t t = j * P::THREADS + threadIdx.x;
    const uint32_t k = stage[t];
    pos[j] = gofs[__builtin_amdgcn_ubfe(k, shift, P::BITS)] + t;
    if (t < nloc) kout[pos[j]] = (K)k;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) stage[rank[j]] = val[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const uint32_t t = j * P::THREADS + threadIdx.x;
    if (t < nloc) vout[pos[j]] = stage[t];
  }
}

// ---------------------------------------------------------------- few entries
// Depth order of few (view, Gaussian) entries by counting: an entry's place is the number
// of entries with a smaller key, or the same key and a smaller index.  A block places 64
// entries (one per lane); its sixteen waves each count over a sixteenth of the keys, which
// are uniform and come by scalar loads.  The entry, its rectangle and its tile count then go
// straight to their place.  Two instructions a pair and n^2 pairs, but up to one block per
// CU less than the latency of four sorting passes, the gather and the scans (eleven
// launches, these two): whole forward pass of 1000 Gaussians at 256^2 113 -> 65 us, 4000
// 115 -> 77, 12000 125 -> 106, 16384 205 to 220 -> 181.  (All in one block with the keys in
// registers: 73, 81, 130, 192; keys from LDS, or a ballot and a scalar bit count per 64
// pairs: 21 and 22 us instead of 18 for the counting of 10k.)
constexpr int kRankWaves = 16;
constexpr uint32_t kFewEntries = 16384;  // 256 blocks of 64

__global__ __launch_bounds__(64 * kRankWaves) void k_rank_entries(
    const uint32_t* __restrict__ dkey, const uint2* __restrict__ rect, uint32_t n,
    uint32_t* __restrict__ sidx, uint32_t* __restrict__ counts, uint32_t* __restrict__ srx,
    uint32_t* __restrict__ sry) {
  __shared__ uint32_t part[kRankWaves][64];
  const int lane = __lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  const uint32_t i0 = blockIdx.x * 64, i = i0 + lane;
  const uint32_t mine = i < n ? dkey[i] : 0u;
  const uint32_t per = (n + kRankWaves - 1) / kRankWaves;
  const uint32_t lo = min(wave * per, n), hi = min(lo + per, n);
  // before this block's entries equal keys count, after them they do not
  const uint32_t mid0 = max(lo, min(hi, i0)), mid1 = max(lo, min(hi, i0 + 64));
  uint32_t c = 0;
#pragma unroll 16
  for (uint32_t j = lo; j < mid0; ++j) c += dkey[j] <= mine ? 1u : 0u;
#pragma unroll 4
  for (uint32_t j = mid0; j < mid1; ++j) {
    const uint32_t k = dkey[j];
    c += k < mine || (k == mine && j < i) ? 1u : 0u;
  }
#pragma unroll 16
  for (uint32_t j = mid1; j < hi; ++j) c += dkey[j] < mine ? 1u : 0u;
  part[wave][lane] = c;
  __syncthreads();
  if (wave != 0 || i >= n) return;
  uint32_t place = 0;
#pragma unroll
  for (int w = 0; w < kRankWaves; ++w) place += part[w][lane];
  const uint2 r = rect[i];
  const int x0 = (int)(r.x & 0xffffu), y0 = (int)(r.x >> 16);
  const int x1 = (int)(r.y & 0xffffu), y1 = (int)(r.y >> 16);
  sidx[place] = i;
  srx[place] = r.x;
  sry[place] = r.y;
  counts[place] = (x1 < x0 || y1 < y0) ? 0u : (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1));
}

// Their record offsets (counts, in place), the total, and the touched entries' number, by
// one block: sixteen consecutive entries a thread.
__global__ __launch_bounds__(1024) void k_few_offsets(const uint32_t* __restrict__ dkey,
                                                      uint32_t n, uint32_t* __restrict__ counts,
                                                      uint32_t* __restrict__ visible,
                                                      uint64_t* __restrict__ total) {
  static_assert(kFewEntries == 1024 * 16, "sixteen entries a thread");
  __shared__ uint64_t tmp[16];
  const uint32_t i0 = threadIdx.x * 16;
  uint32_t m[16], touched = 0;
  uint64_t sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t i = i0 + 4 * k;
    uint4 q = make_uint4(0u, 0u, 0u, 0u), d = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (i + 4 <= n) {
      q = load4(counts + i);
      d = load4(dkey + i);
    } else if (i < n) {
      q.x = counts[i];
      d.x = dkey[i];
      if (i + 1 < n) q.y = counts[i + 1], d.y = dkey[i + 1];
      if (i + 2 < n) q.z = counts[i + 2], d.z = dkey[i + 2];
    }
    const uint32_t qq[4] = {q.x, q.y, q.z, q.w}, dd[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      m[4 * k + u] = qq[u];
      sum += qq[u];
      touched += (dd[u] >> 24) != 0xffu ? 1u : 0u;
    }
  }
  // the number of touched entries (at most 2^14) above the records (at most 2^45)
  uint64_t all;
  const uint64_t base = block_exclusive_scan<16>(((uint64_t)touched << 48) | sum, tmp, all);
  uint32_t run = (uint32_t)base;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    if (i0 + k < n) counts[i0 + k] = run;
    run += m[k];
  }
  if (threadIdx.x == 0) {
    *total = all & ((1ull << 48) - 1);
    *visible = (uint32_t)(all >> 48);
  }
}

// ---------------------------------------------------------------- emission
// Records of every (view, Gaussian) entry in depth order: (global tile, entry)
// for each tile of its rectangle, row by row.  A wave writes its 64 entries'
// records together: lane r of a pass takes the wave's record r, so
// each pass stores 64 consecutive records and no lane idles behind a large
// rectangle.  The owning entry is the last one that starts at or before the record:
// the starts in a pass are marked in LDS, and their number up to the lane picks the
// entry, whose fields one 16-byte read brings (a search over the wave's prefix sums, seven
// dependent shuffles and six more for the fields, took 587 us instead of 511 for the 216M
// records of two 4096^2 views of 18M Gaussians, 8.8 instead of 6.5 for those of 10k).
// Bound by the stores.  An entry whose records would pass the capacity writes none and
// sets the overflow word.
template <class K>
__global__ __launch_bounds__(256) void k_emit(ViewTable vt,
                                              const uint32_t* __restrict__ sidx,
                                              const uint32_t* __restrict__ srx,
                                              const uint32_t* __restrict__ sry,
                                              const uint32_t* __restrict__ offs, uint32_t count,
                                              uint32_t cap, K* __restrict__ tkey,
                                              uint32_t* __restrict__ tval,
                                              uint32_t* overflow, uint32_t* d_K,
                                              uint2* __restrict__ ranges,
                                              uint32_t tiles, uint32_t* __restrict__ order_words) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = __lane_id();
  // the tiles' ranges start empty (k_ranges, after the sort, writes those with records)
  for (uint32_t t = i; t < tiles; t += gridDim.x * blockDim.x) ranges[t] = make_uint2(0u, 0u);
  // ... and so do the counts of the tile order (null: none is formed)
  if (order_words != nullptr)
    for (uint32_t t = i; t < (uint32_t)kOrderWords; t += gridDim.x * blockDim.x) order_words[t] = 0u;
  uint32_t need = 0, o = 0, idx = 0, key0 = 0, w = 1, tx = 1;
  bool over = false;
  if (i < count) {
    idx = sidx[i];
    const uint2 r = make_uint2(srx[i], sry[i]);  // rect[idx], gathered in depth order by k_counts
    const int x0 = (int)(r.x & 0xffffu), y0 = (int)(r.x >> 16);
    const int x1 = (int)(r.y & 0xffffu), y1 = (int)(r.y >> 16);
    if (x1 >= x0 && y1 >= y0) {
      const int v = view_of_entry(vt, idx);
      tx = (uint32_t)vt.v[v].tiles_x;
      o = offs[i];
      const uint32_t nd = (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1));
      if ((uint64_t)o + nd > cap) {
        over = true;
        if (overflow != nullptr) *overflow = 1u;
        // the records end where the first entry without room begins: nothing that was
        // not written is sorted
        if (d_K != nullptr) atomicMin(d_K, o);
      } else {
        need = nd;
        w = (uint32_t)(x1 - x0 + 1);
        key0 = (uint32_t)vt.v[v].tile_offset + (uint32_t)y0 * tx + (uint32_t)x0;
      }
    }
  }
  // no room for the later ones either (their 32-bit offsets may have wrapped)
  if ((__builtin_amdgcn_ballot_w64(over) & lanemask_lt()) != 0) need = 0;
  // exclusive prefix of the record counts over the wave, and the wave total
  uint32_t incl = need;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = (uint32_t)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += t;
  }
  const uint32_t excl = incl - need;
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  if (total == 0) return;  // (uniform in the wave; no block barrier follows)
  // the entries with records, packed: start in the wave's records, first tile, entry, and
  // the widths of rectangle and image in tiles (at most 65536: less one in 16 bits)
  __shared__ uint4 ent[kWaves][64];
  __shared__ uint32_t mark[kWaves][64];
  uint4* const e = ent[threadIdx.x / 64];
  uint32_t* const mk = mark[threadIdx.x / 64];
  const uint64_t has = __builtin_amdgcn_ballot_w64(need != 0);
  if (need != 0)
    e[__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32),
                                __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u))] =
        make_uint4(excl, key0, idx, (w - 1) | ((tx - 1) << 16));
  mk[lane] = 0;
  wave_sync();
  // the wave's records are adjacent in the output (entries without room for theirs come
  // after all those with)
  const uint32_t o0 = (uint32_t)__builtin_amdgcn_readlane((int)(o - excl), __builtin_ctzll(has));
  uint32_t before = 0;  // entries that start before this pass
  for (uint32_t base = 0, pass = 1; base < total; base += 64, ++pass) {
    // mark the records that start an entry; a record's entry is the last start up to it
    if (need != 0 && excl - base < 64u) mk[excl - base] = pass;
    wave_sync();
    const bool start = mk[lane] == pass;
    const uint64_t m = __builtin_amdgcn_ballot_w64(start);
    const uint32_t lower = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, before));
    const uint4 q = e[lower + (start ? 1u : 0u) - 1u];
    wave_sync();
    before += (uint32_t)__popcll(m);
    const uint32_t rr = base + (uint32_t)lane;
    if (rr < total) {
      const uint32_t li = rr - q.x, wl = (q.w & 0xffffu) + 1, txl = (q.w >> 16) + 1;
      // row and column of the record in its rectangle: a float reciprocal
      // estimate of li / wl is off by at most one below 2^20, so one step
      // corrects it (exact integer division beyond)
      uint32_t yy;
      if (li < (1u << 20)) {
        yy = (uint32_t)((float)li * __builtin_amdgcn_rcpf((float)wl));
        const int32_t rem = (int32_t)(li - yy * wl);
        yy = rem < 0 ? yy - 1u : (rem >= (int32_t)wl ? yy + 1u : yy);
      } else {
        yy = li / wl;
      }
      const uint32_t xx = li - yy * wl;
      tkey[o0 + rr] = (K)(q.y + yy * txl + xx);
      tval[o0 + rr] = q.z;
    }
  }
}

// Per-tile [start, end) of the sorted keys: four keys per thread (one wide
// read, plus the neighbours on either side); a run boundary sets the range.
template <class KT>
__global__ __launch_bounds__(256) void k_ranges(const KT* __restrict__ tkey, uint32_t K_max,
                                                const uint32_t* d_K, uint2* __restrict__ ranges) {
  const uint32_t k0 = 4u * (blockIdx.x * blockDim.x + threadIdx.x);
  const uint32_t K = load_n(K_max, d_K);
  if (k0 >= K) return;
  uint32_t t[6];  // keys k0 - 1 .. k0 + 4 (~0 outside [0, K): differs from every tile)
  t[0] = k0 > 0 ? tkey[k0 - 1] : ~0u;
  if (k0 + 4 <= K) {
    const uint4 q = load4(tkey + k0);
    t[1] = q.x;
    t[2] = q.y;
    t[3] = q.z;
    t[4] = q.w;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u + 1] = k0 + u < K ? tkey[k0 + u] : ~0u;
  }
  t[5] = k0 + 4 < K ? tkey[k0 + 4] : ~0u;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t k = k0 + u;
    if (k >= K) break;
    if (t[u] != t[u + 1]) ranges[t[u + 1]].x = k;
    if (t[u + 2] != t[u + 1]) ranges[t[u + 1]].y = k + 1;
  }
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, uint32_t value, size_t count) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = value;
}

__global__ void k_clamp_count(const uint64_t* __restrict__ total, uint32_t cap,
                              uint32_t* __restrict__ K, uint32_t* __restrict__ overflow) {
  const uint64_t t = *total;
  *K = t < cap ? (uint32_t)t : cap;
  if (t > cap) *overflow = 1u;
}

// Length class of a tile in the longest-first order: 255 minus a log-scale class of its
// list's length (16 classes per octave of length + 1, lengths up to 2^16 - 1
// distinguished): tiles ordered to within 1/16 of an octave are all the schedule needs.
__device__ inline uint32_t length_class(uint2 r) {
  const uint32_t x = r.y - r.x + 1u;                      // >= 1
  const uint32_t e = 31u - (uint32_t)__clz((int)x);       // floor(log2 x)
  const uint32_t m = ((x << (31u - e)) >> 27) & 15u;      // next four bits after the leading one
  const uint32_t cls = e * 16u + m;
  return 255u - (cls < 255u ? cls : 255u);
}

constexpr int kOrderItems = 4;  // tiles per thread

// Tiles per class (counts, cleared before).
__global__ __launch_bounds__(256) void k_order_count(const uint2* __restrict__ ranges,
                                                     uint32_t tiles, uint32_t* __restrict__ counts) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0u;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kOrderItems; ++j) {
    const uint32_t t = (blockIdx.x * kOrderItems + j) * 256 + threadIdx.x;
    if (t < tiles) atomicAdd(&h[length_class(ranges[t])], 1u);
  }
  __syncthreads();
  if (h[threadIdx.x] != 0u) atomicAdd(&counts[threadIdx.x], h[threadIdx.x]);
}

// Tile ids by class; the order within a class is that of the blocks' arrival (no result
// depends on it).
__global__ __launch_bounds__(256) void k_order_place(const uint2* __restrict__ ranges,
                                                     uint32_t tiles,
                                                     const uint32_t* __restrict__ counts,
                                                     uint32_t* __restrict__ cursors,
                                                     uint32_t* __restrict__ order) {
  __shared__ uint32_t h[256], first[256];
  __shared__ uint64_t sw[kWaves];
  h[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t cls[kOrderItems], rank[kOrderItems];
#pragma unroll
  for (int j = 0; j < kOrderItems; ++j) {
    const uint32_t t = (blockIdx.x * kOrderItems + j) * 256 + threadIdx.x;
    cls[j] = t < tiles ? length_class(ranges[t]) : 0u;
    rank[j] = t < tiles ? atomicAdd(&h[cls[j]], 1u) : 0u;
  }
  uint64_t total;
  const uint32_t before = (uint32_t)block_exclusive_scan(counts[threadIdx.x], sw, total);
  const uint32_t mine = h[threadIdx.x];  // (the scan's barriers come after the counting)
  first[threadIdx.x] = before + (mine != 0u ? atomicAdd(&cursors[threadIdx.x], mine) : 0u);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kOrderItems; ++j) {
    const uint32_t t = (blockIdx.x * kOrderItems + j) * 256 + threadIdx.x;
    if (t < tiles) order[first[cls[j]] + rank[j]] = t;
  }
}

template <class KT>
__global__ __launch_bounds__(256) void k_export_keys(const KT* __restrict__ tkey,
                                                     const uint32_t* __restrict__ tval,
                                                     const uint32_t* __restrict__ dkey, uint32_t K,
                                                     uint64_t* __restrict__ out) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= K) return;
  out[k] = ((uint64_t)tkey[k] << 32) | (uint64_t)dkey[tval[k]];
}

inline uint32_t nblocks_of(uint32_t n) {
  return (uint32_t)(((uint64_t)n + kChunk - 1) / kChunk);
}

// After a depth sort (positive float32 depths, untouched entries keyed 0xffffffff) the
// keys whose top byte is below 0xff are the touched entries: all but the total of the last
// pass's row 255.
template <bool RAW>
__global__ void k_visible_count(const uint32_t* __restrict__ hist, uint32_t stride,
                                uint32_t nchunks, uint32_t n, uint32_t* __restrict__ dst) {
  uint32_t before, total;
  digit_row<RAW, kRadix>(hist, stride, nchunks, 0u, 255, before, total);
  *dst = n - total;
}

// Digit tables of up to this many chunks are summed by each scatter block itself instead
// of scanned by a launch of their own (passes of 4 keys a thread: 20 chunks 5.0 us against
// 4.5 and 2.9 for the launch, 63 chunks 7.0 against 4.8 and 2.9, 147 chunks 15.4 against 4.9
// and 3.0).
constexpr uint32_t kRawChunks = 64;

inline uint32_t row_stride(uint32_t nb) { return row_quads(nb) * 4; }

// Keys per thread of a sort of n pairs: a block's chain of ranking steps sets the time of
// a small sort (histogram and scatter with 4 instead of 16 keys a thread: 600k pairs 11.1
// instead of 14.5 us, 1M 13.5 instead of 15.9), the lengths of the digit runs that it writes
// that of a large one.  Its digit table is up to four times that of sixteen keys a thread,
// which serves where there is no room for it.
constexpr uint32_t kSmallSort = 1u << 20;

// Words of a digit table: RADIX rows and their totals.
template <class P>
size_t table_words(uint32_t n) {
  return (size_t)P::RADIX * (row_stride(P::chunks(n)) + 1);
}

// Whether the sorts of n pairs take four keys a thread.
inline bool small_sort(const SortScratch& ss, uint32_t n) {
  return n <= kSmallSort && table_words<PassSmall>(n) * sizeof(uint32_t) <= ss.hist.cap;
}

// The passes of one sort, all of shape P.
template <class P, class K>
gs_status run_passes(const K* ki, const uint32_t* vi, K* const (&kb)[2],
                     uint32_t* const (&vb)[2], uint32_t n, const uint32_t* d_n, int bits,
                     uint32_t* hist, int* result_in_b, hipStream_t s) {
  const uint32_t nb = P::chunks(n), stride = row_stride(nb);
  constexpr bool kMayRaw = P::CHUNK == PassSmall::CHUNK;  // the others start at more chunks
  const bool raw = kMayRaw && nb <= kRawChunks;
  int out = 0;
  for (int shift = 0; shift < bits; shift += P::BITS) {
    hipLaunchKernelGGL((k_radix_hist<P, K>), dim3(nb), dim3(P::THREADS), 0, s, ki, n, d_n, shift,
                       stride, hist);
    GS_LAUNCHED("radix_hist");
    if (!raw) {
      hipLaunchKernelGGL(k_digit_rows<P>, dim3(P::RADIX), dim3(kThreads), 0, s, hist, stride, n,
                         d_n);
      GS_LAUNCHED("digit_rows");
    }
    auto scatter = raw ? k_radix_scatter<kMayRaw, P, K> : k_radix_scatter<false, P, K>;
    hipLaunchKernelGGL(scatter, dim3(nb), dim3(P::THREADS), 0, s, ki, vi, kb[out], vb[out], n,
                       d_n, shift, stride, (const uint32_t*)hist);
    GS_LAUNCHED("radix_scatter");
    ki = kb[out];
    vi = vb[out];
    *result_in_b = out;
    out ^= 1;
  }
  return GS_OK;
}

}  // namespace

gs_status launch_fill_u32(void* p, uint32_t value, size_t count, hipStream_t s) {
  if (count == 0) return GS_OK;
  size_t blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, (uint32_t*)p, value,
                     count);
  GS_LAUNCHED("fill_u32");
  return GS_OK;
}

// Up to this many blocks a down-sweep sums its predecessors' totals itself; above that a
// one-block scan of the totals comes first.
constexpr uint32_t kDirectBlocks = 2048;

static gs_status ensure_scratch(Ctx* ctx, SortScratch& ss, uint32_t nb, size_t hist_entries,
                                hipStream_t s) {
  gs_status st = buf_ensure(ctx, ss.partial, sizeof(uint64_t) * (size_t)(nb + 1), s, ss.prior);
  if (st != GS_OK) return st;
  st = buf_ensure(ctx, ss.total, sizeof(uint64_t) * 2, s, ss.prior);
  if (st != GS_OK) return st;
  return buf_ensure(ctx, ss.hist, sizeof(uint32_t) * (hist_entries + 1), s, ss.prior);
}

gs_status scan_tile_counts(Ctx* ctx, SortScratch& ss, const uint32_t* sidx, const uint2* rect,
                           uint32_t n, uint32_t* offs, uint32_t* srx, uint32_t* sry,
                           uint64_t* d_total, hipStream_t s) {
  const uint32_t nb = nblocks_of(n), ng = (n + 255) / 256;
  // few entries: the gather's blocks leave their totals, which the down-sweep sums (16 to
  // a block of its own); many: totals per chunk by a launch of their own (the gather runs
  // best at one entry per thread)
  const bool fused = ng <= kDirectBlocks &&
                     frame_try(ctx, ss.partial, sizeof(uint64_t) * (size_t)(ng + 1), s, ss.prior);
  const gs_status st = ensure_scratch(ctx, ss, nb, 0, s);
  if (st != GS_OK) return st;
  auto* partial = (uint64_t*)ss.partial.p;
  // gather the counts once (random rect reads), then scan them in place, coalesced
  hipLaunchKernelGGL(k_counts, dim3(ng), dim3(256), 0, s, sidx, rect, n, offs, srx, sry,
                     fused ? partial : nullptr);
  GS_LAUNCHED("counts");
  const ArrayIn f{offs};
  int pre = 0;
  if (!fused) {
    hipLaunchKernelGGL(k_scan_reduce<ArrayIn>, dim3(nb), dim3(kThreads), 0, s, f, n, partial);
    GS_LAUNCHED("scan_reduce");
    pre = nb > kDirectBlocks ? 1 : 0;
    if (pre) {
      hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kThreads), 0, s, partial, nb, d_total);
      GS_LAUNCHED("scan_partials");
    }
  }
  hipLaunchKernelGGL(k_scan_down<ArrayIn>, dim3(nb), dim3(kThreads), 0, s, f, n,
                     (const uint64_t*)partial, offs, d_total, pre,
                     fused ? (uint32_t)(kChunk / 256) : 1u);
  GS_LAUNCHED("scan_down");
  return GS_OK;
}

gs_status sort_pairs(Ctx* ctx, SortScratch& ss, const uint32_t* kin, const uint32_t* vin,
                     uint32_t* kA, uint32_t* vA, uint32_t* kB, uint32_t* vB, uint32_t n,
                     const uint32_t* d_n, int bits, int* result_in_b, hipStream_t s,
                     uint32_t* spare, size_t spare_words) {
  *result_in_b = 0;
  if (n == 0) return GS_OK;
  gs_status st = sort_reserve(ctx, ss, n, s);
  if (st != GS_OK) return st;
  auto* hist = (uint32_t*)ss.hist.p;
  uint32_t* const kb[2] = {kA, kB};
  uint32_t* const vb[2] = {vA, vB};
  if (small_sort(ss, n))
    return run_passes<PassSmall>(kin, vin, kb, vb, n, d_n, bits, hist, result_in_b, s);
  // Keys of 17 to 20 bits (more than 65536 tiles): two passes of nine or ten bits instead of
  // three of eight, where the caller's spare memory holds their table (as large as the
  // 8-bit one or twice that).  Faster from the smallest of these sorts on (forward pass of
  // 1.5M records on 69k tiles 276 -> 259 us, 1.3M on 277k tiles 459 -> 445, 7.5M 526 -> 501
  // and 658 -> 640; the two passes over 216M records 2.2 ms, the three 3.0).
  if (bits > 16 && bits <= 18 && table_words<PassWide9>(n) <= spare_words)
    return run_passes<PassWide9>(kin, vin, kb, vb, n, d_n, bits, spare, result_in_b, s);
  if (bits > 18 && bits <= 20 && table_words<PassWide10>(n) <= spare_words)
    return run_passes<PassWide10>(kin, vin, kb, vb, n, d_n, bits, spare, result_in_b, s);
  return run_passes<PassLarge>(kin, vin, kb, vb, n, d_n, bits, hist, result_in_b, s);
}

gs_status sort_pairs(Ctx* ctx, SortScratch& ss, const uint16_t* kin, const uint32_t* vin,
                     uint16_t* kA, uint32_t* vA, uint16_t* kB, uint32_t* vB, uint32_t n,
                     const uint32_t* d_n, int bits, int* result_in_b, hipStream_t s) {
  *result_in_b = 0;
  if (n == 0) return GS_OK;
  gs_status st = sort_reserve(ctx, ss, n, s);
  if (st != GS_OK) return st;
  auto* hist = (uint32_t*)ss.hist.p;
  uint16_t* const kb[2] = {kA, kB};
  uint32_t* const vb[2] = {vA, vB};
  return small_sort(ss, n)
             ? run_passes<PassSmall>(kin, vin, kb, vb, n, d_n, bits, hist, result_in_b, s)
             : run_passes<PassLarge>(kin, vin, kb, vb, n, d_n, bits, hist, result_in_b, s);
}

bool few_entries(uint32_t n) { return n >= 1 && n <= kFewEntries; }

gs_status launch_few_entries(const uint32_t* dkey, const uint2* rect, uint32_t n, uint32_t* sidx,
                             uint32_t* offs, uint32_t* srx, uint32_t* sry, uint32_t* visible,
                             uint64_t* total, hipStream_t s) {
  hipLaunchKernelGGL(k_rank_entries, dim3((n + 63) / 64), dim3(64 * kRankWaves), 0, s, dkey, rect,
                     n, sidx, offs, srx, sry);
  GS_LAUNCHED("rank_entries");
  hipLaunchKernelGGL(k_few_offsets, dim3(1), dim3(1024), 0, s, dkey, n, offs, visible, total);
  GS_LAUNCHED("few_offsets");
  return GS_OK;
}

gs_status launch_emit(const ViewTable& vt, Frame& f, const uint32_t* sidx, const uint32_t* srx,
                      const uint32_t* sry, uint32_t count, uint32_t* overflow, uint32_t* d_K,
                      hipStream_t s) {
  if (count == 0) return GS_OK;
  const size_t cap_bytes = f.tkey[0].cap < f.tval[0].cap ? f.tkey[0].cap : f.tval[0].cap;
  const uint32_t cap = (uint32_t)(cap_bytes / sizeof(uint32_t));
  auto go = [&](auto kern, auto* tkey) {
    hipLaunchKernelGGL(kern, dim3((count + 255) / 256), dim3(256), 0, s, vt, sidx, srx,
                     sry, (const uint32_t*)f.offs.p, count, cap, tkey,
                     (uint32_t*)f.tval[0].p, overflow, d_K, (uint2*)f.ranges.p,
                     (uint32_t)f.vt.total_tiles,
                     f.ordered ? (uint32_t*)f.words.p + kWordCount : nullptr);
  };
  if (f.short_keys())
    go(k_emit<uint16_t>, (uint16_t*)f.tkey[0].p);
  else
    go(k_emit<uint32_t>, (uint32_t*)f.tkey[0].p);
  GS_LAUNCHED("emit");
  return GS_OK;
}

gs_status launch_ranges(Frame& f, uint32_t n_rec, const uint32_t* d_K, hipStream_t s) {
  if (n_rec == 0) return GS_OK;
  const uint32_t quads = (n_rec + 3) / 4;
  auto go = [&](auto kern, auto* tkey) {
    hipLaunchKernelGGL(kern, dim3((quads + 255) / 256), dim3(256), 0, s, tkey, n_rec, d_K,
                       (uint2*)f.ranges.p);
  };
  if (f.short_keys())
    go(k_ranges<uint16_t>, (const uint16_t*)f.tkey[f.tkey_sel].p);
  else
    go(k_ranges<uint32_t>, (const uint32_t*)f.tkey[f.tkey_sel].p);
  GS_LAUNCHED("ranges");
  return GS_OK;
}

gs_status launch_clamp_count(const uint64_t* total, uint32_t cap, uint32_t* K,
                             uint32_t* overflow, hipStream_t s) {
  hipLaunchKernelGGL(k_clamp_count, dim3(1), dim3(1), 0, s, total, cap, K, overflow);
  GS_LAUNCHED("clamp_count");
  return GS_OK;
}

gs_status sort_reserve(Ctx* ctx, SortScratch& ss, uint32_t n, hipStream_t s) {
  // with the tables of four keys a thread (at most 1024 chunks), also of any smaller sort
  const size_t words = table_words<PassLarge>(n);
  const size_t more = std::max(words, table_words<PassSmall>(std::min(n, kSmallSort)));
  (void)frame_try(ctx, ss.hist, sizeof(uint32_t) * (more + 1), s, ss.prior);
  return ensure_scratch(ctx, ss, nblocks_of(n), words, s);
}

gs_status launch_visible_count(const SortScratch& ss, uint32_t n, uint32_t* dst, hipStream_t s) {
  if (n == 0) return launch_fill_u32(dst, 0u, 1, s);
  const bool small = small_sort(ss, n);
  const uint32_t nb = small ? PassSmall::chunks(n) : PassLarge::chunks(n);
  auto kern = small && nb <= kRawChunks ? k_visible_count<true> : k_visible_count<false>;
  hipLaunchKernelGGL(kern, dim3(1), dim3(1), 0, s, (const uint32_t*)ss.hist.p, row_stride(nb), nb,
                     n, dst);
  GS_LAUNCHED("visible_count");
  return GS_OK;
}

gs_status launch_tile_order(Frame& f, hipStream_t s) {
  const uint32_t tiles = (uint32_t)f.vt.total_tiles;
  const uint32_t blocks = (tiles + 256 * kOrderItems - 1) / (256 * kOrderItems);
  auto* order = (uint32_t*)f.order_at().p;
  auto* counts = (uint32_t*)f.words.p + kWordCount;
  auto* ranges = (const uint2*)f.ranges.p;
  hipLaunchKernelGGL(k_order_count, dim3(blocks), dim3(256), 0, s, ranges, tiles, counts);
  GS_LAUNCHED("order_count");
  hipLaunchKernelGGL(k_order_place, dim3(blocks), dim3(256), 0, s, ranges, tiles,
                     (const uint32_t*)counts, counts + 256, order);
  GS_LAUNCHED("order_place");
  f.tile_order = order;
  return GS_OK;
}

gs_status launch_export_keys(Frame& f, uint64_t* dst, hipStream_t s) {
  if (f.K == 0) return GS_OK;
  auto go = [&](auto kern, auto* tkey) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((f.K + 255) / 256)), dim3(256), 0, s, tkey,
                       (const uint32_t*)f.tval[f.tkey_sel].p, (const uint32_t*)f.dkey.p,
                       (uint32_t)f.K, dst);
  };
  if (f.short_keys())
    go(k_export_keys<uint16_t>, (const uint16_t*)f.tkey[f.tkey_sel].p);
  else
    go(k_export_keys<uint32_t>, (const uint32_t*)f.tkey[f.tkey_sel].p);
  GS_LAUNCHED("export_keys");
  return GS_OK;
}

}  // namespace isogs
