// Atomic-free EmbeddingBag backward on gfx950 ("reverse indices" of Sec. 3.1.4
// of "Memory Layers at Scale": invert the lookup -> row mapping so that each
// gradient row knows which lookups contribute to it).
//
//   1. Stable LSD radix sort of the L = T*H*k lookups by row: 8-bit digits,
//      per pass a tile histogram, a scan of each digit's tile counts (one
//      workgroup per digit), and a stable scatter: each wave ranks a
//      contiguous quarter of the tile with ballots, and the tile goes out
//      through LDS in sorted order.  Keys are rows (< 2^26), values lookup ids.
//      For fewer keys the passes are a short chain instead (k_chain_*), up to
//      8192 one workgroup does everything (k_sort_one).  The search backward
//      sorts its slots with the same passes.
//   2. Segment heads (first lookup of each distinct row) -> seg_start[U + 1],
//      the head flags computed where they are counted and placed; the same
//      kernel lists the segments longer than a threshold.
//   3. One lane group per touched row (two adjacent rows per iteration): read
//      the value row once, then take the contributing lookups in lookup order,
//      a few at a time with their dy rows loaded together, add w * dy into a
//      register accumulator and write grad_w = dy . V[row]; finally one
//      read-modify-write of the fp32 gradient row (dense) or one write of the
//      row's gradient (sparse).  Rows are visited in ascending order, so the
//      value and gradient tables are streamed nearly sequentially, and the
//      result is bitwise deterministic.
//   4. A row with more than LONG_SEG lookups would hold one lane group for
//      its whole length: it is listed, the per-row kernel skips it, and it is
//      cut into chunks of consecutive lookups, each summed by a workgroup of
//      its own whose lane groups take contiguous runs of the chunk (their
//      partial sums meet in LDS); a last kernel adds the chunks' partial rows
//      in chunk order (still deterministic).
#include "pk_device.h"
#include "pk_internal.h"

namespace pk {

constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int SORT_ITEMS = 16;                 // keys per thread per tile
constexpr int SORT_TILE = 256 * SORT_ITEMS;    // keys per workgroup tile
constexpr int SCAN_ITEMS = 8;
constexpr uint32_t LONG_SEG = 1024;  // lookups of a row beyond which it is split
constexpr uint32_t LONG_CHUNK = 1024;  // lookups of a long row per workgroup, at most
// Fewer where the long rows are few: their lookups are spread over LONG_WGS
// workgroups.  A chunk is a serial chain of dy reads in each wave, so the sink
// rows of 3 heads (9003 lookups, D = 640) took 70 us as 9 chunks of 1024 and
// 13 us as 72 of 128.
constexpr uint32_t LONG_WGS = 256;
constexpr uint32_t LONG_CHUNK_MIN = 128;
constexpr int LONG_WAVES = 8;        // waves of the workgroup that takes a chunk
constexpr int SCAN_TILE = 256 * SCAN_ITEMS;
constexpr int64_t SEG_TILES_MAX = 8192;  // tiles whose counts k_seg_place adds up itself

static inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ------------------------------------------------------------------ scan ----
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += wsum[w];
  total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  __syncthreads();
  return before + x - v;
}

// Single workgroup: exclusive scan of the tile sums, in place, any count.
__global__ __launch_bounds__(256) void k_scan_top(uint32_t* __restrict__ sums, int64_t nb) {
  __shared__ uint32_t wsum[4];
  uint32_t carry = 0;
  for (int64_t base = 0; base < nb; base += SCAN_TILE) {
    const int64_t b0 = base + threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
      v[i] = (b0 + i < nb) ? sums[b0 + i] : 0u;
      s += v[i];
    }
    uint32_t total;
    uint32_t run = carry + block_exclusive_scan(s, wsum, total);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
      if (b0 + i < nb) sums[b0 + i] = run;
      run += v[i];
    }
    carry += total;
  }
}

// Per digit d (one workgroup each) of a radix pass: exclusive scan, in place,
// of the tile counts hist[d*nblk .. (d+1)*nblk) (digit-major), and the digit's
// total in totals[d]; the scatter adds the digits' bases (a scan of totals).
__global__ __launch_bounds__(256) void k_scan_digits(uint32_t* __restrict__ hist, int64_t nblk,
                                                     uint32_t* __restrict__ totals) {
  __shared__ uint32_t wsum[4];
  uint32_t* h = hist + (int64_t)blockIdx.x * nblk;
  uint32_t carry = 0;
  for (int64_t base = 0; base < nblk; base += SCAN_TILE) {
    const int64_t i0 = base + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
      v[j] = (i0 + j < nblk) ? h[i0 + j] : 0u;
      sum += v[j];
    }
    uint32_t total;
    uint32_t run = carry + block_exclusive_scan(sum, wsum, total);
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
      if (i0 + j < nblk) h[i0 + j] = run;
      run += v[j];
    }
    carry += total;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// ----------------------------------------------------------- radix sort ----
// KM selects where a pass takes its items: SRC_I64 (an int64 array) and SRC_U32
// (rows of u32 slots, see SortSrc) are first passes, SRC_NEXT a later pass (keys
// and values from the previous pass's output).
constexpr int SRC_I64 = 0, SRC_U32 = 1, SRC_NEXT = 2;

// Key of a pass's item i; false where there is none.  First passes: item i of
// the int64 array (value: the position), or slot i of rows of k u32 keys of
// which row r fills its first counts[r] (the others are dropped; value: the
// slot).
template <int KM>
__device__ __forceinline__ bool item_key(const SortSrc& src, int64_t i, int64_t L, uint32_t& key) {
  if (i >= L) return false;
  if constexpr (KM == SRC_I64) {
    key = (uint32_t)reinterpret_cast<const int64_t*>(src.keys)[i];
  } else if constexpr (KM == SRC_NEXT) {
    key = reinterpret_cast<const uint32_t*>(src.keys)[i];
  } else {
    const uint32_t r = (uint32_t)i / (uint32_t)src.k;
    if ((uint32_t)i - r * (uint32_t)src.k >= src.counts[r]) return false;
    key = reinterpret_cast<const uint32_t*>(src.keys)[i];
  }
  return true;
}

// Ldev: the item count of a later pass after one over slots (null: L).
template <int KM>
__global__ __launch_bounds__(256) void k_radix_hist(SortSrc src, int64_t L,
                                                    const uint32_t* __restrict__ Ldev, int shift,
                                                    int bits, int64_t nblk,
                                                    uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[RADIX];
  h[threadIdx.x] = 0;
  __syncthreads();
  if (Ldev) L = *Ldev;
  const uint32_t mask = (1u << bits) - 1u;
  const int64_t tile = (int64_t)blockIdx.x * SORT_TILE;
#pragma unroll 4
  for (int i = 0; i < SORT_ITEMS; ++i) {
    uint32_t key;
    if (item_key<KM>(src, tile + i * 256 + threadIdx.x, L, key)) atomicAdd(&h[(key >> shift) & mask], 1u);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of one radix pass.  Wave w of the workgroup ranks the w-th
// quarter of the tile (positions in order: 16 rounds of 64), each key's rank
// within its digit coming from ballots and the wave's own digit counters in
// LDS (a wave's LDS accesses stay in program order, so no barrier is needed
// between rounds).  One block scan then gives each digit's start in the tile
// and each wave's start within the digit; the tile is written to LDS in
// sorted order and from there to its digits' runs, consecutive threads
// writing consecutive addresses.  Keys of equal digit keep their order.
template <int KM>
__global__ __launch_bounds__(256) void k_radix_scatter(
    SortSrc src, const uint32_t* __restrict__ vals_in, int64_t L, const uint32_t* __restrict__ Ldev,
    int shift, int bits, int64_t nblk, const uint32_t* __restrict__ offsets,
    const uint32_t* __restrict__ totals, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, uint32_t* __restrict__ total_out) {
  constexpr int PER_WAVE = SORT_TILE / 4;  // contiguous keys ranked by one wave
  constexpr int ROUNDS = PER_WAVE / WAVE;
  const int64_t tile = (int64_t)blockIdx.x * SORT_TILE;
  if (Ldev) L = *Ldev;
  if (tile >= L) return;  // the whole workgroup
  __shared__ uint32_t run[RADIX];      // global start of each digit's run for this tile
  __shared__ uint32_t tstart[RADIX];   // start of each digit within the tile
  __shared__ uint32_t wcnt[4][RADIX];  // per-wave digit counts, then per-wave starts
  __shared__ uint32_t wsum[4];
  __shared__ uint32_t skey[SORT_TILE];
  __shared__ uint32_t sval[SORT_TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  {  // thread tid = digit: where the digit starts overall, plus this tile's offset in it
    uint32_t all;
    const uint32_t dbase = block_exclusive_scan(totals[tid], wsum, all);
    run[tid] = dbase + offsets[(int64_t)tid * nblk + blockIdx.x];
    if (total_out && blockIdx.x == 0 && tid == 0) *total_out = all;
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0;
  __syncthreads();
  const uint32_t mask = (1u << bits) - 1u;
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t wbase = tile + (int64_t)wave * PER_WAVE;
  uint32_t key[ROUNDS], val[ROUNDS], rk[ROUNDS];
  uint32_t have = 0;  // bit i: the lane has an item in round i
#pragma unroll
  for (int i = 0; i < ROUNDS; ++i) {
    const int64_t pos = wbase + i * WAVE + lane;
    key[i] = 0;
    const bool valid = item_key<KM>(src, pos, L, key[i]);
    val[i] = valid ? (KM != SRC_NEXT ? (uint32_t)pos : vals_in[pos]) : 0u;
    have |= valid ? 1u << i : 0u;
    const uint32_t dig = (key[i] >> shift) & mask;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (dig >> b) & 1u;
      const uint64_t set = __ballot(bit);
      peers &= bit ? set : ~set;
    }
    const uint32_t r = (uint32_t)__popcll(peers & below);
    rk[i] = wcnt[wave][dig] + r;  // keys of this digit in the wave's earlier rounds, then lanes
    if (valid && r == 0) wcnt[wave][dig] += (uint32_t)__popcll(peers);
  }
  __syncthreads();
  uint32_t n;  // items of the tile
  {  // thread tid = digit: the tile's digit starts and each wave's start within it
    const uint32_t c0 = wcnt[0][tid], c1 = wcnt[1][tid], c2 = wcnt[2][tid], c3 = wcnt[3][tid];
    const uint32_t st = block_exclusive_scan(c0 + c1 + c2 + c3, wsum, n);
    tstart[tid] = st;
    wcnt[0][tid] = st;
    wcnt[1][tid] = st + c0;
    wcnt[2][tid] = st + c0 + c1;
    wcnt[3][tid] = st + c0 + c1 + c2;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ROUNDS; ++i) {
    if ((have >> i) & 1u) {
      const uint32_t p = wcnt[wave][(key[i] >> shift) & mask] + rk[i];
      skey[p] = key[i];
      sval[p] = val[i];
    }
  }
  __syncthreads();
  for (uint32_t e = tid; e < n; e += 256) {
    const uint32_t kk = skey[e];
    const uint32_t dig = (kk >> shift) & mask;
    const uint32_t dst = run[dig] + e - tstart[dig];
    keys_out[dst] = kk;
    vals_out[dst] = sval[e];
  }
}

// ------------------------------------------------------------- segments ----
// Segment heads of the sorted keys (i == 0 or keys[i] != keys[i-1]), counted
// per scan tile (thread: SCAN_ITEMS consecutive keys); k_scan_top then turns
// the counts into each tile's first segment number.
__global__ __launch_bounds__(256) void k_seg_count(const uint32_t* __restrict__ keys, int64_t Lmax,
                                                   const uint32_t* __restrict__ Ldev,
                                                   uint32_t* __restrict__ sums) {
  __shared__ uint32_t wsum[4];
  const int64_t L = (Ldev && (int64_t)*Ldev < Lmax) ? (int64_t)*Ldev : Lmax;
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
  uint32_t prev = (base > 0 && base <= L) ? keys[base - 1] : 0u;
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t x = base + i;
    if (x < L) {
      const uint32_t kx = keys[x];
      s += (x == 0 || kx != prev) ? 1u : 0u;
      prev = kx;
    }
  }
  uint32_t total;
  block_exclusive_scan(s, wsum, total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Each head i, with u = the number of heads before it, writes seg_start[u] = i;
// the last item writes seg_start[U] = L and U (the number of segments).
// scanned: sums holds each tile's first segment number; otherwise the tiles'
// counts, and the block adds those before it itself (a launch less).  A segment
// of more than thresh items is listed in long_list (in no particular order:
// each is then summed on its own).
__global__ __launch_bounds__(256) void k_seg_place(const uint32_t* __restrict__ keys, int64_t Lmax,
                                                   const uint32_t* __restrict__ Ldev,
                                                   const uint32_t* __restrict__ sums, bool scanned,
                                                   uint32_t* __restrict__ seg_start,
                                                   uint32_t* __restrict__ nseg, uint32_t thresh,
                                                   uint32_t* __restrict__ long_list,
                                                   uint32_t* __restrict__ long_cnt) {
  __shared__ uint32_t wsum[4];
  const int64_t L = (Ldev && (int64_t)*Ldev < Lmax) ? (int64_t)*Ldev : Lmax;
  if ((int64_t)blockIdx.x * SCAN_TILE >= L) return;  // nothing in this tile
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
  uint32_t before = 0;
  if (scanned) {
    before = sums[blockIdx.x];
  } else {
    uint32_t part = 0;
    for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 256) part += sums[i];
    block_exclusive_scan(part, wsum, before);
  }
  uint32_t prev = (base > 0 && base <= L) ? keys[base - 1] : 0u;
  bool head[SCAN_ITEMS], lng[SCAN_ITEMS];
  uint32_t s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t x = base + i;
    head[i] = lng[i] = false;
    if (x < L) {
      const uint32_t kx = keys[x];
      head[i] = (x == 0 || kx != prev);
      lng[i] = head[i] && x + thresh < L && keys[x + thresh] == kx;
      prev = kx;
    }
    s += head[i] ? 1u : 0u;
  }
  uint32_t total;
  uint32_t run = before + block_exclusive_scan(s, wsum, total);
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int64_t x = base + i;
    if (head[i]) seg_start[run] = (uint32_t)x;
    if (lng[i]) long_list[atomicAdd(long_cnt, 1u)] = run;
    run += head[i] ? 1u : 0u;
    if (x == L - 1) {
      seg_start[run] = (uint32_t)L;
      *nseg = run;
    }
  }
}

// ------------------------------------------------------- few keys ----
// For few keys a radix pass of three launches is mostly launches and
// the latency of 16 serial rounds per wave on a few workgroups (65536 keys:
// 6 + 4 + 15 us a pass).  The chain takes one launch per pass after a first
// histogram: workgroups of 16 waves with 4 rounds each; every scatter adds up
// the tile counts before its own itself (at most 256 tiles) and counts the next
// pass's digits of the tiles it writes to with integer atomics (the counts
// cleared by the first launch).  The result is the same stable sort.
constexpr int CHAIN_ITEMS = 4;                       // keys per thread
constexpr int CHAIN_TILE = 1024 * CHAIN_ITEMS;
constexpr int ONE_ITEMS = 8;
constexpr int64_t ONE_MAX = 1024 * ONE_ITEMS;        // keys one workgroup sorts by itself
// Keys the chain takes.  Each workgroup reads every tile's counts, so past some
// number three launches a pass are the faster form.  Lookups: 2^19 of them 25 us
// faster in the chain, 2^20 no faster (729 / 735 us with the rows), 2^21 5%
// slower.  Slots (the whole search backward, d = 32): 2^20 of them 172 in the
// chain and 181 us in three launches a pass, 2^21 271 and 230, 3.3M (100 tokens
// of 512 heads) 1719 and 1521.
constexpr int64_t CHAIN_MAX = (int64_t)1 << 19, CHAIN_MAX_SLOTS = (int64_t)1 << 20;

// Exclusive scan over the first 256 threads of a workgroup (thread = digit) of
// their v; every thread of the workgroup takes part.
__device__ __forceinline__ uint32_t scan_digits256(uint32_t v, uint32_t* wsum, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  if (lane == 63 && wave < 4) wsum[wave] = x;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave && w < 4; ++w) before += wsum[w];
  total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  __syncthreads();
  return before + x - v;
}

template <int KM>
__global__ __launch_bounds__(1024) void k_chain_hist(SortSrc src, int64_t L, int bits, int passes,
                                                     uint32_t* __restrict__ hist,
                                                     uint32_t* __restrict__ misc) {
  __shared__ uint32_t h[RADIX];
  const int tid = threadIdx.x;
  if (tid < RADIX) h[tid] = 0;
  if (blockIdx.x == 0 && tid < 4) misc[tid] = 0;
  __syncthreads();
  const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
  for (int i = 0; i < CHAIN_ITEMS; ++i) {
    uint32_t key;
    if (item_key<KM>(src, (int64_t)blockIdx.x * CHAIN_TILE + i * 1024 + tid, L, key))
      atomicAdd(&h[key & mask], 1u);
  }
  __syncthreads();
  if (tid < RADIX) {
    const int64_t at = (int64_t)blockIdx.x * RADIX + tid;
    hist[at] = h[tid];
    for (int p = 1; p < passes; ++p) hist[(int64_t)p * gridDim.x * RADIX + at] = 0;
  }
}

// One stable pass.  hist: this pass's counts per (tile, digit); hist_next (null
// on the last pass): the next pass's, with next_bits digits.  Ldev: the item
// count of a later pass (null: L).  The first pass writes it to total_out.
template <int KM>
__global__ __launch_bounds__(1024) void k_chain_scatter(
    SortSrc src, const uint32_t* __restrict__ vals_in, int64_t L, const uint32_t* __restrict__ Ldev,
    int shift, int bits, int next_bits, const uint32_t* __restrict__ hist,
    uint32_t* __restrict__ hist_next, uint32_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, uint32_t* __restrict__ total_out) {
  constexpr int PER_WAVE = CHAIN_ITEMS * WAVE;
  __shared__ uint32_t red[2][4][RADIX];
  __shared__ uint32_t run[RADIX], tstart[RADIX];
  __shared__ uint32_t wcnt[16][RADIX];
  __shared__ uint32_t wsum[4];
  __shared__ uint32_t skey[CHAIN_TILE], sval[CHAIN_TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nblk = gridDim.x;
  if (Ldev) L = *Ldev;
  const int64_t tile = (int64_t)blockIdx.x * CHAIN_TILE;
  if (tile >= L) return;  // whole block (block 0 never, unless there is nothing)
  const int64_t wbase = tile + (int64_t)wave * PER_WAVE;
  uint32_t key[CHAIN_ITEMS], val[CHAIN_ITEMS], rk[CHAIN_ITEMS];
  bool valid[CHAIN_ITEMS];
#pragma unroll
  for (int i = 0; i < CHAIN_ITEMS; ++i) {
    const int64_t pos = wbase + i * WAVE + lane;
    key[i] = 0;
    if constexpr (KM == SRC_NEXT) {
      valid[i] = pos < L;
      if (valid[i]) key[i] = reinterpret_cast<const uint32_t*>(src.keys)[pos];
      val[i] = valid[i] ? vals_in[pos] : 0u;
    } else {
      valid[i] = item_key<KM>(src, pos, L, key[i]);
      val[i] = (uint32_t)pos;
    }
  }
  {  // digit tid & 255, every fourth tile: all its keys, and those of earlier tiles
    const int d = tid & 255, qd = tid >> 8;
    uint32_t tot = 0, pre = 0;
#pragma unroll 8
    for (int b = qd; b < nblk; b += 4) {
      const uint32_t v = hist[(int64_t)b * RADIX + d];
      tot += v;
      pre += b < (int)blockIdx.x ? v : 0u;
    }
    red[0][qd][d] = tot;
    red[1][qd][d] = pre;
  }
#pragma unroll
  for (int i = 0; i < 16 * RADIX / 1024; ++i) (&wcnt[0][0])[i * 1024 + tid] = 0;
  __syncthreads();
  {
    uint32_t tot = 0, pre = 0, all;
    if (tid < RADIX) {
      tot = red[0][0][tid] + red[0][1][tid] + red[0][2][tid] + red[0][3][tid];
      pre = red[1][0][tid] + red[1][1][tid] + red[1][2][tid] + red[1][3][tid];
    }
    const uint32_t dbase = scan_digits256(tot, wsum, all);
    if (tid < RADIX) run[tid] = dbase + pre;
    if (total_out && blockIdx.x == 0 && tid == 0) *total_out = all;
  }
  const uint32_t mask = (1u << bits) - 1u;
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < CHAIN_ITEMS; ++i) {
    const uint32_t dig = (key[i] >> shift) & mask;
    uint64_t peers = __ballot(valid[i]);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (dig >> b) & 1u;
      const uint64_t set = __ballot(bit);
      peers &= bit ? set : ~set;
    }
    const uint32_t r = (uint32_t)__popcll(peers & below);
    rk[i] = wcnt[wave][dig] + r;
    if (valid[i] && r == 0) wcnt[wave][dig] += (uint32_t)__popcll(peers);
  }
  __syncthreads();
  uint32_t n;  // items of this tile
  {
    uint32_t cnt = 0;
    if (tid < RADIX)
      for (int w = 0; w < 16; ++w) cnt += wcnt[w][tid];
    const uint32_t st = scan_digits256(cnt, wsum, n);
    if (tid < RADIX) {
      tstart[tid] = st;
      uint32_t at = st;
      for (int w = 0; w < 16; ++w) {
        const uint32_t c = wcnt[w][tid];
        wcnt[w][tid] = at;
        at += c;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < CHAIN_ITEMS; ++i)
    if (valid[i]) {
      const uint32_t p = wcnt[wave][(key[i] >> shift) & mask] + rk[i];
      skey[p] = key[i];
      sval[p] = val[i];
    }
  __syncthreads();
  const uint32_t nmask = (1u << next_bits) - 1u;
  const int tbits = 32 - __builtin_clz((uint32_t)nblk);
  for (uint32_t e0 = 0; e0 < n; e0 += 1024) {
    const uint32_t e = e0 + tid;
    const bool in = e < n;
    const uint32_t kk = in ? skey[e] : 0u;
    const uint32_t dig = (kk >> shift) & mask;
    const uint32_t dst = in ? run[dig] + e - tstart[dig] : 0u;
    if (in) {
      keys_out[dst] = kk;
      vals_out[dst] = sval[e];
    }
    if (hist_next) {  // one atomic per distinct (tile, digit) of the wave: few hot ones
                      // (a sub-key table's upper digits, a sink row) serialise otherwise
      const uint32_t at = (dst / CHAIN_TILE) * RADIX + ((kk >> (shift + bits)) & nmask);
      uint64_t peers = __ballot(in);
      for (int b = 0; b < next_bits; ++b) {
        const bool bit = (at >> b) & 1u;
        const uint64_t set = __ballot(bit);
        peers &= bit ? set : ~set;
      }
      for (int b = RADIX_BITS; b < RADIX_BITS + tbits; ++b) {
        const bool bit = (at >> b) & 1u;
        const uint64_t set = __ballot(bit);
        peers &= bit ? set : ~set;
      }
      if (in && (peers & below) == 0) atomicAdd(&hist_next[at], (uint32_t)__popcll(peers));
    }
  }
}

// All passes, the segments and the long list of up to ONE_MAX keys by one
// workgroup, the keys in LDS between the passes.
template <int KM>
__global__ __launch_bounds__(1024) void k_sort_one(SortSrc src, int L, int key_bits,
                                                   uint32_t* __restrict__ keys_out,
                                                   uint32_t* __restrict__ vals_out,
                                                   uint32_t* __restrict__ seg_start,
                                                   uint32_t* __restrict__ misc, uint32_t thresh,
                                                   uint32_t* __restrict__ long_list,
                                                   uint32_t* __restrict__ long_cnt) {
  __shared__ uint32_t wcnt[16][RADIX];
  __shared__ uint32_t wsum[16];
  __shared__ uint32_t skey[ONE_MAX], sval[ONE_MAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (1ull << lane) - 1ull;
  if (tid == 0) *long_cnt = 0;
  uint32_t key[ONE_ITEMS], val[ONE_ITEMS], rk[ONE_ITEMS];
  bool valid[ONE_ITEMS];
  for (int shift = 0; shift < key_bits; shift += RADIX_BITS) {
    const int bits = key_bits - shift < RADIX_BITS ? key_bits - shift : RADIX_BITS;
    const uint32_t mask = (1u << bits) - 1u;
    // wave w takes the w-th run of whole 64s, as few rounds as the count needs
    const int rounds = (L + 1023) / 1024;
    const int wbase = wave * rounds * WAVE;
#pragma unroll
    for (int i = 0; i < ONE_ITEMS; ++i) {
      const int pos = wbase + i * WAVE + lane;
      key[i] = val[i] = 0;
      valid[i] = false;
      if (i < rounds) {
        if (shift == 0) {
          valid[i] = item_key<KM>(src, pos, L, key[i]);
          val[i] = (uint32_t)pos;
        } else if (pos < L) {
          valid[i] = true;
          key[i] = skey[pos];
          val[i] = sval[pos];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 16 * RADIX / 1024; ++i) (&wcnt[0][0])[i * 1024 + tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ONE_ITEMS; ++i) {
      if (i >= rounds) break;  // the same for the whole workgroup
      const uint32_t dig = (key[i] >> shift) & mask;
      uint64_t peers = __ballot(valid[i]);
      for (int b = 0; b < bits; ++b) {
        const bool bit = (dig >> b) & 1u;
        const uint64_t set = __ballot(bit);
        peers &= bit ? set : ~set;
      }
      const uint32_t r = (uint32_t)__popcll(peers & below);
      rk[i] = wcnt[wave][dig] + r;
      if (valid[i] && r == 0) wcnt[wave][dig] += (uint32_t)__popcll(peers);
    }
    __syncthreads();
    uint32_t n;
    {
      uint32_t cnt = 0;
      if (tid < RADIX)
        for (int w = 0; w < 16; ++w) cnt += wcnt[w][tid];
      uint32_t at = scan_digits256(cnt, wsum, n);
      if (tid < RADIX)
        for (int w = 0; w < 16; ++w) {
          const uint32_t c = wcnt[w][tid];
          wcnt[w][tid] = at;
          at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ONE_ITEMS; ++i)
      if (valid[i]) {
        const uint32_t p = wcnt[wave][(key[i] >> shift) & mask] + rk[i];
        skey[p] = key[i];
        sval[p] = val[i];
      }
    L = (int)n;  // dropped slots are gone after the first pass
    __syncthreads();
  }
  for (int i = tid; i < L; i += 1024) {
    keys_out[i] = skey[i];
    vals_out[i] = sval[i];
  }
  // segments: thread t takes items [t * per, (t + 1) * per)
  const int per = (L + 1023) / 1024;
  const int i0 = tid * per < L ? tid * per : L, i1 = i0 + per < L ? i0 + per : L;
  uint32_t heads = 0;
  for (int i = i0; i < i1; ++i) heads += (i == 0 || skey[i] != skey[i - 1]) ? 1u : 0u;
  uint32_t x = heads;
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, WAVE);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint32_t u = x - heads;
  for (int w = 0; w < wave; ++w) u += wsum[w];
  for (int i = i0; i < i1; ++i) {
    const uint32_t kx = skey[i];
    if (i == 0 || kx != skey[i - 1]) {
      seg_start[u] = (uint32_t)i;
      if (i + thresh < (uint32_t)L && skey[i + thresh] == kx) long_list[atomicAdd(long_cnt, 1u)] = u;
      ++u;
    }
    if (i == L - 1) {
      seg_start[u] = (uint32_t)L;
      misc[0] = u;
    }
  }
  if (L == 0 && tid == 0) {
    seg_start[0] = 0;
    misc[0] = 0;
  }
}

// ------------------------------------------------------- per-row backward ----
// One lane group per touched row.  A row with more than LONG_SEG lookups is
// taken as empty here (its gradient row is written back unchanged, or as zero
// in the sparse form) and summed afterwards by k_bag_bwd_long, in stream
// order.  Value and gradient rows are streamed once
// per step with non-temporal accesses, so they do not push the re-read dy rows
// and metadata out of the caches.  A lane group takes SB adjacent segments per
// iteration (loads of all of them, then all of their gradient-row stores: one
// longer read burst and one contiguous write burst), with the next batch's
// bounds prefetched; the old gradient row is read into the accumulator
// together with the value row.
// Lookups of a segment taken together: more for narrow rows (fewer registers
// per dy row), capped by the lane group's width.
template <int NQ, int CL>
struct RowsBatch {
  static constexpr int raw = NQ >= 16 ? 1 : (NQ >= 8 ? 2 : (NQ >= 4 ? 4 : 8));
  static constexpr int value = raw < CL ? raw : CL;
};

template <typename V, int NQ, int CL, bool SPARSE, int SB>
__global__ __launch_bounds__(256) void k_bag_bwd_rows(
    const V* __restrict__ dy, const V* __restrict__ values, int D, const float* __restrict__ w,
    int bag, const uint32_t* __restrict__ rows_sorted, const uint32_t* __restrict__ lookups,
    const uint32_t* __restrict__ seg_start, const uint32_t* __restrict__ nseg,
    float* __restrict__ grad_values, int64_t* __restrict__ rows_out,
    float* __restrict__ grad_rows_out, float* __restrict__ grad_w) {
  using Q = Quad<V>;
  constexpr int G = WAVE / CL;
  constexpr int PB = RowsBatch<NQ, CL>::value;
  const int lane = threadIdx.x & 63;
  const int grp = lane / CL, cl = lane % CL;
  const int nquad = D / 4;
  const int64_t U = *nseg;
  const bool dense = !SPARSE && grad_values != nullptr;
  bool ok[NQ];
#pragma unroll
  for (int m = 0; m < NQ; ++m) ok[m] = (m * CL + cl) < nquad;

  const int64_t step = (int64_t)gridDim.x * 4 * G * SB;
  int64_t u0 = (((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * G + grp) * SB;
  uint32_t s0[SB], s1[SB];
  int64_t row[SB];
#pragma unroll
  for (int b = 0; b < SB; ++b) {
    const bool live = u0 + b < U;
    s0[b] = live ? seg_start[u0 + b] : 0;
    s1[b] = live ? seg_start[u0 + b + 1] : 0;
    if (s1[b] - s0[b] > LONG_SEG) s1[b] = s0[b];  // summed by k_bag_bwd_long
    row[b] = live ? (int64_t)rows_sorted[s0[b]] : 0;
  }
  while (u0 < U) {
    typename Q::raw vraw[SB][NQ];
    float acc[SB][NQ][4];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
      const bool live = u0 + b < U;
#pragma unroll
      for (int m = 0; m < NQ; ++m) {
        const size_t e0 = (size_t)(m * CL + cl) * 4;
        vraw[b][m] = (ok[m] && live) ? Q::load_nt(values + row[b] * D + e0) : Q::zero();
        const uint4 g = (ok[m] && dense && live)
                            ? ld16_hint<PK_GRAD_NT_LOAD>(grad_values + row[b] * D + e0)
                            : uint4{0, 0, 0, 0};
        acc[b][m][0] = __uint_as_float(g.x); acc[b][m][1] = __uint_as_float(g.y);
        acc[b][m][2] = __uint_as_float(g.z); acc[b][m][3] = __uint_as_float(g.w);
      }
    }
    const int64_t un = u0 + step;
    uint32_t s0n[SB], s1n[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) {
      const bool live = un + b < U;
      s0n[b] = live ? seg_start[un + b] : 0;
      s1n[b] = live ? seg_start[un + b + 1] : 0;
      if (s1n[b] - s0n[b] > LONG_SEG) s1n[b] = s0n[b];
    }
#pragma unroll
    for (int b = 0; b < SB; ++b) {
      // The segment's lookups PB at a time: the group's lanes read PB lookup
      // ids and weights with one load each, then all PB dy rows are in flight
      // before the first is accumulated (lookup order is kept).
      // The next batch's lookup ids are loaded while this batch's dy rows are
      // in flight, so a long segment costs one dependent round trip per batch.
      uint32_t lid_next = (uint32_t)cl < s1[b] - s0[b] ? lookups[s0[b] + cl] : 0u;
      for (uint32_t s = s0[b]; s < s1[b]; s += PB) {
        const uint32_t nb = (s1[b] - s) < (uint32_t)PB ? (s1[b] - s) : (uint32_t)PB;
        const uint32_t lid = lid_next;
        const float wl = (uint32_t)cl < nb ? w[lid] : 0.f;
        lid_next = (uint32_t)cl + PB < s1[b] - s ? lookups[s + PB + cl] : 0u;
        typename Q::raw graw[PB][NQ];
        uint32_t lp[PB];
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) {
          lp[pp] = __shfl(lid, pp, CL);
          const int64_t t = lp[pp] / (uint32_t)bag;
#pragma unroll
          for (int m = 0; m < NQ; ++m)
            graw[pp][m] = (ok[m] && (uint32_t)pp < nb) ? Q::load(dy + t * D + (size_t)(m * CL + cl) * 4)
                                                       : Q::zero();
        }
        float part[PB];
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) {
          const float ww = __shfl(wl, pp, CL);
          part[pp] = 0.f;
#pragma unroll
          for (int m = 0; m < NQ; ++m) {
            float g[4], v[4];
            Q::unpack(graw[pp][m], g);
            Q::unpack(vraw[b][m], v);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              acc[b][m][e] = fmaf(ww, g[e], acc[b][m][e]);
              part[pp] = fmaf(g[e], v[e], part[pp]);
            }
          }
        }
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) part[pp] = group_sum<CL>(part[pp]);
        float mine = part[0];
#pragma unroll
        for (int pp = 1; pp < PB; ++pp) mine = (cl == pp) ? part[pp] : mine;
        if ((uint32_t)cl < nb) grad_w[lid] = mine;
      }
    }
    int64_t rown[SB];
#pragma unroll
    for (int b = 0; b < SB; ++b) rown[b] = (un + b < U) ? (int64_t)rows_sorted[s0n[b]] : 0;
    if (SPARSE || dense) {
#pragma unroll
      for (int b = 0; b < SB; ++b) {
        if (u0 + b >= U) continue;
        float* dst = SPARSE ? grad_rows_out + (size_t)(u0 + b) * D : grad_values + row[b] * D;
#pragma unroll
        for (int m = 0; m < NQ; ++m)
          if (ok[m])
            st16_hint<PK_GRAD_NT_STORE>(dst + (size_t)(m * CL + cl) * 4,
                                        uint4{__float_as_uint(acc[b][m][0]), __float_as_uint(acc[b][m][1]),
                                              __float_as_uint(acc[b][m][2]), __float_as_uint(acc[b][m][3])});
      }
    }
    if (SPARSE && cl == 0) {
#pragma unroll
      for (int b = 0; b < SB; ++b)
        if (u0 + b < U) rows_out[u0 + b] = row[b];
    }
    u0 = un;
#pragma unroll
    for (int b = 0; b < SB; ++b) {
      s0[b] = s0n[b];
      s1[b] = s1n[b];
      row[b] = rown[b];
    }
  }
}

// -------------------------------------------------------------- launcher ----
struct SortedWs {
  uint32_t *keys_a, *vals_a, *keys_b, *vals_b, *hist, *sums, *seg, *misc, *long_list, *totals,
      *long_base;
};
static int64_t max_long(int64_t L) { return L / LONG_SEG + 1; }

static SortedWs carve(void* ws, int64_t L) {
  const int64_t nblk = cdiv(L, SORT_TILE);
  const int64_t hist_n = (int64_t)RADIX * nblk;
  const int64_t scan_n = (hist_n > L + 1 ? hist_n : L + 1);
  char* p = reinterpret_cast<char*>(ws);
  SortedWs w;
  auto take = [&](size_t bytes) { uint32_t* r = reinterpret_cast<uint32_t*>(p); p += align256(bytes); return r; };
  w.keys_a = take(4 * (size_t)L);
  w.vals_a = take(4 * (size_t)L);
  w.keys_b = take(4 * (size_t)L);
  w.vals_b = take(4 * (size_t)L);
  w.hist = take(4 * (size_t)scan_n);
  w.sums = take(4 * (size_t)(cdiv(scan_n, SCAN_TILE) + 1));
  w.seg = take(4 * (size_t)(L + 1));
  w.misc = take(256);  // [0] segments, [1] long rows listed, [2] their chunk length, [3] items
  w.long_list = take(4 * (size_t)max_long(L));
  w.totals = take(4 * (size_t)RADIX);  // a radix pass's count per digit
  w.long_base = take(4 * (size_t)(max_long(L) + 1));  // first chunk of each listed long row
  return w;
}

size_t sorted_workspace_bytes(int64_t L) {
  const int64_t nblk = cdiv(L, SORT_TILE);
  const int64_t hist_n = (int64_t)RADIX * nblk;
  const int64_t scan_n = (hist_n > L + 1 ? hist_n : L + 1);
  return 4 * align256(4 * (size_t)L) + align256(4 * (size_t)scan_n) +
         align256(4 * (size_t)(cdiv(scan_n, SCAN_TILE) + 1)) + align256(4 * (size_t)(L + 1)) + 256 +
         align256(4 * (size_t)max_long(L)) + align256(4 * (size_t)RADIX) +
         align256(4 * (size_t)(max_long(L) + 1));
}

// Partial rows of the long-row chunks: at most L / LONG_CHUNK + max_long(L)
// chunks of D fp32 each.
size_t long_partial_bytes(int64_t L, int D) {
  return align256((size_t)(L / LONG_CHUNK + max_long(L)) * (size_t)D * sizeof(float));
}

// Stable LSD radix sort of the source's keys (< 2^key_bits) with their
// positions as values, then the segment starts of equal keys:
// seg[0..U] in b.seg, U in b.misc[0]; the segments of more than thresh items in
// long_list, their number in b.misc[1].  *ks / *vs receive the sorted arrays.
// L is the item count, of slots its upper bound.
static hipError_t sort_segments(const SortSrc& src, int64_t L, int key_bits, const SortedWs& b,
                                uint32_t thresh, uint32_t* long_list, const uint32_t** ks,
                                const uint32_t** vs, hipStream_t st) {
  const bool slots = src.counts != nullptr;
  const uint32_t* Ldev = nullptr;  // the items' number, when on the device
  uint32_t *kout = b.keys_a, *vout = b.vals_a;
  if (L <= ONE_MAX) {
    *ks = kout;
    *vs = vout;
    if (slots)
      hipLaunchKernelGGL(k_sort_one<SRC_U32>, dim3(1), dim3(1024), 0, st, src, (int)L, key_bits, kout,
                         vout, b.seg, b.misc, thresh, long_list, b.misc + 1);
    else
      hipLaunchKernelGGL(k_sort_one<SRC_I64>, dim3(1), dim3(1024), 0, st, src, (int)L, key_bits, kout,
                         vout, b.seg, b.misc, thresh, long_list, b.misc + 1);
    return hipGetLastError();
  }
  const int passes = (key_bits + RADIX_BITS - 1) / RADIX_BITS;
  if (L <= (slots ? CHAIN_MAX_SLOTS : CHAIN_MAX)) {
    const int64_t nblk = cdiv(L, CHAIN_TILE);  // up to four histograms fit b.hist: 1024 * nblk <= L
    const dim3 g((unsigned)nblk), blk(1024);
    const int bits0 = key_bits < RADIX_BITS ? key_bits : RADIX_BITS;
    if (slots)
      hipLaunchKernelGGL(k_chain_hist<SRC_U32>, g, blk, 0, st, src, L, bits0, passes, b.hist, b.misc);
    else
      hipLaunchKernelGGL(k_chain_hist<SRC_I64>, g, blk, 0, st, src, L, bits0, passes, b.hist, b.misc);
    SortSrc in = src;
    const uint32_t* vin = nullptr;
    for (int p = 0; p < passes; ++p) {
      const int shift = p * RADIX_BITS;
      auto width = [&](int q) { return key_bits - q * RADIX_BITS < RADIX_BITS ? key_bits - q * RADIX_BITS : RADIX_BITS; };
      const uint32_t* hist = b.hist + (int64_t)p * nblk * RADIX;
      uint32_t* next = p + 1 < passes ? b.hist + (int64_t)(p + 1) * nblk * RADIX : nullptr;
      const int nbits = next ? width(p + 1) : 1;
      const uint32_t* count = p > 0 ? b.misc + 3 : nullptr;
      uint32_t* total = p == 0 ? b.misc + 3 : nullptr;
      if (p > 0)
        hipLaunchKernelGGL(k_chain_scatter<SRC_NEXT>, g, blk, 0, st, in, vin, L, count, shift, width(p), nbits, hist, next, kout, vout, total);
      else if (slots)
        hipLaunchKernelGGL(k_chain_scatter<SRC_U32>, g, blk, 0, st, in, vin, L, count, shift, width(p), nbits, hist, next, kout, vout, total);
      else
        hipLaunchKernelGGL(k_chain_scatter<SRC_I64>, g, blk, 0, st, in, vin, L, count, shift, width(p), nbits, hist, next, kout, vout, total);
      in = SortSrc{kout, nullptr, 0};
      vin = vout;
      if (kout == b.keys_a) { kout = b.keys_b; vout = b.vals_b; }
      else { kout = b.keys_a; vout = b.vals_a; }
    }
    *ks = reinterpret_cast<const uint32_t*>(in.keys);
    *vs = vin;
    Ldev = b.misc + 3;
  } else {
    hipError_t e = launch_fill_u32(b.misc, 0u, 2, st);
    if (e != hipSuccess) return e;
    const int64_t nblk = cdiv(L, SORT_TILE);
    SortSrc in = src;
    const uint32_t* vin = nullptr;
    for (int shift = 0; shift < key_bits; shift += RADIX_BITS) {
      const int bits = (key_bits - shift) < RADIX_BITS ? (key_bits - shift) : RADIX_BITS;
      const dim3 g((unsigned)nblk), blk(256);
      uint32_t* total = slots && shift == 0 ? b.misc + 3 : nullptr;
      auto pass = [&](auto hist, auto scatter) {
        hipLaunchKernelGGL(hist, g, blk, 0, st, in, L, Ldev, shift, bits, nblk, b.hist);
        hipLaunchKernelGGL(k_scan_digits, dim3(RADIX), blk, 0, st, b.hist, nblk, b.totals);
        hipLaunchKernelGGL(scatter, g, blk, 0, st, in, vin, L, Ldev, shift, bits, nblk, b.hist,
                           b.totals, kout, vout, total);
      };
      if (shift > 0) pass(k_radix_hist<SRC_NEXT>, k_radix_scatter<SRC_NEXT>);
      else if (slots) pass(k_radix_hist<SRC_U32>, k_radix_scatter<SRC_U32>);
      else pass(k_radix_hist<SRC_I64>, k_radix_scatter<SRC_I64>);
      if (total) Ldev = total;
      in = SortSrc{kout, nullptr, 0};
      vin = vout;
      if (kout == b.keys_a) { kout = b.keys_b; vout = b.vals_b; }
      else { kout = b.keys_a; vout = b.vals_a; }
    }
    *ks = reinterpret_cast<const uint32_t*>(in.keys);
    *vs = vin;
  }
  const int64_t nb = cdiv(L, SCAN_TILE);
  const bool scanned = nb > SEG_TILES_MAX;
  hipLaunchKernelGGL(k_seg_count, dim3((unsigned)nb), dim3(256), 0, st, *ks, L, Ldev, b.sums);
  if (scanned) hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, st, b.sums, nb);
  hipLaunchKernelGGL(k_seg_place, dim3((unsigned)nb), dim3(256), 0, st, *ks, L, Ldev, b.sums, scanned,
                     b.seg, b.misc, thresh, long_list, b.misc + 1);
  return hipGetLastError();
}

// Sort of up to nslots slots in rows of k with their counts (values: the slots)
// for other kernels of the library.
hipError_t sort_slots_segments(const SortSrc& slots, int64_t nslots, int key_bits, void* ws,
                               uint32_t thresh, uint32_t* long_list, const uint32_t** ks,
                               const uint32_t** vs, const uint32_t** seg, const uint32_t** nseg,
                               const uint32_t** nlong, hipStream_t st) {
  SortedWs b = carve(ws, nslots);
  *seg = b.seg;
  *nseg = b.misc;
  *nlong = b.misc + 1;
  return sort_segments(slots, nslots, key_bits, b, thresh, long_list, ks, vs, st);
}

// Rows listed with the segments (more than LONG_SEG lookups) are cut into chunks
// of consecutive lookups (in lookup order), and every chunk of
// every listed row is summed by a workgroup of its own, so a row chosen by a
// large share of the tokens is spread over many CUs:
//   k_long_bases    (one workgroup) the chunk length, from the listed rows'
//                   lookups, and the first chunk number of each listed row
//                   (an exclusive scan of the chunk counts, in list order),
//   k_bag_bwd_long  (persistent grid over the chunks) the chunk's lane groups
//                   take contiguous runs of its lookups, write their grad_w and
//                   sum w * dy into partial rows in LDS, added in group order
//                   into the chunk's partial row in the workspace,
//   k_long_reduce   (one workgroup per listed row) adds the row's partial rows
//                   to the old gradient row (dense) or writes their sum as the
//                   row's gradient (sparse): each of the workgroup's thread
//                   groups a contiguous run of them in chunk order, the runs in
//                   order.
// The list's order varies from run to run, but a row's value depends only on
// its own chunks and their length, which depends only on the lengths of the
// listed rows: bitwise deterministic.
// chunk_cap: L / LONG_CHUNK.  With n lookups in the listed rows there are at most
// n / c whole chunks of c and one more per row; n / c <= chunk_cap both for
// c >= n / chunk_cap and for c = LONG_CHUNK, which long_partial_bytes holds.
__global__ __launch_bounds__(256) void k_long_bases(const uint32_t* __restrict__ seg_start,
                                                    const uint32_t* __restrict__ long_list,
                                                    const uint32_t* __restrict__ long_cnt,
                                                    uint32_t chunk_cap,
                                                    uint32_t* __restrict__ chunk_out,
                                                    uint32_t* __restrict__ long_base) {
  __shared__ uint32_t wsum[4];
  const uint32_t nlong = *long_cnt;
  if (nlong == 0) {
    if (threadIdx.x == 0) long_base[0] = 0;
    return;
  }
  uint32_t mine = 0, lookups;
  for (uint32_t i = threadIdx.x; i < nlong; i += 256) {
    const uint32_t u = long_list[i];
    mine += seg_start[u + 1] - seg_start[u];
  }
  block_exclusive_scan(mine, wsum, lookups);
  const uint32_t parts = chunk_cap < LONG_WGS ? chunk_cap : LONG_WGS;  // a listed row: at least 1
  uint32_t chunk = (lookups + parts - 1) / parts;
  if (chunk < LONG_CHUNK_MIN) chunk = LONG_CHUNK_MIN;
  if (chunk > LONG_CHUNK) chunk = LONG_CHUNK;
  if (threadIdx.x == 0) *chunk_out = chunk;
  uint32_t carry = 0;
  for (uint32_t i0 = 0; i0 < nlong; i0 += 256) {
    const uint32_t i = i0 + threadIdx.x;
    uint32_t nch = 0;
    if (i < nlong) {
      const uint32_t u = long_list[i];
      nch = (seg_start[u + 1] - seg_start[u] + chunk - 1) / chunk;
    }
    uint32_t total;
    const uint32_t before = block_exclusive_scan(nch, wsum, total);
    if (i < nlong) long_base[i] = carry + before;
    carry += total;
  }
  if (threadIdx.x == 0) long_base[nlong] = carry;
}

template <typename V, int NQ, int CL>
__global__ __launch_bounds__(64 * LONG_WAVES) void k_bag_bwd_long(
    const V* __restrict__ dy, const V* __restrict__ values, int D, const float* __restrict__ w,
    int bag, const uint32_t* __restrict__ rows_sorted, const uint32_t* __restrict__ lookups,
    const uint32_t* __restrict__ seg_start, const uint32_t* __restrict__ long_list,
    const uint32_t* __restrict__ long_cnt, const uint32_t* __restrict__ chunk_p,
    const uint32_t* __restrict__ long_base, float* __restrict__ part,
    float* __restrict__ grad_w) {
  using Q = Quad<V>;
  constexpr int G = WAVE / CL;
  constexpr int PB = RowsBatch<NQ, CL>::value;
  extern __shared__ float lpart[];  // [ng][D]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = wave * G + lane / CL, cl = lane % CL;
  const int nquad = D / 4;
  int ng = LONG_WAVES * G;
  if (ng > 16384 / D) ng = 16384 / D;  // 64 KiB of partial rows
  const bool mine = grp < ng;
  bool ok[NQ];
#pragma unroll
  for (int m = 0; m < NQ; ++m) ok[m] = mine && (m * CL + cl) < nquad;
  const uint32_t nlong = *long_cnt;
  const uint32_t nchunk = long_base[nlong];
  const uint32_t chunk = *chunk_p;
  for (uint32_t g = blockIdx.x; g < nchunk; g += gridDim.x) {
    // the listed row holding chunk g: long_base is ascending
    uint32_t lo = 0, hi = nlong;  // long_base[lo] <= g < long_base[hi]
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (long_base[mid] <= g) lo = mid;
      else hi = mid;
    }
    const uint32_t u = long_list[lo];
    const uint32_t c = g - long_base[lo];
    const uint32_t s_end = seg_start[u + 1];
    const uint32_t c0 = seg_start[u] + c * chunk;
    const uint32_t c1 = c0 + chunk < s_end ? c0 + chunk : s_end;
    const int64_t row = (int64_t)rows_sorted[c0];
    const uint32_t len = c1 - c0;
    const uint32_t per = (len + (uint32_t)ng - 1) / (uint32_t)ng;
    uint32_t a = mine ? (uint32_t)grp * per : len, z = mine ? (uint32_t)(grp + 1) * per : len;
    a = (a < len ? a : len) + c0;
    z = (z < len ? z : len) + c0;
    typename Q::raw vraw[NQ];
    float acc[NQ][4];
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      vraw[m] = ok[m] ? Q::load(values + row * D + (size_t)(m * CL + cl) * 4) : Q::zero();
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[m][e] = 0.f;
    }
    for (uint32_t s = a; s < z; s += PB) {
      const uint32_t nb = (z - s) < (uint32_t)PB ? (z - s) : (uint32_t)PB;
      const uint32_t lid = (uint32_t)cl < nb ? lookups[s + cl] : 0u;
      const float wl = (uint32_t)cl < nb ? w[lid] : 0.f;
      typename Q::raw graw[PB][NQ];
#pragma unroll
      for (int pp = 0; pp < PB; ++pp) {
        const uint32_t lp = __shfl(lid, pp, CL);
        const int64_t t = lp / (uint32_t)bag;
#pragma unroll
        for (int m = 0; m < NQ; ++m)
          graw[pp][m] = (ok[m] && (uint32_t)pp < nb) ? Q::load(dy + t * D + (size_t)(m * CL + cl) * 4)
                                                     : Q::zero();
      }
      float part_w[PB];
#pragma unroll
      for (int pp = 0; pp < PB; ++pp) {
        const float ww = __shfl(wl, pp, CL);
        part_w[pp] = 0.f;
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          float gg[4], v[4];
          Q::unpack(graw[pp][m], gg);
          Q::unpack(vraw[m], v);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[m][e] = fmaf(ww, gg[e], acc[m][e]);
            part_w[pp] = fmaf(gg[e], v[e], part_w[pp]);
          }
        }
      }
#pragma unroll
      for (int pp = 0; pp < PB; ++pp) part_w[pp] = group_sum<CL>(part_w[pp]);
      float gwv = part_w[0];
#pragma unroll
      for (int pp = 1; pp < PB; ++pp) gwv = (cl == pp) ? part_w[pp] : gwv;
      if ((uint32_t)cl < nb) grad_w[lid] = gwv;
    }
#pragma unroll
    for (int m = 0; m < NQ; ++m)
      if (ok[m]) {
        float* d = lpart + (size_t)grp * D + (size_t)(m * CL + cl) * 4;
        d[0] = acc[m][0]; d[1] = acc[m][1]; d[2] = acc[m][2]; d[3] = acc[m][3];
      }
    __syncthreads();
    for (int qd = threadIdx.x; qd < nquad; qd += blockDim.x) {
      float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int gi = 0; gi < ng; ++gi) {
        const float* sp = lpart + (size_t)gi * D + (size_t)qd * 4;
        tot.x += sp[0]; tot.y += sp[1]; tot.z += sp[2]; tot.w += sp[3];
      }
      *reinterpret_cast<float4*>(part + (size_t)g * D + (size_t)qd * 4) = tot;
    }
    __syncthreads();  // the LDS partial rows are reused for the next chunk
  }
}

constexpr int REDUCE_THREADS = 1024;
template <bool SPARSE>
__global__ __launch_bounds__(REDUCE_THREADS) void k_long_reduce(
    int D, const uint32_t* __restrict__ rows_sorted, const uint32_t* __restrict__ seg_start,
    const uint32_t* __restrict__ long_list, const uint32_t* __restrict__ long_cnt,
    const uint32_t* __restrict__ long_base, const float* __restrict__ part,
    float* __restrict__ grad_values, int64_t* __restrict__ rows_out,
    float* __restrict__ grad_rows_out) {
  constexpr int U = 8;  // partial rows in flight per thread
  __shared__ float4 run[REDUCE_THREADS];
  const uint32_t nlong = *long_cnt;
  const int nquad = D / 4;  // at most 1024
  const bool dense = !SPARSE && grad_values != nullptr;
  const int ng = REDUCE_THREADS / nquad;
  const int grp = (int)threadIdx.x / nquad, qd = (int)threadIdx.x - grp * nquad;
  for (uint32_t i = blockIdx.x; i < nlong; i += gridDim.x) {
    const uint32_t u = long_list[i];
    const int64_t row = (int64_t)rows_sorted[seg_start[u]];
    const uint32_t b0 = long_base[i], cnt = long_base[i + 1] - b0;
    const uint32_t per = (cnt + (uint32_t)ng - 1) / (uint32_t)ng;
    if (grp < ng) {
      const uint32_t a = (uint32_t)grp * per < cnt ? (uint32_t)grp * per : cnt;
      const uint32_t z = a + per < cnt ? a + per : cnt;
      const float* src = part + (size_t)b0 * D + (size_t)qd * 4;
      float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
      for (uint32_t g = a; g < z; g += U) {
        float4 pv[U];
#pragma unroll
        for (int j = 0; j < U; ++j)
          pv[j] = g + j < z ? *reinterpret_cast<const float4*>(src + (size_t)(g + j) * D)
                            : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int j = 0; j < U; ++j) {
          tot.x += pv[j].x; tot.y += pv[j].y; tot.z += pv[j].z; tot.w += pv[j].w;
        }
      }
      run[threadIdx.x] = tot;
    }
    __syncthreads();
    if (grp == 0 && (SPARSE || dense)) {
      float* dst = (SPARSE ? grad_rows_out + (size_t)u * D : grad_values + row * D) + (size_t)qd * 4;
      float4 tot = make_float4(0.f, 0.f, 0.f, 0.f);
      if (dense) tot = *reinterpret_cast<const float4*>(dst);
      // the groups with partial rows (narrow rows: up to 512 groups, often fewer rows)
      const int used = (int)((cnt + per - 1) / per);
      for (int j = 0; j < used; ++j) {
        const float4 pv = run[j * nquad + qd];
        tot.x += pv.x; tot.y += pv.y; tot.z += pv.z; tot.w += pv.w;
      }
      *reinterpret_cast<float4*>(dst) = tot;
    }
    if (SPARSE && threadIdx.x == 0) rows_out[u] = row;
    __syncthreads();  // run is reused for the next row
  }
}

hipError_t launch_bag_backward_sorted(bool bf16, const void* dy, const void* values, int64_t N,
                                      int D, const int64_t* idx, const float* w, int64_t T,
                                      int bag, float* grad_values, int64_t* rows_out,
                                      float* grad_rows_out, float* grad_w, void* ws, float* part,
                                      uint32_t** num_rows_dev, hipStream_t st) {
  const int64_t L = T * bag;
  SortedWs b = carve(ws, L);
  if (num_rows_dev) *num_rows_dev = b.misc;
  if (L == 0) return launch_fill_u32(b.misc, 0u, 2, st);
  hipError_t e = hipSuccess;
  const uint32_t* ks = nullptr;
  const uint32_t* vs = nullptr;

  // 1. radix sort of (row, lookup) by row; 2. segments of equal rows
  {
    LaunchTimer lt_sort("sort_by_row", st);
    int key_bits = 1;
    while (key_bits < 32 && (int64_t(1) << key_bits) < N) ++key_bits;
    e = sort_segments(SortSrc{idx, nullptr, 0}, L, key_bits, b, (uint32_t)LONG_SEG, b.long_list, &ks,
                      &vs, st);
    if (e != hipSuccess) return e;
  }

  // 3. one lane group per touched row
  const int nquad = D / 4;
  int64_t blocks = cdiv(L, 4 * PK_ROWS_BATCH);
  if (blocks > 16384) blocks = 16384;
  const dim3 grid((unsigned)blocks), block(256);
  const bool sparse = rows_out != nullptr;
  int64_t lblocks = L / LONG_CHUNK + max_long(L);  // chunks of long rows, at most
  if (lblocks > 1024) lblocks = 1024;
  int64_t rblocks = max_long(L);
  if (rblocks > 512) rblocks = 512;
  const int ngrp_cap = 16384 / D;  // partial rows that fit 64 KiB
  hipLaunchKernelGGL(k_long_bases, dim3(1), dim3(256), 0, st, (const uint32_t*)b.seg,
                     (const uint32_t*)b.long_list, (const uint32_t*)(b.misc + 1),
                     (uint32_t)(L / LONG_CHUNK), b.misc + 2, b.long_base);
  LaunchTimer lt("bag_backward_rows", st);
#define PK_ROWS_ONE(VT, NQ, CL, SP)                                                                \
  {                                                                                                \
    hipLaunchKernelGGL((k_bag_bwd_rows<VT, NQ, CL, SP, PK_ROWS_BATCH>), grid, block, 0, st,       \
                       (const VT*)dy, (const VT*)values, D, w, bag, ks, vs, b.seg, b.misc,         \
                       grad_values, rows_out, grad_rows_out, grad_w);                             \
    const int ng = (LONG_WAVES * (WAVE / CL)) < ngrp_cap ? LONG_WAVES * (WAVE / CL) : ngrp_cap;    \
    hipLaunchKernelGGL((k_bag_bwd_long<VT, NQ, CL>), dim3((unsigned)lblocks),                      \
                       dim3(64 * LONG_WAVES), (size_t)ng * D * sizeof(float), st, (const VT*)dy,   \
                       (const VT*)values, D, w, bag, ks, vs, b.seg, b.long_list, b.misc + 1,       \
                       b.misc + 2, b.long_base, part, grad_w);                                    \
    hipLaunchKernelGGL((k_long_reduce<SP>), dim3((unsigned)rblocks), dim3(REDUCE_THREADS), 0, st, D, ks,      \
                       b.seg, b.long_list, b.misc + 1, b.long_base, part, grad_values, rows_out,   \
                       grad_rows_out);                                                             \
  }
#define PK_ROWS(NQ, CL)                                                                           \
  if (bf16) {                                                                                     \
    if (sparse) PK_ROWS_ONE(uint16_t, NQ, CL, true) else PK_ROWS_ONE(uint16_t, NQ, CL, false)     \
  } else {                                                                                        \
    if (sparse) PK_ROWS_ONE(float, NQ, CL, true) else PK_ROWS_ONE(float, NQ, CL, false)           \
  }
  if (nquad > 512) { PK_ROWS(16, 64); }
  else if (nquad > 256) { PK_ROWS(8, 64); }
  else if (nquad > 128) { PK_ROWS(4, 64); }
  else if (nquad > 64) { PK_ROWS(2, 64); }
  else if (nquad > 32) { PK_ROWS(1, 64); }
  else if (nquad > 16) { PK_ROWS(1, 32); }
  else if (nquad > 8) { PK_ROWS(1, 16); }
  else if (nquad > 4) { PK_ROWS(1, 8); }
  else if (nquad > 2) { PK_ROWS(1, 4); }
  else { PK_ROWS(1, 2); }
#undef PK_ROWS
#undef PK_ROWS_ONE
  return hipGetLastError();
}

}  // namespace pk
