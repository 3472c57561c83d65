// Search backward on gfx950: gradients of the selected scores into queries and
// sub-keys (the keys are trainable parameters, Sec. 3 of "Memory Layers at
// Scale"; the selection passes no gradient).  With the composed index
// i = i1*S + i2 of Sec. 3.1.1 the score of rank j is
//   z_j = q[:d] . K[h,0,i1_j] + q[d:] . K[h,1,i2_j],
// so grad_q[:d] = sum_j gz_j K[h,0,i1_j] and grad_K[h,0,i] += sum_{j: i1_j = i}
// gz_j q[:d] (same for half 1).
//
// grad_q: one wave per (token, head).  The k lookups sit one per lane; per
// half, each lane finds the leader of its sub-key group (lowest rank with the
// same sub-key index) and the group's summed gradient, in rank order; the wave
// reads each distinct sub-key row once.
//
// grad_K: every sub-key row is hot (only S rows per head and half), and fp32
// atomics, in global memory or in LDS, serialise on them.  Instead the same
// wave emits one (head, half, sub-key) sort key per group leader, with the
// group's gradient sum, at the front of its (token, head, half) row of k
// slots, and counts them; the leaders are then brought into sub-key order, equal
// ones in token order: by a counting sort over the sub-keys (k_bin_*), or, for
// few leaders, by the library's radix sort.  One wave per sub-key sums gsum * q over
// its tokens (in token order; each token's query half is read once) and
// adds the sum into the sub-key row with one plain read-modify-write: no
// atomics, bitwise deterministic.  A segment longer than 2048 pairs (a
// sub-key that thousands of tokens chose) goes to a workgroup of 16 waves
// instead, whose contiguous runs are added in run order.
#include "pk_device.h"
#include "pk_internal.h"

namespace pk {

// k > 32 (k_search_bwd_q32 below otherwise):
// Per (token, head) wave, per half: lane j holds rank j's sub-key; each lane
// finds the ranks sharing its sub-key (one ballot per index bit), the lowest
// of them leads the group and adds the group's gradients in rank order.  Then
//   * grad_q (if wanted): the distinct sub-key rows are read QU at a time (all
//     loads in flight together), lane l owning elements 4l..4l+3;
//   * sort input (if wanted): row rp = (t*H + h)*2 + half gets its leaders'
//     keys (h*2 + half)*S + sub-key and group sums at slots rp*k + 0, 1, ...
//     (in rank order of the leaders) and their number at counts[rp].  Lookups
//     whose index lies outside [0, S*S) count as absent.
// idx and gz rows are kst >= k slots apart; with a sink (a fixed key-value
// pair per head scored as q . sink[h]) slot k of each row is the sink's and
// grad_q gains gz[sink slot] * sink[h] (its index is never read).
// With qstats (the forward normalised the queries, LayerNorm without affine)
// the two halves' gradients g with respect to the normalised query qhat stay
// in registers and grad_q = rstd * (g - mean(g) - xhat * mean(g * xhat)) over
// the query's n elements, xhat = (q - mean) * rstd in fp32 (the rounding of
// qhat to the query dtype passes the gradient unchanged).
#ifndef PK_SBWD_QU
#define PK_SBWD_QU 8
#endif
template <typename T>
__global__ __launch_bounds__(256) void k_search_bwd_q(const T* __restrict__ q,
                                                      const T* __restrict__ subkeys, int64_t ntok,
                                                      int H, int n, int S, int k, int kst,
                                                      const int64_t* __restrict__ idx,
                                                      const float* __restrict__ gz,
                                                      const T* __restrict__ sink,
                                                      const float2* __restrict__ qstats,
                                                      float* __restrict__ grad_q,
                                                      uint32_t* __restrict__ keys,
                                                      float* __restrict__ gvals,
                                                      uint32_t* __restrict__ counts) {
  constexpr int QU = PK_SBWD_QU;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = (int)(blockIdx.x % (unsigned)H);
  const int64_t t = (int64_t)(blockIdx.x / (unsigned)H) * 4 + wave;
  if (t >= ntok) return;
  const int d = n >> 1;
  const bool qlane = lane * 4 < d;
  const int ql = qlane ? lane * 4 : 0;
  const size_t r = (size_t)t * H + h;
  const int64_t ix = lane < k ? idx[r * kst + lane] : -1;
  const bool okl = ix >= 0 && ix < (int64_t)S * S;
  // the two sub-key indices (S * S <= 2^26: a 32-bit division)
  const int ix1 = okl ? (int)((uint32_t)ix / (uint32_t)S) : 0;
  const int ix2 = okl ? (int)((uint32_t)ix - (uint32_t)ix1 * (uint32_t)S) : 0;
  const float g = okl ? gz[r * kst + lane] : 0.f;
  const float gsink = sink ? gz[r * kst + k] : 0.f;
  const uint64_t below = (1ull << lane) - 1ull;
  const int nbits = S > 1 ? 32 - __builtin_clz((unsigned)(S - 1)) : 0;  // bits of a sub-key index
  float gh[2][4];  // with qstats: both halves' gradients with respect to qhat

#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int mine = okl ? (p == 0 ? ix1 : ix2) : -1;
    // the ranks sharing this lane's sub-key, as a mask over the wave's lanes:
    // one ballot per bit of the sub-key index
    uint64_t peers = __ballot(okl);
    for (int bt = 0; bt < nbits; ++bt) {
      const bool bit = (mine >> bt) & 1;
      const uint64_t set = __ballot(bit);
      peers &= bit ? set : ~set;
    }
    const bool leader = okl && (peers & below) == 0ull;
    // the leader's group sum, added in rank order; every lane takes part in
    // each exchange, the leaders keep what their own mask asks for
    float gsum = 0.f;
    uint64_t pm = leader ? peers : 0ull;
    while (__ballot(pm != 0ull) != 0ull) {
      const int j = pm != 0ull ? __builtin_ctzll(pm) : 0;
      const float v = __shfl(g, j, WAVE);
      if (pm != 0ull) {
        gsum += v;
        pm &= pm - 1ull;
      }
    }
    if (keys) {
      const uint64_t lm = __ballot(leader);
      const size_t rp = r * 2 + p;
      if (leader) {
        const size_t x = rp * k + __popcll(lm & below);
        keys[x] = (uint32_t)(h * 2 + p) * (uint32_t)S + (uint32_t)mine;
        gvals[x] = gsum;
      }
      if (lane == 0) counts[rp] = (uint32_t)__popcll(lm);
    }
    if (grad_q) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
      const T* kh = subkeys + (size_t)(h * 2 + p) * S * d + ql;
      uint64_t m = __ballot(leader);
      while (m) {
        QQuad<T> kq[QU];
        float gg[QU];
        const int first = __builtin_ctzll(m);
#pragma unroll
        for (int j = 0; j < QU; ++j) {
          const bool has = m != 0;
          const int L = has ? __builtin_ctzll(m) : first;
          m = has ? (m & (m - 1)) : m;
          const int i = __builtin_amdgcn_readlane(mine, L);
          const float gj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gsum), L));
          gg[j] = has ? gj : 0.f;
          kq[j].load(kh + (size_t)i * d);
        }
#pragma unroll
        for (int j = 0; j < QU; ++j) kq[j].fma_into(gg[j], acc);
      }
      if (sink) {
        QQuad<T> sq;
        sq.load(sink + (size_t)h * n + (size_t)p * d + ql);
        sq.fma_into(gsink, acc);
      }
      if (qstats) {
#pragma unroll
        for (int i = 0; i < 4; ++i) gh[p][i] = qlane ? acc[i] : 0.f;
      } else if (qlane) {
        *reinterpret_cast<float4*>(grad_q + r * n + (size_t)p * d + ql) =
            make_float4(acc[0], acc[1], acc[2], acc[3]);
      }
    }
  }
  if (qstats && grad_q) {
    const float2 st = qstats[r];
    float xh[2][4];
    float sg = 0.f, sgx = 0.f;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      QQuad<T> xq;
      xq.load(q + r * n + (size_t)p * d + ql);
      float v[4];
      xq.to_f32(v);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        xh[p][i] = qlane ? qn_apply(v[i], st.x, st.y) : 0.f;
        sg += gh[p][i];
        sgx = fmaf(gh[p][i], xh[p][i], sgx);
      }
    }
    sg = group_sum<WAVE>(sg);
    sgx = group_sum<WAVE>(sgx);
    const float mg = sg / (float)n, mgx = sgx / (float)n;
    if (qlane) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = st.y * (gh[p][i] - mg - xh[p][i] * mgx);
        *reinterpret_cast<float4*>(grad_q + r * n + (size_t)p * d + ql) =
            make_float4(o[0], o[1], o[2], o[3]);
      }
    }
  }
}

// 16 bytes of a query or sub-key half row.
template <typename T>
struct Seg16;
template <>
struct Seg16<uint16_t> {
  static constexpr int N = 8;
  uint4 raw;
  __device__ __forceinline__ void load(const uint16_t* p) { raw = ld16(p); }
  __device__ __forceinline__ void to_f32(float* v) const {
    v[0] = bf16_lo(raw.x); v[1] = bf16_hi(raw.x); v[2] = bf16_lo(raw.y); v[3] = bf16_hi(raw.y);
    v[4] = bf16_lo(raw.z); v[5] = bf16_hi(raw.z); v[6] = bf16_lo(raw.w); v[7] = bf16_hi(raw.w);
  }
};
template <>
struct Seg16<float> {
  static constexpr int N = 4;
  uint4 raw;
  __device__ __forceinline__ void load(const float* p) { raw = ld16(p); }
  __device__ __forceinline__ void to_f32(float* v) const {
    v[0] = __uint_as_float(raw.x); v[1] = __uint_as_float(raw.y);
    v[2] = __uint_as_float(raw.z); v[3] = __uint_as_float(raw.w);
  }
};

// k_search_bwd_q for k <= 32, where a half wave holds all ranks: lanes 0-31
// work on half 0 and lanes 32-63 on half 1 through every step, so the grouping
// is done once instead of twice (with 32-bit masks), and a sub-key row is read
// by 32 lanes of 16 bytes, a row of each half per instruction.  The kernel is
// bound by its vector instructions, not by the row reads from L2: 1052 per wave
// and 231 us as two passes (32768 tokens, 4 heads, S = 2048, k = 32), 709 and
// 177 us like this.  Every sum is the other form's, in its order.
template <typename T>
__global__ __launch_bounds__(256) void k_search_bwd_q32(
    const T* __restrict__ q, const T* __restrict__ subkeys, int64_t ntok, int H, int n, int S,
    int k, int kst, const int64_t* __restrict__ idx, const float* __restrict__ gz,
    const T* __restrict__ sink, const float2* __restrict__ qstats, float* __restrict__ grad_q,
    uint32_t* __restrict__ keys, float* __restrict__ gvals, uint32_t* __restrict__ counts) {
  using Seg = Seg16<T>;
  constexpr int N = Seg::N;
  constexpr int QU = PK_SBWD_QU;
  __shared__ uint2 list[4][2][32];  // the leaders' (sub-key, gradient sum bits), per half
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int p = lane >> 5, j = lane & 31;
  const int h = (int)(blockIdx.x % (unsigned)H);
  const int64_t t = (int64_t)(blockIdx.x / (unsigned)H) * 4 + wave;
  if (t >= ntok) return;
  const int d = n >> 1;
  const size_t r = (size_t)t * H + h;
  const int64_t ix = j < k ? idx[r * kst + j] : -1;
  const bool okl = ix >= 0 && ix < (int64_t)S * S;
  // the half's sub-key index (S * S <= 2^26: a 32-bit division)
  const uint32_t ix1 = okl ? (uint32_t)ix / (uint32_t)S : 0u;
  const int mine = okl ? (int)(p == 0 ? ix1 : (uint32_t)ix - ix1 * (uint32_t)S) : -1;
  const float g = okl ? gz[r * kst + j] : 0.f;
  const uint32_t below = (1u << j) - 1u;
  const int nbits = S > 1 ? 32 - __builtin_clz((unsigned)(S - 1)) : 0;  // bits of a sub-key index
  auto of_half = [&](uint64_t m) { return p == 0 ? (uint32_t)m : (uint32_t)(m >> 32); };
  // the ranks of this half sharing the lane's sub-key
  uint32_t peers = of_half(__ballot(okl));
  for (int bt = 0; bt < nbits; ++bt) {
    const int bit = __builtin_amdgcn_sbfe(mine, bt, 1);  // 0 or -1
    peers &= ~(of_half(__ballot(bit != 0)) ^ (uint32_t)bit);
  }
  const bool leader = okl && (peers & below) == 0u;
  // the leader's group sum, in rank order (the leader is its group's first); a
  // lane with nothing left takes a value it drops
  float gsum = g;
  uint32_t pm = leader ? peers & (peers - 1u) : 0u;
  while (__ballot(pm != 0u) != 0ull) {
    const int v = __builtin_amdgcn_ds_bpermute((p << 7) + (__builtin_ctz(pm | 0x80000000u) << 2),
                                               __float_as_int(g));
    gsum += pm != 0u ? __int_as_float(v) : 0.f;
    pm &= pm - 1u;
  }
  const uint64_t lm = __ballot(leader);
  const uint32_t lmh = of_half(lm);
  const uint32_t pos = (uint32_t)__builtin_popcount(lmh & below);
  const uint32_t cnt = (uint32_t)__builtin_popcount(lmh);
  if (keys) {
    const size_t rp = r * 2 + p;
    if (leader) {
      keys[rp * k + pos] = (uint32_t)(h * 2 + p) * (uint32_t)S + (uint32_t)mine;
      gvals[rp * k + pos] = gsum;
    }
    if (j == 0) counts[rp] = cnt;
  }
  if (!grad_q) return;
  const int e0 = j * N;
  const bool has = e0 < d;
  const int eo = has ? e0 : 0;
  // The leaders' list, as byte offsets into the head's two tables (at most
  // 2 * 8192 rows of 512 bytes): a row costs an LDS read at a constant offset
  // and one addition.  The last batch of QU is filled with its own first leader
  // at weight 0, so that only sub-keys the row selected are ever read (an
  // infinity in another one stays out of the sum); each half stops at its own.
  const uint32_t row_bytes = (uint32_t)d * (uint32_t)sizeof(T);
  uint2* const lst = list[wave][p];
  if (leader)
    lst[pos] = make_uint2((p == 0 ? 0u : (uint32_t)S * row_bytes) + (uint32_t)mine * row_bytes,
                          __float_as_uint(gsum));
  static_assert((QU & (QU - 1)) == 0 && 32 % QU == 0, "batches of the 32 list entries");
  const uint32_t last = cnt & ~(uint32_t)(QU - 1);  // start of a last, partial batch
  if ((uint32_t)j >= cnt && (uint32_t)j < last + QU && last < cnt) lst[j] = make_uint2(lst[last].x, 0u);
  const char* const kb = reinterpret_cast<const char*>(subkeys + (size_t)(h * 2) * S * d);
  const uint32_t lo = (uint32_t)eo * (uint32_t)sizeof(T);
  float acc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) acc[i] = 0.f;
  for (uint32_t b = 0; b < cnt; b += QU) {
    Seg ks[QU];
    uint2 e[QU];
#pragma unroll
    for (int u = 0; u < QU; ++u) e[u] = lst[b + u];
#pragma unroll
    for (int u = 0; u < QU; ++u) ks[u].load(reinterpret_cast<const T*>(kb + (e[u].x + lo)));
#pragma unroll
    for (int u = 0; u < QU; ++u) {
      float v[N];
      ks[u].to_f32(v);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] = fmaf(__uint_as_float(e[u].y), v[i], acc[i]);
    }
  }
  if (sink) {
    const float gsink = gz[r * kst + k];
    Seg sk;
    sk.load(sink + (size_t)h * n + (size_t)p * d + eo);
    float v[N];
    sk.to_f32(v);
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = fmaf(gsink, v[i], acc[i]);
  }
  if (qstats) {  // through the LayerNorm, over both halves
    const float2 st = qstats[r];
    Seg xq;
    xq.load(q + r * n + (size_t)p * d + eo);
    float v[N], xh[N], sg = 0.f, sgx = 0.f;
    xq.to_f32(v);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (!has) acc[i] = 0.f;
      xh[i] = has ? qn_apply(v[i], st.x, st.y) : 0.f;
      sg += acc[i];
      sgx = fmaf(acc[i], xh[i], sgx);
    }
    sg = group_sum<WAVE>(sg);
    sgx = group_sum<WAVE>(sgx);
    const float mg = sg / (float)n, mgx = sgx / (float)n;
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = st.y * (acc[i] - mg - xh[i] * mgx);
  }
  if (has) {
    float* o = grad_q + r * n + (size_t)p * d + e0;
#pragma unroll
    for (int i = 0; i < N; i += 4)
      *reinterpret_cast<float4*>(o + i) = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
  }
}

// Counting sort of the leaders by sub-key, each (head, half) for itself: its
// leaders go to its own T * k places of the pair array, so only the S sub-keys
// of one table are sorted over.  The leaders of one (token, head, half) row have
// distinct sub-keys, so a wave that takes a run of tile_tok tokens row by row
// ranks them with one returning LDS add per row, without ballots:
//   k_bin_count    counts per (head, half, tile, sub-key),
//   k_bin_scan     per sub-key an exclusive scan over the tiles, and its total,
//   k_bin_scatter  the sub-keys' starts (a scan of the totals by every wave),
//                  then (token, gradient sum) of each leader to its place; the
//                  first tile's waves also list the sub-keys of more than
//                  SBWD_LONG tokens.
// The keys come straight from the slots, the sub-key sums read their pairs in
// order.  At 32768 tokens, 4 heads, S = 2048, k = 32 (2.9M leaders) 22 + 9 + 65
// us, the scatter's 8-byte writes to 2048 running places per table being most of
// it (neither non-temporal reads nor reading a batch ahead changed that).  A scan
// of the counts, a packing of the leaders, two radix passes and the marking of
// segments in 13 launches took 157, and left the sums another gather (221 us
// with it, 179 without).
constexpr uint32_t SBWD_LONG = 2048;  // pairs of a sub-key beyond which k_sbwd_long sums them
constexpr int BIN_U = 16;             // rows in flight per wave

// f(token, lane's slot is filled, key, gradient sum) for the tile's rows in order.
template <bool VALS, typename F>
__device__ __forceinline__ void bin_rows(const uint32_t* __restrict__ keys,
                                         const float* __restrict__ gvals,
                                         const uint32_t* __restrict__ counts, int64_t t0, int64_t t1,
                                         int H, int hp, int k, F f) {
  const int lane = threadIdx.x;
  const int HP = 2 * H;
  const bool slot = lane < k;
  for (int64_t tb = t0; tb < t1; tb += WAVE) {
    const uint32_t c = tb + lane < t1 ? counts[(tb + lane) * HP + hp] : 0u;
    const int nt = t1 - tb < WAVE ? (int)(t1 - tb) : WAVE;
    for (int i = 0; i < nt; i += BIN_U) {
      uint32_t key[BIN_U];
      float g[BIN_U];
#pragma unroll
      for (int u = 0; u < BIN_U; ++u) {
        const bool has = slot && i + u < nt;
        const size_t x = has ? (size_t)((tb + i + u) * HP + hp) * k + lane : 0;
        key[u] = has ? keys[x] : 0u;
        g[u] = VALS && has ? gvals[x] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < BIN_U; ++u) {  // past nt the counts are 0 (i + u < 64)
        const uint32_t cu = (uint32_t)__builtin_amdgcn_readlane((int)c, i + u);
        f((uint32_t)(tb + i + u), (uint32_t)lane < cu, key[u], g[u]);
      }
    }
  }
}

__global__ __launch_bounds__(64) void k_bin_count(const uint32_t* __restrict__ keys,
                                                  const uint32_t* __restrict__ counts, int64_t ntok,
                                                  int H, int S, int k, int tile_tok,
                                                  uint32_t* __restrict__ mat,
                                                  uint32_t* __restrict__ long_cnt) {
  extern __shared__ uint32_t cnt[];  // [S]
  const int lane = threadIdx.x;
  const int hp = (int)(blockIdx.x % (unsigned)(2 * H));
  const int64_t tile = blockIdx.x / (unsigned)(2 * H);
  if (blockIdx.x == 0 && lane == 0) *long_cnt = 0;
  for (int b = lane; b < S; b += WAVE) cnt[b] = 0;
  __syncthreads();
  const int64_t t0 = tile * tile_tok, t1 = t0 + tile_tok < ntok ? t0 + tile_tok : ntok;
  const uint32_t key0 = (uint32_t)hp * (uint32_t)S;
  bin_rows<false>(keys, nullptr, counts, t0, t1, H, hp, k,
                  [&](uint32_t, bool has, uint32_t key, float) {
                    if (has) atomicAdd(&cnt[key - key0], 1u);
                  });
  __syncthreads();
  uint32_t* out = mat + (size_t)blockIdx.x * S;  // [tile][head, half][sub-key]
  for (int b = lane; b < S; b += WAVE) out[b] = cnt[b];
}

// 64 bins per workgroup, each by 16 threads with a run of the tiles each.
__global__ __launch_bounds__(1024) void k_bin_scan(uint32_t* __restrict__ mat, int64_t nbins,
                                                   int ntile, uint32_t* __restrict__ totals) {
  constexpr int U = 8;
  __shared__ uint32_t part[16][WAVE];
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t bin = (int64_t)blockIdx.x * WAVE + lane;
  const bool live = bin < nbins;
  const int per = (ntile + 15) / 16;
  const int a = grp * per < ntile ? grp * per : ntile;
  const int z = a + per < ntile ? a + per : ntile;
  uint32_t* m = mat + (live ? bin : 0);
  uint32_t sum = 0;
  for (int i = a; i < z; i += U) {
    uint32_t v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) v[j] = i + j < z ? m[(int64_t)(i + j) * nbins] : 0u;
#pragma unroll
    for (int j = 0; j < U; ++j) sum += v[j];
  }
  part[grp][lane] = sum;
  __syncthreads();
  uint32_t run = 0, all = 0;
#pragma unroll
  for (int g = 0; g < 16; ++g) {
    const uint32_t v = part[g][lane];
    run += g < grp ? v : 0u;
    all += v;
  }
  if (!live) return;
  if (grp == 0) totals[bin] = all;
  for (int i = a; i < z; i += U) {
    uint32_t v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) v[j] = i + j < z ? m[(int64_t)(i + j) * nbins] : 0u;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (i + j < z) m[(int64_t)(i + j) * nbins] = run;
      run += v[j];
    }
  }
}

__global__ __launch_bounds__(64) void k_bin_scatter(
    const uint32_t* __restrict__ keys, const float* __restrict__ gvals,
    const uint32_t* __restrict__ counts, int64_t ntok, int H, int S, int k, int tile_tok,
    const uint32_t* __restrict__ mat, const uint32_t* __restrict__ totals,
    uint32_t* __restrict__ starts, uint2* __restrict__ pairs, uint32_t* __restrict__ long_list,
    uint32_t* __restrict__ long_cnt) {
  extern __shared__ uint32_t cnt[];  // [S] the next place of each sub-key
  const int lane = threadIdx.x;
  const int hp = (int)(blockIdx.x % (unsigned)(2 * H));
  const int64_t tile = blockIdx.x / (unsigned)(2 * H);
  const uint32_t key0 = (uint32_t)hp * (uint32_t)S;
  const uint32_t* pre = mat + (size_t)blockIdx.x * S;
  uint32_t carry = (uint32_t)hp * (uint32_t)(ntok * k);  // the (head, half)'s own places
#pragma unroll 4
  for (int b0 = 0; b0 < S; b0 += 4 * WAVE) {
    const int b = b0 + lane * 4;
    uint32_t v[4], w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = b + i < S ? totals[key0 + b + i] : 0u;
      w[i] = b + i < S ? pre[b + i] : 0u;
    }
    const uint32_t mine = v[0] + v[1] + v[2] + v[3];
    uint32_t x = mine;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, WAVE);
      if (lane >= o) x += y;
    }
    uint32_t at = carry + x - mine;
    carry += (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (b + i < S) {
        cnt[b + i] = at + w[i];
        if (tile == 0) {
          starts[key0 + b + i] = at;
          if (v[i] > SBWD_LONG) long_list[atomicAdd(long_cnt, 1u)] = key0 + (uint32_t)(b + i);
        }
      }
      at += v[i];
    }
  }
  __syncthreads();
  const int64_t t0 = tile * tile_tok, t1 = t0 + tile_tok < ntok ? t0 + tile_tok : ntok;
  bin_rows<true>(keys, gvals, counts, t0, t1, H, hp, k,
                 [&](uint32_t t, bool has, uint32_t key, float g) {
                   if (has) pairs[atomicAdd(&cnt[key - key0], 1u)] = make_uint2(t, __float_as_uint(g));
                 });
}

// Where the sums find the sorted leaders: the counting sort's pairs with each
// sub-key's start and number, or the radix sort's keys, slots and segments.
struct SbwdPairs {
  const uint2* pairs;
  const uint32_t *starts, *totals;
  const float* gvals;
  const uint32_t *ks, *vs, *seg, *nseg;
};

// Adds gsum * (query half as scored) of the sorted pairs [a, z) of one
// (head h, half) segment into acc, in pair order: the pairs are taken 64 at a
// time and consumed QU at a time, with their query-quad loads issued
// together; lane l owns elements 4l..4l+3 of the half (qh points at them).
template <typename T, bool QN, bool BINS>
__device__ __forceinline__ void sbwd_sum_run(const T* qh, int H, int n, int h, uint32_t hk2,
                                             const float2* __restrict__ qstats,
                                             const SbwdPairs& in, uint32_t a, uint32_t z,
                                             int lane, float* acc) {
  constexpr int QU = PK_SBWD_QU;
  for (uint32_t b0 = a; b0 < z; b0 += 64) {
    const uint32_t e = b0 + lane;
    const bool ok = e < z;
    uint32_t t;
    float gx;
    if constexpr (BINS) {
      const uint2 pr = ok ? in.pairs[e] : uint2{0, 0};
      t = pr.x;
      gx = __uint_as_float(pr.y);
    } else {
      const uint32_t x = ok ? in.vs[e] : 0u;
      t = x / hk2;
      gx = ok ? in.gvals[x] : 0.f;
    }
    float2 st = make_float2(0.f, 1.f);
    if constexpr (QN) st = qstats[(size_t)t * H + h];
    const uint32_t cnt = (z - b0) < 64u ? (z - b0) : 64u;
    for (uint32_t j0 = 0; j0 < cnt; j0 += QU) {
      QQuad<T> qq[QU];
      float gg[QU], mj[QU], rj[QU];
#pragma unroll
      for (int j = 0; j < QU; ++j) {
        const bool has = j0 + j < cnt;
        const int L = has ? (int)(j0 + j) : (int)j0;
        const uint32_t tj = (uint32_t)__builtin_amdgcn_readlane((int)t, L);
        const float xj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gx), L));
        gg[j] = has ? xj : 0.f;
        if constexpr (QN) {
          mj[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st.x), L));
          rj[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st.y), L));
        }
        qq[j].load(qh + (size_t)tj * H * n);
      }
#pragma unroll
      for (int j = 0; j < QU; ++j) {
        if constexpr (QN) qq[j].fma_into_norm(gg[j], acc, mj[j], rj[j]);
        else qq[j].fma_into(gg[j], acc);
      }
    }
  }
}

// A segment of more than SBWD_LONG pairs (a sub-key chosen by that many
// tokens) is summed by k_sbwd_long instead of one wave.
constexpr int SBWD_LWAVES = 16;
static int64_t sbwd_max_long(int64_t np) { return np / SBWD_LONG + 1; }

// Segment u: its sub-key (over all heads and halves) and its pairs [s0, s1).
template <bool BINS>
__device__ __forceinline__ uint32_t sbwd_segment(const SbwdPairs& in, uint32_t u, uint32_t& s0,
                                                 uint32_t& s1) {
  if constexpr (BINS) {
    s0 = in.starts[u];
    s1 = s0 + in.totals[u];
    return u;
  } else {
    s0 = in.seg[u];
    s1 = in.seg[u + 1];
    return in.ks[s0];
  }
}

// One wave per segment (grid-stride) of the sorted pairs; a segment is one
// (head, half, sub-key) and holds at most one pair per token, in token order.
// Lane l owns elements 4l..4l+3 of the d-element row (d <= 256).  The sum is
// added into the sub-key row with one read-modify-write.
template <typename T, bool QN, bool BINS>
__global__ __launch_bounds__(256) void k_sbwd_segments(const T* __restrict__ q, int H, int n,
                                                       int S, int k,
                                                       const float2* __restrict__ qstats,
                                                       SbwdPairs in, float* __restrict__ grad_K) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t nbins = (uint32_t)(2 * H) * (uint32_t)S;
  const uint32_t nseg = BINS ? nbins : *in.nseg;
  const int d = n >> 1;
  const bool qlane = lane * 4 < d;
  const int ql = qlane ? lane * 4 : 0;
  const uint32_t hk2 = 2u * (uint32_t)H * (uint32_t)k;  // slots per token
  // Workgroups go to the 8 XCDs in turn; each XCD takes one contiguous eighth of
  // the segments (with 2H = 8 one head's half), whose waves walk the tokens at
  // about the same pace, so that a query half read for one sub-key is still in
  // the XCD's L2 for the others its token chose (245 -> 222 us at 32768 tokens,
  // 4 heads, S = 2048, and 178 with the counting sort's pairs; 36% of the requests
  // hit against 19%, no more as the paces drift apart).
  const uint32_t per = (nseg + 7u) / 8u;
  const uint32_t u0 = (blockIdx.x & 7u) * per;
  const uint32_t u1 = u0 + per < nseg ? u0 + per : nseg;
  for (uint32_t u = u0 + (blockIdx.x >> 3) * 4u + wave; u < u1; u += (gridDim.x >> 3) * 4u) {
    uint32_t s0, s1;
    const uint32_t bin = sbwd_segment<BINS>(in, u, s0, s1);
    if (bin >= nbins || s0 == s1 || s1 - s0 > SBWD_LONG) continue;
    const int hp = (int)(bin / (uint32_t)S);
    const int h = hp >> 1, p = hp & 1;
    const T* qh = q + (size_t)h * n + (size_t)p * d + ql;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    sbwd_sum_run<T, QN, BINS>(qh, H, n, h, hk2, qstats, in, s0, s1, lane, acc);
    if (qlane) {
      float4* dst = reinterpret_cast<float4*>(grad_K + (size_t)bin * d + ql);
      float4 o = *dst;
      o.x += acc[0]; o.y += acc[1]; o.z += acc[2]; o.w += acc[3];
      *dst = o;
    }
  }
}

// The segments listed in long_list, one workgroup of SBWD_LWAVES waves per
// segment at a time: wave w sums the w-th contiguous run of the segment's
// pairs (in pair order) into a partial row; the partial rows meet in LDS and
// are added, in wave order, to the sub-key row with one read-modify-write.
template <typename T, bool QN, bool BINS>
__global__ __launch_bounds__(64 * SBWD_LWAVES) void k_sbwd_long(
    const T* __restrict__ q, int H, int n, int S, int k, const float2* __restrict__ qstats,
    SbwdPairs in, const uint32_t* __restrict__ long_list, const uint32_t* __restrict__ long_cnt,
    float* __restrict__ grad_K) {
  __shared__ float part[SBWD_LWAVES][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d = n >> 1;
  const bool qlane = lane * 4 < d;
  const int ql = qlane ? lane * 4 : 0;
  const uint32_t nbins = (uint32_t)(2 * H) * (uint32_t)S;
  const uint32_t hk2 = 2u * (uint32_t)H * (uint32_t)k;
  const uint32_t nlong = *long_cnt;
  for (uint32_t it = blockIdx.x; it < nlong; it += gridDim.x) {
    uint32_t s0, s1;
    const uint32_t bin = sbwd_segment<BINS>(in, long_list[it], s0, s1);
    if (bin >= nbins) continue;  // the same for every wave of the workgroup
    const int hp = (int)(bin / (uint32_t)S);
    const int h = hp >> 1, p = hp & 1;
    const T* qh = q + (size_t)h * n + (size_t)p * d + ql;
    const uint32_t len = s1 - s0;
    const uint32_t per = (len + SBWD_LWAVES - 1) / SBWD_LWAVES;
    uint32_t a = (uint32_t)wave * per, z = a + per;
    a = s0 + (a < len ? a : len);
    z = s0 + (z < len ? z : len);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    sbwd_sum_run<T, QN, BINS>(qh, H, n, h, hk2, qstats, in, a, z, lane, acc);
    if (qlane) {
#pragma unroll
      for (int i = 0; i < 4; ++i) part[wave][ql + i] = acc[i];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < d; e += 64 * SBWD_LWAVES) {
      float sum = grad_K[(size_t)bin * d + e];
#pragma unroll
      for (int w = 0; w < SBWD_LWAVES; ++w) sum += part[w][e];
      grad_K[(size_t)bin * d + e] = sum;
    }
    __syncthreads();
  }
}

// grad_sink[h] += sum_t gz[t,h,sink slot] q[t,h], in two deterministic
// passes.  k_sink_partial: one workgroup per (chunk of SINK_TCH tokens, head);
// wave w takes the chunk's tokens w, w + 4, ... in order (SINK_U loads in
// flight), lane l owns elements 4l..4l+3 of each half; the four waves' sums
// are added in wave order into the chunk's partial row.  k_sink_reduce adds
// the partial rows in chunk order into grad_sink.
constexpr int SINK_TCH = 256;
constexpr int SINK_U = 8;
constexpr int SINK_NMAX = 512;  // n = 2d, d <= 256
int64_t sink_chunks(int64_t T) { return (T + SINK_TCH - 1) / SINK_TCH; }

template <typename T>
__global__ __launch_bounds__(256) void k_sink_partial(const T* __restrict__ q, int64_t ntok, int H,
                                                      int n, int kst, int k,
                                                      const float* __restrict__ gz,
                                                      float* __restrict__ part) {
  __shared__ float red[4][SINK_NMAX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = (int)(blockIdx.x % (unsigned)H);
  const int64_t c = blockIdx.x / (unsigned)H;
  const int d = n >> 1;
  const bool qlane = lane * 4 < d;
  const int ql = qlane ? lane * 4 : 0;
  const int64_t t0 = c * SINK_TCH;
  const int64_t t1 = t0 + SINK_TCH < ntok ? t0 + SINK_TCH : ntok;
  float acc[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int64_t tb = t0 + wave; tb < t1; tb += 4 * SINK_U) {
    QQuad<T> qa[SINK_U], qb[SINK_U];
    float g[SINK_U];
#pragma unroll
    for (int j = 0; j < SINK_U; ++j) {
      const int64_t t = tb + 4 * j;
      const bool has = t < t1;
      const size_t r = (size_t)(has ? t : tb) * H + h;
      g[j] = has ? gz[r * kst + k] : 0.f;
      qa[j].load(q + r * n + ql);
      qb[j].load(q + r * n + d + ql);
    }
#pragma unroll
    for (int j = 0; j < SINK_U; ++j) {
      qa[j].fma_into(g[j], acc[0]);
      qb[j].fma_into(g[j], acc[1]);
    }
  }
  if (qlane) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wave][p * d + ql + i] = acc[p][i];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += 256)
    part[((size_t)c * H + h) * n + e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
}

__global__ __launch_bounds__(256) void k_sink_reduce(const float* __restrict__ part, int64_t nch,
                                                     int Hn, float* __restrict__ grad_sink) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= Hn) return;
  float s = 0.f;
  for (int64_t c = 0; c < nch; ++c) s += part[(size_t)c * Hn + e];
  grad_sink[e] += s;
}

// Workspace: keys and group sums per slot (2*T*H*k each), the row counts, a
// spare part (a query for its size gives the same as ever), the list of long
// segments, then the sort of up to 2*T*H*k leaders: the radix sort's, or the
// counting sort's pairs (8 bytes each), tile counts, totals and starts.
static size_t a256(size_t x) { return (x + 255) / 256 * 256; }
static size_t sbwd_spare(int64_t rows) { return a256((size_t)((rows + 2048) / 2048 + 1) * 4); }
size_t search_backward_ws_bytes(int64_t T, int H, int k) {
  const int64_t rows = 2 * T * H;
  const int64_t np = rows * k;
  return 2 * a256((size_t)np * 4) + a256((size_t)(rows + 2) * 4) + sbwd_spare(rows) +
         a256((size_t)sbwd_max_long(np) * 4) + sorted_workspace_bytes(np);
}

// Tokens per wave of the counting sort, 0 where the radix sort is taken.  A wave's
// rows are a serial chain, so a tile is small, but it writes and twice reads S
// counts, so it has at least S / 2 slots, and there are at most about 2048 waves
// (whole search backward, us, at 16 / 32 / 64 / 128 / 256 tokens: 512 tokens S 512 28 /
// 31 / 37 / 50 / 77; 4096 tokens S 1024 68 / 65 / 68 / 81 / 107; 16384 tokens
// 235 / 217 / 205 / 207 / 228; 32768 tokens S 2048 - / 468 / 447 / 453 / 465).  Up
// to 8192 slots one workgroup sorts them all in one launch instead of three.
// The counts, totals and starts have to fit the radix sort's share of the
// workspace (sorted_workspace_bytes holds at least 6 words per slot, the pairs
// take 2), which larger tiles give for T * k >= S; below that the radix sort is
// taken.  It is also taken where S / 2 slots are many tokens, whose chain then
// lasts longer than its passes (radix / counting sort, H = 1, k = 1, S = 8192, 8192
// tokens 48 / 1528; k = 4, S = 2048, 4096 tokens, tiles of 256, 45 / 77; H = 4,
// k = 8, S = 8192, 32768 tokens, tiles of 512, 230 / 290; but 54 / 48 at k = 16,
// S = 2048, 4096 tokens, tiles of 64).  Tiles of 128 break even at about 2^20
// slots: k = 32, S = 8192, H = 1, 8192 tokens 87 / 107, H = 2 145 / 136.
constexpr int64_t BIN_TILE = 64, BIN_TILE_MANY = 128, BIN_MANY = (int64_t)1 << 20;
static int bin_tile_tokens(int64_t T, int H, int S, int k) {
  const int64_t np = 2 * T * H * k;
  if (np <= 8192) return 0;
  int tile = 16;
  while (tile * k < S / 2) tile *= 2;
  auto fits = [&](int t) { return ((T + t - 1) / t + 2) * 2 * H * S + 192 <= 4 * np; };
  while (tile < T && !fits(tile)) tile *= 2;
  if (tile > (np >= BIN_MANY ? BIN_TILE_MANY : BIN_TILE) || !fits(tile)) return 0;
  while (2 * H * (T / tile) > 2048) tile *= 2;
  return tile;
}

template <typename T>
static hipError_t launch_sbwd(const void* q, const void* subkeys, int64_t T_, int H, int n, int S,
                              int k, int kst, const int64_t* idx, const float* gz,
                              const float2* qstats, const void* sink, float* grad_q, float* grad_K,
                              float* grad_sink, float* sink_part, void* ws, hipStream_t st) {
  LaunchTimer lt("search_backward", st);
  hipError_t e = hipSuccess;
  if (grad_sink) {
    const int64_t nch = sink_chunks(T_);
    hipLaunchKernelGGL(k_sink_partial<T>, dim3((unsigned)(nch * H)), dim3(256), 0, st, (const T*)q,
                       T_, H, n, kst, k, gz, sink_part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int Hn = H * n;
    hipLaunchKernelGGL(k_sink_reduce, dim3((unsigned)((Hn + 255) / 256)), dim3(256), 0, st,
                       (const float*)sink_part, nch, Hn, grad_sink);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (!grad_q && !grad_K) return hipSuccess;
  const int64_t rows = 2 * T_ * H;
  const int64_t np = rows * k;
  char* p = reinterpret_cast<char*>(ws);
  uint32_t* keys = reinterpret_cast<uint32_t*>(p);
  p += a256((size_t)np * 4);
  float* gvals = reinterpret_cast<float*>(p);
  p += a256((size_t)np * 4);
  uint32_t* counts = reinterpret_cast<uint32_t*>(p);  // leaders per row
  p += a256((size_t)(rows + 2) * 4);
  void* ws_spare = p;
  p += sbwd_spare(rows);
  uint32_t* long_list = reinterpret_cast<uint32_t*>(p);
  p += a256((size_t)sbwd_max_long(np) * 4);
  void* sort_ws = p;
  const auto kq = k <= 32 ? k_search_bwd_q32<T> : k_search_bwd_q<T>;
  hipLaunchKernelGGL(kq, dim3((unsigned)(((T_ + 3) / 4) * H)), dim3(256), 0, st,
                     (const T*)q, (const T*)subkeys, T_, H, n, S, k, kst, idx, gz,
                     grad_q ? (const T*)sink : nullptr, qstats, grad_q,
                     grad_K ? keys : nullptr, grad_K ? gvals : nullptr, grad_K ? counts : nullptr);
  e = hipGetLastError();
  if (e != hipSuccess || !grad_K) return e;
  const uint32_t nbins = (uint32_t)(2 * H) * (uint32_t)S;
  const int tile = bin_tile_tokens(T_, H, S, k);
  SbwdPairs in{};
  const uint32_t* long_cnt;
  if (tile > 0) {
    const int64_t ntile = (T_ + tile - 1) / tile;
    uint2* pairs = reinterpret_cast<uint2*>(p);
    p += a256((size_t)np * 8);
    uint32_t* mat = reinterpret_cast<uint32_t*>(p);
    p += a256((size_t)ntile * nbins * 4);
    uint32_t* totals = reinterpret_cast<uint32_t*>(p);
    p += a256((size_t)nbins * 4);
    uint32_t* starts = reinterpret_cast<uint32_t*>(p);
    uint32_t* lcnt = reinterpret_cast<uint32_t*>(ws_spare);
    const dim3 g((unsigned)(ntile * 2 * H));
    const size_t lds = (size_t)S * 4;
    hipLaunchKernelGGL(k_bin_count, g, dim3(WAVE), lds, st, keys, counts, T_, H, S, k, tile, mat, lcnt);
    hipLaunchKernelGGL(k_bin_scan, dim3((nbins + WAVE - 1) / WAVE), dim3(1024), 0, st, mat,
                       (int64_t)nbins, (int)ntile, totals);
    hipLaunchKernelGGL(k_bin_scatter, g, dim3(WAVE), lds, st, keys, gvals, counts, T_, H, S, k, tile,
                       mat, totals, starts, pairs, long_list, lcnt);
    e = hipGetLastError();
    in.pairs = pairs;
    in.starts = starts;
    in.totals = totals;
    long_cnt = lcnt;
  } else {
    int key_bits = 1;
    while (key_bits < 32 && (uint64_t(1) << key_bits) < nbins) ++key_bits;
    in.gvals = gvals;
    e = sort_slots_segments(SortSrc{keys, counts, k}, np, key_bits, sort_ws, SBWD_LONG, long_list,
                            &in.ks, &in.vs, &in.seg, &in.nseg, &long_cnt, st);
  }
  if (e != hipSuccess) return e;
  int64_t maxseg = (int64_t)nbins < np ? (int64_t)nbins : np;
  if (tile > 0) maxseg = nbins;
  int64_t blocks = ((maxseg + 7) / 8 + 3) / 4 * 8;  // an eighth of the segments per XCD
  if (blocks > 16384) blocks = 16384;
  int64_t lblocks = sbwd_max_long(np) < maxseg ? sbwd_max_long(np) : maxseg;
  if (lblocks > 256) lblocks = 256;
  auto sums = [&](auto seg_kernel, auto long_kernel) {
    hipLaunchKernelGGL(seg_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const T*)q, H, n, S, k,
                       qstats, in, grad_K);
    hipLaunchKernelGGL(long_kernel, dim3((unsigned)lblocks), dim3(64 * SBWD_LWAVES), 0, st,
                       (const T*)q, H, n, S, k, qstats, in, (const uint32_t*)long_list, long_cnt,
                       grad_K);
  };
  if (tile > 0) {
    if (qstats) sums(k_sbwd_segments<T, true, true>, k_sbwd_long<T, true, true>);
    else sums(k_sbwd_segments<T, false, true>, k_sbwd_long<T, false, true>);
  } else {
    if (qstats) sums(k_sbwd_segments<T, true, false>, k_sbwd_long<T, true, false>);
    else sums(k_sbwd_segments<T, false, false>, k_sbwd_long<T, false, false>);
  }
  return hipGetLastError();
}

hipError_t launch_search_backward(bool bf16, const void* q, const void* subkeys, int64_t T, int H,
                                  int n, int S, int k, int kst, const int64_t* idx, const float* gz,
                                  const float2* qstats, const void* sink, float* grad_q,
                                  float* grad_K, float* grad_sink, float* sink_part, void* ws,
                                  hipStream_t st) {
  if (T <= 0) return hipSuccess;
  if (bf16)
    return launch_sbwd<uint16_t>(q, subkeys, T, H, n, S, k, kst, idx, gz, qstats, sink, grad_q,
                                 grad_K, grad_sink, sink_part, ws, st);
  return launch_sbwd<float>(q, subkeys, T, H, n, S, k, kst, idx, gz, qstats, sink, grad_q, grad_K,
                            grad_sink, sink_part, ws, st);
}

}  // namespace pk
