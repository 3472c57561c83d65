// Product-key search for few (token, head, half) rows on gfx950 (Sec. 3.1.1 of
// "Memory Layers at Scale"): decode batches and short prompts.
//
// k_score_topk gives a workgroup 512 tokens and all S sub-keys, so few tokens
// leave most of the chip idle and each workgroup still walks the whole table
// (1 token, S = 1024: 63 us on 8 workgroups, then four more launches).  Here
// the sub-keys are split instead:
//   * A workgroup of W waves owns R = 32 * W * TPW consecutive sub-keys of one
//     (head, half), a "part"; each wave holds its 32 sub-keys as MFMA A
//     fragments in registers and the tokens stream past them in groups of 32
//     (B fragments through LDS), so a workgroup reads its sub-keys once.
//     `slices` workgroups share a part and take every slices-th group.
//   * The products are the same chains of the same MFMAs as k_score_topk's,
//     so the scores are bitwise its scores.  A group's 32 x R scores go to LDS
//     and each wave selects for its share of the tokens: a lane holds R / 64
//     scores, the k-th largest of the 64 lane maxima (their upper 16 ordered
//     bits, found bit by bit with ballots) is a threshold that at least k
//     scores reach, and the scores at or above it (about 37 of 512 at k = 32)
//     are the part's records.  More than 64 of them (large k, ties) are cut to
//     the exact top k, lower index first on ties, by a bit search over the
//     scores themselves.  So every part has at most 64 records per token, none
//     of its top k is ever lost, and there is no rescan, no counter to clear
//     and no launch for either.
//   * A part's 64 record slots per token (64-bit (score, ~row) keys, empty
//     slots 0) lie in the candidate runs of the workspace: 8192 per group of
//     32 tokens, head and half, which bounds the parts (split_plan).
// k_cartesian merges the parts of both halves itself.
#include "pk_device.h"
#include "pk_internal.h"
#include "pk_mfma.h"

namespace pk {

constexpr int SPLIT_RECS = 64;  // record slots per token and part

template <typename T, int NSTEP, int W, int TPW>
__global__ __launch_bounds__(64 * W, 4) void k_score_split(
    const T* __restrict__ q, const T* __restrict__ subkeys, int64_t ntok, int H, int n, int S,
    int k, const float2* __restrict__ qstats, const T* __restrict__ sink,
    float* __restrict__ sink_part, int parts, int cap, int slices, uint64_t* __restrict__ cand) {
  using M = MfmaOp<T>;
  constexpr int DPAD = NSTEP * M::KSTEP;
  constexpr int NCOL = DPAD * M::ESIZE / 16;  // 16-byte segments per query half
  constexpr int RBP = (NCOL + 1) * 16;        // query pitch in LDS: an odd number of them
  constexpr int EPS = 16 / M::ESIZE;
  constexpr int R = 32 * W * TPW;             // sub-keys per part
  constexpr int E = R / WAVE;                 // scores per lane and token
  constexpr int PITCH = R + 4;                // floats per token: odd in 16-byte units
  constexpr int NT = TPW > 1 ? 1 : 2;         // tokens a wave selects for side by side
  constexpr int NQ = (32 * NCOL + 64 * W - 1) / (64 * W);
  constexpr int CS = NCOL < 8 ? NCOL : 8;     // segments of a row loaded together
  constexpr int KL = (CS + 1) / 2;            // loads for 32 rows of them
  constexpr int SPC = CS * EPS / M::KSTEP;    // MFMA steps in them
  constexpr int KP = ((CS + 1) | 1) * 16;     // their pitch in LDS
  constexpr int KBUF = 32 * KP;               // one wave's
  constexpr int SMEM = 32 * PITCH * 4 > W * KBUF ? 32 * PITCH * 4 : W * KBUF;
  __shared__ __align__(16) unsigned char qbuf[32 * RBP];
  // the group's scores; the key rows on their way in before that
  __shared__ __align__(16) unsigned char smem[SMEM];
  float* const sc = reinterpret_cast<float*>(smem);
  __shared__ uint2 stage[W][NT][SPLIT_RECS];  // (row, score bits)

  const int d = n >> 1;
  const int HP = 2 * H;
  const int hp = blockIdx.x % HP;
  const int part = (int)(blockIdx.x / HP) % parts;
  const int64_t slice = blockIdx.x / HP / parts;
  const int h = hp >> 1, p = hp & 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kh = lane >> 5, col = lane & 31;
  const int64_t ngroups = (ntok + 31) / 32;
  const uint32_t rot = (uint32_t)(cap / parts);
  const T* kbase = subkeys + (size_t)hp * S * d;

  // The wave's 32 sub-keys of tile i as A fragments.  A fragment load straight
  // from memory touches 32 bytes of each of 32 rows, and 16 waves of them
  // outrun the 32 KiB L1, so every line would come four times; instead the
  // rows are read CS segments (up to a whole 128-byte line) at a time and
  // turned into fragments through the wave's own LDS.
  typename M::frag ak[NSTEP];
  auto load_keys = [&](int i) PK_INLINE {
    const int row0 = part * R + (wave * TPW + i) * 32;
    if constexpr (TPW > 1) {  // smem holds scores by now, and one tile's fragments are all
                              // the registers there are
      const int r = row0 + col;
      const T* kr = kbase + (size_t)(r < S ? r : S - 1) * d;
#pragma unroll
      for (int s = 0; s < NSTEP; ++s) {
        const int e0 = s * M::KSTEP + kh * M::LANE_K;
        ak[s] = e0 + M::LANE_K <= d ? M::load(kr + e0) : M::zero();
      }
      return;
    }
    unsigned char* const kb = reinterpret_cast<unsigned char*>(smem) + wave * KBUF;
    uint4 raw[NCOL / CS][KL];
#pragma unroll
    for (int c = 0; c < NCOL / CS; ++c)
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        const int x = j * WAVE + lane;  // row x / CS, segment c * CS + x % CS
        const int r = row0 + x / CS;
        const int e0 = (c * CS + x % CS) * EPS;
        raw[c][j] = x < 32 * CS && e0 < d ? ld16(kbase + (size_t)(r < S ? r : S - 1) * d + e0)
                                          : uint4{0, 0, 0, 0};
      }
#pragma unroll
    for (int c = 0; c < NCOL / CS; ++c) {
#pragma unroll
      for (int j = 0; j < KL; ++j) {
        const int x = j * WAVE + lane;
        if (x < 32 * CS) *reinterpret_cast<uint4*>(kb + x / CS * KP + x % CS * 16) = raw[c][j];
      }
#pragma unroll
      for (int s = 0; s < SPC; ++s)
        ak[c * SPC + s] = M::load(kb + col * KP + (s * M::KSTEP + kh * M::LANE_K) * M::ESIZE);
    }
  };
  // Segment tid + j * 64 W of the group's 32 x NCOL query segments (zeros past
  // the tokens and past d), normalised when qstats is given.
  uint4 qseg[NQ];
  auto load_queries = [&](int64_t g) PK_INLINE {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int i = tid + j * 64 * W;
      const int64_t t = g * 32 + i / NCOL;
      const int e0 = i % NCOL * EPS;
      const bool ok = i < 32 * NCOL && t < ntok && e0 < d;
      const size_t qr = ok ? (size_t)t * H + h : 0;
      uint4 u = ok ? ld16(q + qr * n + (size_t)p * d + e0) : uint4{0, 0, 0, 0};
      if (qstats && ok) {
        const float2 qs = qstats[qr];
        if constexpr (M::ESIZE == 2) {
          u = __builtin_bit_cast(uint4, M::normalize(__builtin_bit_cast(typename M::frag, u), qs.x, qs.y));
        } else {
          u.x = __float_as_uint(qn_apply(__uint_as_float(u.x), qs.x, qs.y));
          u.y = __float_as_uint(qn_apply(__uint_as_float(u.y), qs.x, qs.y));
          u.z = __float_as_uint(qn_apply(__uint_as_float(u.z), qs.x, qs.y));
          u.w = __float_as_uint(qn_apply(__uint_as_float(u.w), qs.x, qs.y));
        }
      }
      qseg[j] = u;
    }
  };
  // A staged record: element e of the lane, row part * R + e * 64 + lane.
  const uint32_t row0 = (uint32_t)(part * R + lane);
  auto put = [&](uint2* st, uint32_t at, float z, int e) PK_INLINE {
    st[at] = make_uint2(row0 + (uint32_t)(e * WAVE), __float_as_uint(z));
  };
  auto rank_in = [](uint64_t m, uint32_t base) PK_INLINE {  // base + lanes of m below this one
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
  };

  load_queries(slice);
  if constexpr (TPW == 1) load_keys(0);
  for (int64_t g = slice; g < ngroups; g += slices) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int i = tid + j * 64 * W;
      if (i < 32 * NCOL) *reinterpret_cast<uint4*>(qbuf + i / NCOL * RBP + i % NCOL * 16) = qseg[j];
    }
    __syncthreads();  // the queries are in LDS; the previous group's scores are used up
#pragma unroll 1
    for (int i = 0; i < TPW; ++i) {
      if constexpr (TPW > 1) load_keys(i);
      const unsigned char* qp = qbuf + col * RBP + kh * M::LANE_K * M::ESIZE;
      f32x16_t acc{};
      typename M::frag bq[2];
      bq[0] = M::load(qp);
#pragma unroll
      for (int s = 0; s < NSTEP; ++s) {
        if (s + 1 < NSTEP) bq[(s + 1) & 1] = M::load(qp + (s + 1) * M::KSTEP * M::ESIZE);
        __builtin_amdgcn_sched_barrier(0);  // one step ahead of its use, no further (registers)
        acc = M::mma(ak[s], bq[s & 1], acc);
        __builtin_amdgcn_sched_barrier(0);
      }
      const int r0 = (wave * TPW + i) * 32;
      if (part * R + r0 + 32 > S) {  // rows past S: NaN, at or above no threshold
#pragma unroll
        for (int j = 0; j < 16; ++j)
          acc[j] = part * R + r0 + acc_row(j, kh) < S ? acc[j] : __uint_as_float(0xFFC00000u);
      }
#pragma unroll
      for (int j = 0; j < 16; j += 4)
        *reinterpret_cast<float4*>(&sc[col * PITCH + r0 + acc_row(j, kh)]) =
            make_float4(acc[j], acc[j + 1], acc[j + 2], acc[j + 3]);
    }
    const int64_t t0 = g * 32;
    const int nt = ntok - t0 < 32 ? (int)(ntok - t0) : 32;
    if (sink && part == 0) {  // this half's part of q . sink[h], from the queries in LDS
      const bool has = lane * 4 < d;
      for (int tl = wave; tl < nt; tl += W) {
        float a = 0.f;
        if (has) {
          QQuad<T> qa, sa;
          qa.load(reinterpret_cast<const T*>(qbuf + tl * RBP) + lane * 4);
          sa.load(sink + (size_t)h * n + (size_t)p * d + lane * 4);
          float fa[4], fs[4];
          qa.to_f32(fa);
          sa.to_f32(fs);
#pragma unroll
          for (int i = 0; i < 4; ++i) a = fmaf(fa[i], fs[i], a);
        }
        a = group_sum<WAVE>(a);
        if (lane == 0) sink_part[((size_t)(t0 + tl) * H + h) * 2 + p] = a;
      }
    }
    __syncthreads();  // the scores are in LDS; the queries are used up
    if (g + slices < ngroups) load_queries(g + slices);  // in flight under the selection

    uint64_t* const run = cand + ((size_t)g * HP + hp) * (32 * CAND_CAP);
    for (int tl = wave; tl < nt; tl += NT * W) {
      float v[NT][E];
      uint32_t u[NT], thr[NT];
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        const int t = tl + a * W < nt ? tl + a * W : tl;
#pragma unroll
        for (int e = 0; e < E; ++e) v[a][e] = sc[t * PITCH + e * WAVE + lane];
        float mx = v[a][0];
#pragma unroll
        for (int e = 1; e < E; ++e) mx = fmaxf(mx, v[a][e]);
        u[a] = mx == mx ? f32_to_ordered(mx) : 0u;  // 0: no row in this lane
        thr[a] = 0;
      }
#pragma unroll
      for (int b = 31; b >= 16; --b)
#pragma unroll
        for (int a = 0; a < NT; ++a) {
          const uint32_t c = thr[a] | (1u << b);
          if (__popcll(__builtin_amdgcn_ballot_w64(u[a] >= c)) >= k) thr[a] = c;
        }
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        if (tl + a * W >= nt) break;  // the same for the whole wave
        uint2* const st = stage[wave][a];
        // as a float; -inf (which a product past the float range may be) where
        // fewer than k lanes hold a row
        const float tf = thr[a] < 0x00800000u ? -INFINITY : ordered_to_f32(thr[a]);
        uint32_t cnt = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) cnt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(v[a][e] >= tf));
        if (cnt <= (uint32_t)cap) {
          uint32_t base = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(v[a][e] >= tf);
            if (v[a][e] >= tf) put(st, rank_in(m, base), v[a][e], e);
            base += (uint32_t)__popcll(m);
          }
        } else {  // the exact top k of the part
          // A score that is no number (products past the float range of both
          // signs) counts below every other, as in the compares that take the
          // records: its sign is set, as that of the rows past S is.
#pragma unroll
          for (int e = 0; e < E; ++e)
            v[a][e] = v[a][e] == v[a][e] ? v[a][e] : __uint_as_float(0xFFC00000u);
          uint32_t x = 0;  // the k-th largest score (at least k lie at or above tf)
          for (int b = 31; b >= 0; --b) {
            const uint32_t c = x | (1u << b);
            uint32_t have = 0;
#pragma unroll
            for (int e = 0; e < E; ++e)
              have += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(f32_to_ordered(v[a][e]) >= c));
            if (have >= (uint32_t)k) x = c;
          }
          const float xf = ordered_to_f32(x);
          uint32_t base = 0;
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(v[a][e] > xf);
            if (v[a][e] > xf) put(st, rank_in(m, base), v[a][e], e);
            base += (uint32_t)__popcll(m);
          }
#pragma unroll
          for (int e = 0; e < E; ++e) {  // ties in row order
            const uint64_t m = __builtin_amdgcn_ballot_w64(v[a][e] == xf);
            const uint32_t at = rank_in(m, base);
            if (v[a][e] == xf && at < (uint32_t)k) put(st, at, v[a][e], e);
            base += (uint32_t)__popcll(m);
          }
          cnt = base < (uint32_t)k ? base : (uint32_t)k;  // the records staged
        }
        // Slots rotated by part, so that the merge's lanes (every 64th slot of
        // the token's each) hold about as many records each.
        const uint2 rec = st[lane];
        const uint64_t key = (uint32_t)lane < cnt ? make_key(__uint_as_float(rec.y), rec.x) : 0ull;
        const uint32_t slot = ((uint32_t)lane + (uint32_t)part * rot) & (uint32_t)(cap - 1);
        if (lane < cap) run[((size_t)(tl + a * W) * parts + part) * cap + slot] = key;
      }
    }
  }
}

// The most rows (T * 2H) for which the path is taken, besides rows * S < 2^26
// (split / many as ratios of whole searches, over d 8 to 256 and both dtypes):
//   * up to k = 36, by the sub-keys: a part costs the same however few of its rows
//     exist, while the many-row kernel fills the chip from 2^15 to 2^17 rows in
//     three steps, whatever S.  k = 8: S = 64 2^15 rows 1.08-1.19, 2^17 1.43-1.57; S = 128
//     2^15 0.99-1.05, 2^16 1.06-1.14; S = 256 70000 0.87-0.98, 90000 0.98-1.07; S = 400 90000
//     0.80-0.97, 2^17 1.02-1.19.  k = 32: S = 64 2^16 0.93-1.04, 90000 1.05-1.14; S = 128
//     90000 0.95-1.02, 2^17 1.17-1.27; S = 400 2^17 0.99-1.10.
//   * from there to k = 56 more and more parts have over 64 records and take the
//     exact cut, so the rows are counted once per part.  k = 40: S = 128 90000 0.90-0.97;
//     S = 1024 2^15 rows 121 / 96 us, fp32 154 / 162; S = 2048 2^14 rows 115 / 96, fp32 147 /
//     222.  k = 44: S = 512 2^15 101 / 91, 2^16 186 / 144; S = 1024 2^14 94 / 83, 2^15 167 / 106;
//     S = 2048 2^13 89 / 96, 2^14 162 / 108.
//   * past k = 56 the many-row kernel's threshold leaves so many records that it
//     rescans (k = 60, S = 1024, 2^14 rows 115 / 211 us; k = 64, S = 512, 2^15 128 / 1429),
//     but not of 256 sub-keys or fewer (k = 64: S = 64 90000 0.80-0.86, S = 128 2^16 0.99-1.02,
//     90000 1.22-1.25; S = 256 90000 0.95-0.98).
static int64_t split_rows_max(bool bf16, int S, int k, int parts) {
  if (k <= 16) {
    if (S <= 128) return 1 << 15;
    if (S <= 256) return k > 4 ? 5 << 14 : 1 << 16;
    return k > 8 ? 7 << 14 : 3 << 15;
  }
  if (k <= 36) return S <= 64 ? 1 << 16 : S <= 256 ? 3 << 15 : 1 << 17;
  if (k <= 40) return S <= 256 ? 3 << 15 : (1 << 16) / parts;
  if (k <= 56) return (bf16 ? 1 << 15 : 1 << 16) / parts;
  if (S <= 256) return S > 64 && S <= 128 ? 1 << 16 : 3 << 15;
  return INT64_MAX;
}

// Which calls take this path, the sub-keys per part, the record slots per token
// and part, and how many workgroups share a part (whole searches in us, as HIP
// graphs; bf16, H = 4, n = 512, k = 32 where nothing else is said; rows = T * 2H).
//   * rows * S < 2^26: below it the split is the faster path.  S = 2048: 16
//     against 130 at 32 tokens, 66 against 106 at 2000 (k_score_topk at its
//     best workgroup size), 115 against 118 at 4000, 210 against 167 at 8000;
//     S = 1024: 73 against 90 at 4000, 127 against 128 at 8000.
//   * split_rows_max above.
//   * Parts of 1024 rows read their keys from L2 for every group, so rows * parts *
//     max(d, 128) <= 3072 * S (S = 2049, 3 parts: d = 64 12000 rows 60 / 71, 16000 90 / 73;
//     d = 256 8192 rows 82 / 91, 10000 102 / 92; S = 4096, d = 256: 10000 rows 126 / 143,
//     16000 195 / 147).
//   * R = 512 where the call then still has a workgroup per CU (fewer records
//     to merge: S = 1024, 2000 tokens 44 against 48), else 256 (32 tokens: 14
//     against 16).  R = 128 gains nothing (T = 1: 12.5 against 11.7).
//   * The parts must fit the token's share of its group's run (8192 records for
//     up to 32 tokens) and the merge's 16 records per lane.  Tables past that
//     take R = 1024 in bf16 (the keys then come from L2 for every group, as
//     two tiles' fragments outgrow the registers), and past that, up to
//     k = 32, slots for exactly the top k: S = 8192, 64 tokens 56 against 243,
//     but 190 against 250 at 500 tokens, so only for rows * S < 2^25.
bool split_plan(bool bf16, int64_t T, int H, int n, int S, int k, SplitPlan* plan) {
  const int64_t work = T * H * 2 * S;
  if (work >= (int64_t)1 << 26) return false;
  const int slots = 32 * CAND_CAP / (T < 32 ? (int)T : 32);
  const int64_t groups = (T + 31) / 32;
  int cap = SPLIT_RECS;
  auto parts_of = [&](int R) { return (S + R - 1) / R; };
  auto fits = [&](int R) { return parts_of(R) <= SPLIT_PARTS_MAX && parts_of(R) * cap <= slots; };
  int R = 2 * H * parts_of(512) * groups >= 256 ? 512 : 256;
  if (!fits(R)) R = 512;
  if (!fits(R)) {
    if (!bf16) return false;
    R = 1024;
    if (!fits(R) && k <= 32 && work < (int64_t)1 << 25) cap = 32;
    if (!fits(R)) return false;
  }
  const int parts = parts_of(R);
  const int64_t rows = T * 2 * H;
  if (rows > split_rows_max(bf16, S, k, parts)) return false;
  if (R == 1024 && rows * parts * (n > 256 ? n / 2 : 128) > (int64_t)3072 * S) return false;
  // One workgroup per CU of 16 waves, two of 8, and none beyond: a few more would
  // run as a second round on nearly idle CUs (3 parts of 8 tables, 128 groups,
  // k = 32: 122 us as 264 workgroups, 86 as 240).  With parts of 1024 rows, which
  // are bound by their key reads, a short last part ends early and rounding up
  // is better on the whole (8 tables, 32 groups, 264 / 192 workgroups: S = 2049 52
  // / 63 us, S = 2500 57 / 65; but 64 groups of S = 3000 122 / 104).
  const int64_t cus = R >= 512 ? 256 : 512, unit = (int64_t)2 * H * parts;
  int64_t slices = R == 1024 ? (cus + unit - 1) / unit : cus / unit;
  if (slices > groups) slices = groups;
  if (slices < 1) slices = 1;
  const int64_t per = (groups + slices - 1) / slices;  // groups per workgroup, evened out
  *plan = SplitPlan{R, parts, cap, (int)((groups + per - 1) / per)};
  return true;
}

template <typename T, int NSTEP>
static hipError_t split_launch(const void* q, const void* subkeys, int64_t T_, int H, int n, int S,
                               int k, const float2* qstats, const void* sink, float* sink_part,
                               const SplitPlan& pl, uint64_t* cand, hipStream_t st) {
  const dim3 g((unsigned)(2 * H * pl.parts) * (unsigned)pl.slices);
  LaunchTimer lt("score_topk", st);
#define PK_SPLIT(W, TPW)                                                                          \
  hipLaunchKernelGGL((k_score_split<T, NSTEP, W, TPW>), g, dim3(64 * W), 0, st, (const T*)q,      \
                     (const T*)subkeys, T_, H, n, S, k, qstats, (const T*)sink, sink_part,        \
                     pl.parts, pl.cap, pl.slices, cand)
  if (pl.rows == 256) PK_SPLIT(8, 1);
  else if (pl.rows == 512) PK_SPLIT(16, 1);
  else if constexpr (sizeof(T) == 2) PK_SPLIT(16, 2);
#undef PK_SPLIT
  return hipGetLastError();
}

hipError_t launch_search_split(bool bf16, const void* q, const void* subkeys, int64_t T, int H,
                               int n, int S, int k, const float2* qstats, const void* sink,
                               float* sink_part, const SplitPlan& pl, uint64_t* cand,
                               hipStream_t st) {
  const int d = n / 2;
#define PK_STEPS(TY, N) \
  return split_launch<TY, N>(q, subkeys, T, H, n, S, k, qstats, sink, sink_part, pl, cand, st)
  if (bf16) {
    const int steps = (d + 15) / 16;
    if (steps <= 1) PK_STEPS(uint16_t, 1);
    if (steps <= 2) PK_STEPS(uint16_t, 2);
    if (steps <= 4) PK_STEPS(uint16_t, 4);
    if (steps <= 8) PK_STEPS(uint16_t, 8);
    PK_STEPS(uint16_t, 16);
  }
  const int steps = (d + 1) / 2;
  if (steps <= 2) PK_STEPS(float, 2);
  if (steps <= 4) PK_STEPS(float, 4);
  if (steps <= 8) PK_STEPS(float, 8);
  if (steps <= 16) PK_STEPS(float, 16);
  PK_STEPS(float, 32);
#undef PK_STEPS
}

}  // namespace pk
