// Sparse contraction S_raw[i][j] = (1 / l_i) sum over the distinct words u of
// target sentence j of T'[i][u] (Sec. 4), with the logistic scorer fused into
// its epilogue.
//
// Y is a 0/1 matrix with a few dozen ones per row: a target sentence's score
// against a source sentence is a sum of that many entries of T', far fewer
// than the words of a 64 x 64 tile's vocabulary.
//
// k_tgt_lists   one workgroup per column tile: each target sentence's distinct
//               words, ascending, and the tile's sentences ordered by how many
//               they hold.
// k_score_s     one workgroup per SROWS source sentences x up to SCOLS column
//               tiles.  The merged dictionary rows become a dense LDS table
//               over their own vocabulary (one line of SROWS values per word;
//               line 0 is all zero) and a table that takes a word to its line
//               (absent words to line 0).  Each wave then takes groups of 16
//               target sentences and sums the lines of their words.
//
// Lane l of a group works for sentence l & 15; kq = l >> 4 is its place among
// the four lanes of that sentence.
//   BF16: v_mfma_f32_16x16x32_bf16 does the sums.  Its B operand is two words'
//         lines as they lie in LDS (lane: 8 rows of word kq >> 1), its A
//         operand the constant 0/1 matrix that adds the two.
//   FP32: lane kq adds rows 4 kq .. 4 kq + 3 of every word, in ascending word
//         order, each partial sum rounded to FP32: bit for bit the chain of
//         FP32 multiply-adds that v_mfma_f32_16x16x4_f32 performs over the
//         same words in ascending K order (measured: it rounds after every K
//         step), at a fraction of its time.
// In both, the lane ends with rows 4 kq .. 4 kq + 3 of its sentence.
//
// What bounds it: the LDS reads of the lines (about 9 cycles per 16-byte read
// of a wave at random lines, 16 rows x 16 sentences x 2 words for BF16, 1 for
// FP32) and the integer work of finding them, at 12 to 16 waves a compute unit;
// on short runs the table's construction (about 11k cycles of mostly memory
// latency).  Sixteen rows, because their vocabulary (530 to 820 words) leaves
// room for four workgroups a compute unit; the tile's sentences in order of
// length, because a group walks as many words as its longest sentence holds
// (23 instead of 31 on average).  Measured on the benchmark corpora, against
// k_score_c: 64 pairs of 5000 x 5000, V = 16384, BF16 4.96 -> 3.61 ms; 4096
// pairs, V = 4096, FP32 1.56 -> 0.67 ms (BF16 0.43 -> 0.46 ms, the expansion
// before it 0.45 -> 0.40 ms); one pair of 200 x 220, FP32 57 -> 13 us.
#include "nwm_internal.h"
#include "libnwmine.h"
#include "nwm_score.h"

#include <algorithm>

namespace nwm {

static __device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

static __device__ __forceinline__ int s_uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

typedef unsigned int s_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int s_u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 s_bf16x8 __attribute__((ext_vector_type(8)));
typedef float s_f32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t LIST_NONE = 0xFFFFFFF0u;   // buffer offset past any list

// Word lists, in granules of 8 16-bit slots (16 bytes), a list's last granule
// padded.  Word u is slot u + 32; slot 0 is padding (its table entry is empty).
// Lane kq of k_score_s wants words c and c + 4 of every granule, c = 0, 2, 1, 3
// for kq = 0..3, as one dword, and up to four granules in one 16-byte load: a
// block of four granules (fewer at the list's end) holds the dwords of lane
// kq = 0 for each of its granules, then those of lane 1, 2, 3.
// First granule of target sentence `sent` whose tokens start at `off`: a list
// of at most the sentence's tokens ends before the next one starts.
static __device__ __forceinline__ int64_t list_granule(int64_t off, int64_t sent) { return (off + 8 * sent) >> 3; }
// 16-bit place of word i of a list of ng granules
static __device__ __forceinline__ int slot_place(int i, int ng) {
  const int c = i & 3, kq = (c >> 1) | ((c & 1) << 1), blk = i >> 5, g = min(4, ng - 4 * blk);
  return 32 * blk + 2 * (kq * g + ((i >> 3) & 3)) + ((i >> 2) & 1);
}
constexpr int LIST_SLACK = 64;   // bytes past the last list a 16-byte load may touch

// ---- target lists -------------------------------------------------------------

// k_tgt_lists is bound by instruction issue: a rank by comparison with every
// other word took 262 us for the 4096-pair benchmark workload, the network 103.
// Each half of a wave sorts one sentence's first 32 tokens (one per lane) and,
// when either sentence is longer, its next 32, then merges the two: a sorting
// network of DPP and lane-row exchanges, no LDS.  Lane l of a half exchanges
// with lane l ^ D of the half and keeps the smaller value where (l & BIT) is
// clear.
template <int D>
static __device__ __forceinline__ uint32_t half_xor(uint32_t x) {
  auto dpp = [](uint32_t v, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, true);
  };
  if constexpr (D == 1) return dpp(x, std::integral_constant<int, 0xB1>{});          // quad_perm 1,0,3,2
  else if constexpr (D == 2) return dpp(x, std::integral_constant<int, 0x4E>{});     // quad_perm 2,3,0,1
  else if constexpr (D == 3) return dpp(x, std::integral_constant<int, 0x1B>{});     // quad_perm 3,2,1,0
  else if constexpr (D == 7) return dpp(x, std::integral_constant<int, 0x141>{});    // row_half_mirror
  else if constexpr (D == 15) return dpp(x, std::integral_constant<int, 0x140>{});   // row_mirror
  else if constexpr (D == 8) return dpp(x, std::integral_constant<int, 0x128>{});    // row_ror 8
  else if constexpr (D == 4) return half_xor<3>(half_xor<7>(x));
  else {
    static_assert(D == 16 || D == 31, "exchange distance");
    const uint32_t y = D == 31 ? half_xor<15>(x) : x;
    const auto s = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    return (threadIdx.x & 16) ? s[0] : s[1];
  }
}
template <int D, int BIT>
static __device__ __forceinline__ uint32_t sort_step(uint32_t x) {
  const uint32_t y = half_xor<D>(x);
  return (threadIdx.x & BIT) ? max(x, y) : min(x, y);
}
// the last steps of a 32-lane merge
static __device__ __forceinline__ uint32_t sort_clean(uint32_t x) {
  return sort_step<1, 1>(sort_step<2, 2>(sort_step<4, 4>(sort_step<8, 8>(x))));
}
static __device__ __forceinline__ uint32_t sort32(uint32_t x) {
  x = sort_step<1, 1>(x);
  x = sort_step<1, 1>(sort_step<3, 2>(x));
  x = sort_step<1, 1>(sort_step<2, 2>(sort_step<7, 4>(x)));
  x = sort_step<1, 1>(sort_step<2, 2>(sort_step<4, 4>(sort_step<15, 8>(x))));
  return sort_clean(sort_step<31, 16>(x));
}

constexpr int TL_WAVES = 4;

__global__ __launch_bounds__(64 * TL_WAVES) void k_tgt_lists(const TileMeta *__restrict__ ct_meta, int c0,
                                                             const int64_t *__restrict__ tgt_off,
                                                             const int32_t *__restrict__ tgt_tok, int V,
                                                             uint16_t *__restrict__ list, uint2 *__restrict__ rec,
                                                             float *__restrict__ tlen) {
  extern __shared__ __align__(16) uint32_t tl_bits[];   // TL_WAVES x ceil(V / 32)
  __shared__ int tl_cnt[TN];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int words = (V + 31) / 32;
  uint32_t *bits = tl_bits + wave * words;
  const TileMeta tm = ct_meta[c0 + (int)blockIdx.x];
  constexpr int PER = TN / TL_WAVES;   // sentences per wave, two at a time
  constexpr uint32_t NONE = 0xFFFFFFFFu;
  const int hl = lane & 31, half = lane >> 5;
  // the half's sentence of round k: wave's sentences are PER wave ..
  auto sent_of = [&](int k) { return PER * wave + 2 * k + half; };
  // a lane's token x of its half's sentence
  int64_t off[PER / 2];
  int len[PER / 2];
  uint32_t t0[PER / 2], t1[PER / 2];
#pragma unroll
  for (int k = 0; k < PER / 2; ++k) {
    const bool v = sent_of(k) < tm.count;
    const int64_t s = tm.first + (v ? sent_of(k) : 0);
    off[k] = tgt_off[s];
    len[k] = v ? (int)min(tgt_off[s + 1] - off[k], (int64_t)0x7FFFFFFF) : 0;
  }
#pragma unroll
  for (int k = 0; k < PER / 2; ++k) {
    t0[k] = hl < len[k] ? (uint32_t)tgt_tok[off[k] + hl] : NONE;
    t1[k] = 32 + hl < len[k] ? (uint32_t)tgt_tok[off[k] + 32 + hl] : NONE;
  }
#pragma unroll
  for (int k = 0; k < PER / 2; ++k) {
    if (s_uniform(PER * wave + 2 * k) >= tm.count) break;
    const bool v = sent_of(k) < tm.count;
    const int64_t sent = tm.first + sent_of(k);
    uint16_t *out = list + 8 * list_granule(off[k], sent);
    // (a token outside the vocabulary is dropped)
    uint32_t a = sort32(t0[k] < (uint32_t)V ? t0[k] : NONE), b = NONE;
    const bool two = __ballot(len[k] > 32) != 0ull;
    if (two) {
      b = half_xor<31>(sort32(t1[k] < (uint32_t)V ? t1[k] : NONE));
      const uint32_t lo = min(a, b), hi = max(a, b);
      a = sort_clean(sort_step<16, 16>(lo));
      b = sort_clean(sort_step<16, 16>(hi));
    }
    // distinct words: a lane whose value differs from the one before it
    auto before = [&](uint32_t x) {   // lane l <- lane l - 1
      return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, true);
    };
    // (every lane takes part in both exchanges: a masked-off lane gives 0)
    const uint32_t ap = before(a), bp = before(b);
    const bool fa = a != NONE && (hl == 0 || a != ap);
    const uint32_t alast = half ? (uint32_t)__builtin_amdgcn_readlane((int)a, 63)
                                : (uint32_t)__builtin_amdgcn_readlane((int)a, 31);
    const bool fb = b != NONE && b != (hl == 0 ? alast : bp);
    auto of_half = [&](uint64_t m) { return half ? (uint32_t)(m >> 32) : (uint32_t)m; };
    const uint32_t ma = of_half(__ballot(fa)), mb = of_half(__ballot(fb));
    const uint32_t below = (1u << hl) - 1u;
    const int na = __popc(ma), n = na + __popc(mb), ng = (n + 7) >> 3;
    if (v && len[k] <= 64) {
      if (fa) out[slot_place(__popc(ma & below), ng)] = (uint16_t)(a + 32u);
      if (fb) out[slot_place(na + __popc(mb & below), ng)] = (uint16_t)(b + 32u);
      if (hl < 8 && n + hl < 8 * ng) out[slot_place(n + hl, ng)] = 0;
      if (hl == 0) tl_cnt[sent_of(k)] = n;
    }
    for (int h = 0; h < 2; ++h) {
      // a long sentence: its bitmap, then the set bits in order
      const int ln = __builtin_amdgcn_readlane(len[k], 32 * h);
      if (ln <= 64) continue;
      const int64_t o = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(off[k] >> 32), 32 * h) << 32 |
                                  (uint32_t)__builtin_amdgcn_readlane((int)off[k], 32 * h));
      uint16_t *lout = list + 8 * list_granule(o, tm.first + PER * wave + 2 * k + h);
      for (int w = lane; w < words; w += 64) bits[w] = 0u;
      wave_sync();
      for (int x = lane; x < ln; x += 64) {
        const uint32_t u = (uint32_t)tgt_tok[o + x];
        if (u < (uint32_t)V) atomicOr(&bits[u >> 5], 1u << (u & 31));
      }
      wave_sync();
      int all = 0;
      for (int w = lane; w < words; w += 64) all += __popc(bits[w]);
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) all += __shfl_xor(all, d, 64);
      const int lg = (all + 7) >> 3;
      int done = 0;
      for (int w0 = 0; w0 < words; w0 += 64) {
        uint32_t m = w0 + lane < words ? bits[w0 + lane] : 0u;
        int incl = __popc(m);
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const int y = __shfl_up(incl, d, 64);
          if (lane >= d) incl += y;
        }
        int p = done + incl - __popc(m);
        for (; m != 0u; m &= m - 1u)
          lout[slot_place(p++, lg)] = (uint16_t)(32 * (w0 + lane) + __builtin_ctz(m) + 32);
        done += __builtin_amdgcn_readlane(incl, 63);
      }
      wave_sync();
      if (lane < 8 && all + lane < 8 * lg) lout[slot_place(all + lane, lg)] = 0;
      if (lane == 0) tl_cnt[PER * wave + 2 * k + h] = all;
    }
  }
  __syncthreads();
  // the tile's sentences by word count, most first: position p's record is
  // {first granule, quads of words << 6 | sentence of the tile}
  if (threadIdx.x < (unsigned)tm.count) {
    const int n = tl_cnt[lane];
    int p = 0;
    for (int j = 0; j < tm.count; ++j) {
      const int x = tl_cnt[j];
      p += x > n || (x == n && j < lane) ? 1 : 0;
    }
    const int64_t sent = tm.first + lane;
    const int64_t off = tgt_off[sent];
    rec[tm.first + p] = make_uint2((uint32_t)list_granule(off, sent), (uint32_t)((n + 3) >> 2) << 6 | (uint32_t)lane);
    tlen[sent] = (float)(tgt_off[sent + 1] - off);
  }
}

// ---- contraction ----------------------------------------------------------------

// LDS of k_score_s: the word table (per 32 words a bitmap of the vocabulary
// and the line of its first word; entry 0 empty), the lines in planes (16
// bytes of every line each, so the 16-byte reads of a wave spread over all
// banks), the waves' totals and the rows' lengths, and per wave a tile's sums on
// their way from the lists' order of columns to the sentences'.
struct SparseLds {
  int line, plane, tot, stage, bytes;
};
constexpr int STAGE_ROW = 68;                       // floats per staged row of 64 cells
constexpr int STAGE_TILE = SROWS * STAGE_ROW * 4;   // bytes of a tile in flight: two per four waves,
constexpr int STAGE_WAVE = 4 * STAGE_ROW * 4;       // or four rows per wave (wide runs)
static __host__ __device__ inline SparseLds sparse_lds(int nch, int cap, int esize, int waves, bool wide) {
  SparseLds L;
  L.line = (8 * (nch + 1) + 15) & ~15;
  L.plane = (cap + 1) * 16;
  L.tot = L.line + L.plane * (SROWS * esize / 16);
  L.stage = L.tot + 128;
  L.bytes = L.stage + (wide ? waves * STAGE_WAVE : waves / 4 * 2 * STAGE_TILE);
  return L;
}

template <bool BF16, int WAVES, bool RAW, bool WIDE>
__global__ __launch_bounds__(64 * WAVES, 4) void k_score_s(PlanDev P, const int64_t *__restrict__ src_off,
                                                           const int64_t *__restrict__ tgt_off,
                                                           const uint2 *__restrict__ merged,
                                                           const int32_t *__restrict__ mcnt,
                                                           const uint16_t *__restrict__ list,
                                                           const uint2 *__restrict__ rec,
                                                           const float *__restrict__ tlen, nwm_scorer sc,
                                                           float *__restrict__ S, float *__restrict__ S_raw,
                                                           int g0, int cap) {
  constexpr int ES = BF16 ? 2 : 4;
  constexpr int RPP = 16 / ES;              // rows per plane
  constexpr int NT = 64 * WAVES;
  constexpr int RPW = SROWS / WAVES;        // rows per wave while building
  constexpr int EREG = 2;                   // entries per lane and row held in registers
  static_assert(SROWS == 16 && RPW * WAVES == SROWS, "rows per wave");
  extern __shared__ __align__(16) char sm[];
  const GtMeta g = P.gs_meta[g0 + (int)blockIdx.x];
  const int V = P.V, nch = P.nch;
  const SparseLds L = sparse_lds(nch, cap, ES, WAVES, WIDE);
  uint2 *tab = reinterpret_cast<uint2 *>(sm);
  int *tot = reinterpret_cast<int *>(sm + L.tot);            // [16]
  float *rlen = reinterpret_cast<float *>(sm + L.tot + 64);   // [SROWS]
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, kq = lane >> 4;

  // this wave's rows wave + WAVES k: lane k holds the row's entry count and base
  const int myrow = wave + WAVES * lane;
  const bool vrow = lane < RPW && myrow < g.rows;
  const int64_t srow = g.s_first + (vrow ? myrow : 0);
  const int rc_ld = mcnt[srow], tile_ld = BF16 ? mcnt[g.s_first + min(lane, g.rows - 1)] : 0;
  const int64_t rb = src_off[srow] * (int64_t)P.max_deg;
  const int rc = vrow ? rc_ld & ROW_COUNT : 0;
  auto row_cnt = [&](int k) { return __builtin_amdgcn_readlane(rc, k); };
  auto row_base = [&](int k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)rb, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)rb >> 32), k);
    return (int64_t)(((uint64_t)hi << 32) | lo);
  };
  // the run's lists, from its first record's tile on (offsets within a run
  // stay 32-bit: the plan bounds the batch's tokens)
  const int64_t lbase = list_granule(tgt_off[g.t_first], g.t_first);
  const __amdgpu_buffer_rsrc_t r_list =
      __builtin_amdgcn_make_buffer_rsrc((void *)(list + 8 * lbase), (short)0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_rec =
      __builtin_amdgcn_make_buffer_rsrc((void *)(rec + g.t_first), (short)0, 8 * g.cols, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_len =
      __builtin_amdgcn_make_buffer_rsrc((void *)(tlen + g.t_first), (short)0, 4 * g.cols, 0x00020000);
  const int64_t so0 = g.s_off + (int64_t)g.row0 * g.m + g.col0;
  const __amdgpu_buffer_rsrc_t r_S =
      __builtin_amdgcn_make_buffer_rsrc((void *)(S + so0), (short)0, 0x7FFFFFFF, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_R =
      __builtin_amdgcn_make_buffer_rsrc((void *)((RAW ? S_raw : S) + so0), (short)0, 0x7FFFFFFF, 0x00020000);
  auto clear = [&](int b0, int b1) {
    for (int o = b0 + 16 * tid; o < b1; o += 16 * NT) *reinterpret_cast<uint4 *>(sm + o) = make_uint4(0u, 0u, 0u, 0u);
  };
  clear(0, L.line);
  if (tid < SROWS) {
    const int64_t x = g.s_first + min(tid, g.rows - 1);
    rlen[tid] = (float)(src_off[x + 1] - src_off[x]);
  }
  __syncthreads();
  // (BF16) rows with an operand that is not finite: the sums take 0 x every
  // other row of a line, so such a row stands alone, its neighbours' sums going
  // nowhere
  const uint32_t odd = BF16 ? (uint32_t)__ballot((tile_ld & ROW_ODD) != 0) & ((1u << g.rows) - 1u) : 0u;
  // all rows at once unless their vocabulary exceeds the table (then fewer at
  // a time; one row always fits) or some stand alone
  int rs = 0, re = g.rows;
  while (rs < g.rows) {
    if (odd != 0u) {
      const uint32_t after = odd >> rs;
      re = min(re, (after & 1u) ? rs + 1 : after ? rs + __builtin_ctz(after) : re);
    }
    // the first 64 EREG entries of every row of this wave, loaded together
    uint2 e[RPW][EREG];
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
          (void *)(merged + row_base(k)), (short)0, min(row_cnt(k), 64 * EREG) * 8, 0x00020000);
#pragma unroll
      for (int q = 0; q < EREG; ++q) {
        const s_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (uint32_t)(64 * q + lane) * 8u, 0, 0);
        e[k][q] = make_uint2(64 * q + lane < row_cnt(k) ? v.x : 0xFFFFFFFFu, v.y);
      }
    }
    // every entry (row, word, value) of this wave's rows in [rs, re)
    auto entries = [&](auto &&f) {
#pragma unroll
      for (int k = 0; k < RPW; ++k) {
        const int r = wave + WAVES * k;
        if (r < rs || r >= re) continue;
#pragma unroll
        for (int q = 0; q < EREG; ++q)
          if (e[k][q].x < (uint32_t)V) f(r, e[k][q].x, e[k][q].y);
        const int c = row_cnt(k);
        for (int x = 64 * EREG + lane; x < c; x += 64) {
          const uint2 v = merged[row_base(k) + x];
          if (v.x < (uint32_t)V) f(r, v.x, v.y);
        }
      }
    };
    entries([&](int, uint32_t u, uint32_t) { atomicOr(&tab[1 + (u >> 5)].x, 1u << (u & 31)); });
    __syncthreads();
    // lines in word order: each thread counts a run of the bitmap, wave
    // scans, then the waves' totals
    int total = 0;
    {
      const int run = (nch + NT - 1) / NT;
      const int w0 = min(tid * run, nch), w1 = min(w0 + run, nch);
      int sum = 0;
      for (int w = w0; w < w1; ++w) sum += __popc(tab[1 + w].x);
      int incl = sum;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
      }
      if (lane == 63) tot[wave] = incl;
      __syncthreads();
      int p = 1 + incl - sum;
#pragma unroll
      for (int k = 0; k < WAVES; ++k) {
        const int t = tot[k];
        p += k < wave ? t : 0;
        total += t;
      }
      for (int w = w0; w < w1; ++w) {
        tab[1 + w].y = (uint32_t)p;
        p += __popc(tab[1 + w].x);
      }
      total = s_uniform(total);
    }
    if (total > cap && re - rs > 1) {
      __syncthreads();
      clear(0, L.line);
      re = rs + ((re - rs) >> 1);
      __syncthreads();
      continue;
    }
#pragma unroll
    for (int q = 0; q < SROWS / RPP; ++q) clear(L.line + q * L.plane, L.line + q * L.plane + 16 * (min(total, cap) + 1));
    __syncthreads();
    entries([&](int r, uint32_t u, uint32_t v) {
      const uint2 t = tab[1 + (u >> 5)];
      const int line = (int)t.y + __popc(t.x & ((1u << (u & 31)) - 1u));
      if (line > cap) return;   // (only where a sentence breaks the plan's bound)
      char *at = sm + L.line + (r / RPP) * L.plane + 16 * line + ES * (r % RPP);
      if constexpr (BF16) *reinterpret_cast<uint16_t *>(at) = __builtin_bit_cast(uint16_t, (__bf16)__uint_as_float(v));
      else *reinterpret_cast<uint32_t *>(at) = v;
    });
    __syncthreads();

    const uint32_t plane = (uint32_t)L.line + (uint32_t)(BF16 ? (kq & 1) : kq) * (uint32_t)L.plane;   // the lane's
    // A operand: row l16 of the sum takes element i of k group kq where
    // (kq & 1) * 8 + i is that row
    s_bf16x8 add2;
#pragma unroll
    for (int i = 0; i < 8; ++i) add2[i] = (__bf16)((kq & 1) * 8 + i == l16 ? 1.0f : 0.0f);

    // group gr: positions 16 gr .. 16 gr + 15 of the run in its tiles' order
    // (a position past the run: no words)
    auto load_rec = [&](int gr) {
      const int pos = 16 * gr + l16;
      const s_u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r_rec, 8u * (uint32_t)pos, 0, 0);
      return make_uint2(v.x, v.y);
    };
    // its lane's dwords of granules 4 blk .. 4 blk + 3
    auto load_list = [&](const uint2 &r, int blk) {
      const int ng = (int)(((r.y >> 6) + 1u) >> 1);   // granules of the lane's list
      const uint32_t o = (r.x - (uint32_t)lbase + 4u * (uint32_t)blk) * 16u + 4u * (uint32_t)(kq * min(4, ng - 4 * blk));
      return __builtin_amdgcn_raw_buffer_load_b128(r_list, 4 * blk < ng ? o : LIST_NONE, 0, 0);
    };
    // a slot's line, 0 for a word no row holds
    auto line_of = [&](uint32_t slot, const uint2 &t) {
      const uint32_t l = t.y + (uint32_t)__popc(t.x & ((1u << (slot & 31u)) - 1u));
      return l & (uint32_t)__builtin_amdgcn_sbfe((int)t.x, slot & 31u, 1u);
    };
    // The sums of a group, rows 4 kq .. 4 kq + 3 of the lane's sentence, in
    // steps of four line reads: eight words (BF16) or four (FP32).  Step i's
    // lines are read while step i - 1's are summed and step i + 1's table
    // entries are on their way, so a wave waits for LDS once, at the start.
    constexpr int SQ = BF16 ? 2 : 1;   // quads of words per step
    struct Tabs {
      uint2 t[SQ];
    };
    struct Lines {
      s_u32x4 v[4];
    };
    auto look = [&](const uint32_t (&x)[SQ]) {
      Tabs k;
#pragma unroll
      for (int h = 0; h < SQ; ++h) k.t[h] = *reinterpret_cast<const uint2 *>(sm + ((x[h] >> 2) & 0x3FF8u));
      return k;
    };
    // the lane's lines: lanes kq = 0, 2 looked words 0 and 1 of a quad up, kq
    // = 1, 3 words 2 and 3; swapping rows of 16 lanes (then halves) hands the
    // lines round
    auto read = [&](const uint32_t (&x)[SQ], const Tabs &t) {
      Lines n;
#pragma unroll
      for (int h = 0; h < SQ; ++h) {
        const uint32_t l = line_of(x[h], t.t[h]);
        const auto a = __builtin_amdgcn_permlane16_swap(l, l, false, false);
        if constexpr (BF16) {
#pragma unroll
          for (int i = 0; i < 2; ++i)
            n.v[2 * h + i] = *reinterpret_cast<const s_u32x4 *>(sm + ((a[i] << 4) + plane));
        } else {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const auto b = __builtin_amdgcn_permlane32_swap(a[i], a[i], false, false);
            n.v[2 * i] = *reinterpret_cast<const s_u32x4 *>(sm + ((b[0] << 4) + plane));
            n.v[2 * i + 1] = *reinterpret_cast<const s_u32x4 *>(sm + ((b[1] << 4) + plane));
          }
        }
      }
      return n;
    };
    auto add = [&](const Lines &n, s_f32x4 &acc) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (BF16) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(add2, __builtin_bit_cast(s_bf16x8, n.v[i]), acc, 0, 0, 0);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[r] += __uint_as_float(n.v[i][r]);
        }
      }
    };
    // x0: the first block of the lane's list (32 words)
    auto sums = [&](const uint2 &r, const s_u32x4 &x0) {
      s_f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
      const int ns = (s_uniform((int)(r.y >> 6)) + SQ - 1) / SQ;   // steps of the longest list (the first)
      const int mine = (int)(((r.y >> 6) + 1u) >> 1);              // granules of the lane's own
      constexpr int PB = 8 / SQ;                                   // steps per block of four granules
      s_u32x4 cur = x0, nxt = {0u, 0u, 0u, 0u};
      if (ns > PB) nxt = load_list(r, 1);
      auto mask = [&](s_u32x4 &x, int blk) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (4 * blk + j >= mine) x[j] = 0u;   // past the lane's list
      };
      // the slots of step i of a block (compile-time i)
      auto slots = [&](const s_u32x4 &x, int i, uint32_t (&o)[SQ]) {
        if constexpr (BF16) {
          o[0] = x[i];
          o[1] = x[i] >> 16;
        } else {
          o[0] = (i & 1) ? x[i >> 1] >> 16 : x[i >> 1];
        }
      };
      mask(cur, 0);
      uint32_t sa[SQ], sb[SQ], sc_[SQ];
      slots(cur, 0, sa);
      Tabs ta = look(sa);
      slots(cur, 1, sb);
      Tabs tb = look(sb);
      Lines va = read(sa, ta);
      for (int blk = 0; PB * blk < ns; ++blk) {
        mask(nxt, blk + 1);
#pragma unroll
        for (int i = 0; i < PB; ++i) {
          if (i > 0 && PB * blk + i >= ns) break;
          // step i: its lines are in va, step i + 1's slots and table in sb, tb
          slots(i + 2 < PB ? cur : nxt, (i + 2) % PB, sc_);
          const Tabs tc = look(sc_);
          const Lines vb = read(sb, tb);
          __builtin_amdgcn_sched_barrier(0);
          add(va, acc);
          va = vb;
          tb = tc;
#pragma unroll
          for (int h = 0; h < SQ; ++h) sb[h] = sc_[h];
        }
        cur = nxt;
        nxt = s_u32x4{0u, 0u, 0u, 0u};
        if (PB * (blk + 2) < ns) nxt = load_list(r, blk + 2);
      }
      return acc;
    };
    // A tile's sums pass through LDS (`stage`) from the lists' order of columns
    // into the sentences' own, then row `row` of four is scored and stored, 16
    // bytes a lane.
    auto score4 = [&](const float *stage, int t, int row, int srow_, const s_u32x4 &tl) {
      const s_u32x4 d = *reinterpret_cast<const s_u32x4 *>(stage + STAGE_ROW * srow_ + 4 * l16);
      const float ls = rlen[row], rls = __builtin_amdgcn_rcpf(ls);
      const int left = g.cols - 64 * t - 4 * l16;
      s_u32x4 sv, sr;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float raw;
        const float lt = __uint_as_float(tl[c]);
        sv[c] = __float_as_uint(logistic_cell<true>(__uint_as_float(d[c]), ls, rls, lt, __builtin_amdgcn_rcpf(lt), sc,
                                                    raw));
        sr[c] = __float_as_uint(raw);
      }
      const uint32_t o = row >= rs && row < re && left > 0
                             ? 4u * ((uint32_t)row * (uint32_t)g.m + (uint32_t)(64 * t + 4 * l16))
                             : LIST_NONE;
      if (64 * t + 64 <= g.cols) {
        __builtin_amdgcn_raw_buffer_store_b128(sv, r_S, o, 0, 0);
        if constexpr (RAW) __builtin_amdgcn_raw_buffer_store_b128(sr, r_R, o, 0, 0);
      } else {   // the pair's last columns
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t oc = c < left ? o + 4u * c : LIST_NONE;
          __builtin_amdgcn_raw_buffer_store_b32(sv[c], r_S, oc, 0, 0);
          if constexpr (RAW) __builtin_amdgcn_raw_buffer_store_b32(sr[c], r_R, oc, 0, 0);
        }
      }
    };
    // the lengths of the lane's four sentences of tile t
    auto load_len = [&](int t) {
      return __builtin_amdgcn_raw_buffer_load_b128(r_len, 256u * (uint32_t)t + 16u * (uint32_t)l16, 0, 0);
    };
    const int nt = (g.cols + 63) >> 6, sub = wave & 3;
    if constexpr (WIDE) {
      // a wave per tile: its four groups one after another, then four rows at
      // a time through LDS; no barriers
      float *stage = reinterpret_cast<float *>(sm + L.stage + wave * STAGE_WAVE);
      uint2 r = load_rec(4 * wave);
      s_u32x4 x = load_list(r, 0);
      for (int t = wave; t < nt; t += WAVES) {
        const s_u32x4 tl = load_len(t);
        s_f32x4 acc[4];
        int at[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint2 rn = load_rec(i < 3 ? 4 * t + i + 1 : 4 * (t + WAVES));
          asm volatile("" ::: "memory");   // (keeps the load here: it would sink to its use)
          acc[i] = sums(r, x);
          at[i] = 64 * t + 16 * i + l16 < g.cols ? (int)(r.y & 63u) : 64;   // (64..: never read)
          r = rn;
          x = load_list(r, 0);   // before the tile's stores: a load waits for older stores
          asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          wave_sync();
#pragma unroll
          for (int i = 0; i < 4; ++i) stage[STAGE_ROW * kq + at[i]] = acc[i][q];
          wave_sync();
          score4(stage, t, 4 * kq + q, kq, tl);
        }
      }
    } else {
      // four waves per tile, a group of 16 sentences each
      uint2 r = load_rec(4 * (wave >> 2) + sub);
      s_u32x4 x = load_list(r, 0);
      int buf = 0;
      for (int t0 = 0; t0 < nt; t0 += WAVES / 4) {
        const int t = t0 + (wave >> 2);
        const uint2 rn = load_rec(4 * (t + WAVES / 4) + sub);
        const s_u32x4 tl = load_len(t);
        asm volatile("" ::: "memory");   // (keeps the loads here: they would sink to their uses)
        const s_f32x4 acc = sums(r, x);
        float *stage = reinterpret_cast<float *>(sm + L.stage + (2 * (wave >> 2) + buf) * STAGE_TILE);
        const int at = (int)(r.y & 63u);
        if (64 * t + 16 * sub + l16 < g.cols)
#pragma unroll
          for (int q = 0; q < 4; ++q) stage[STAGE_ROW * (4 * kq + q) + at] = acc[q];
        r = rn;
        x = load_list(r, 0);   // before the tile's stores: a load waits for older stores
        asm volatile("" ::: "memory");
        __syncthreads();
        score4(stage, t, 4 * sub + kq, 4 * sub + kq, tl);
        buf ^= 1;
      }
    }
    rs = re;
    re = g.rows;
    if (rs < g.rows) {
      __syncthreads();
      clear(0, L.line);
      __syncthreads();
    }
  }
}

// Lines of the LDS table: enough for 16 ordinary sentences' vocabulary (530
// to 820 words on average over the benchmark corpora, at most 972 seen) and
// for any single sentence.
static int sparse_cap(int max_entries) { return std::max(928, max_entries); }

template <typename F>
static void sparse_kernel(bool bf16, bool raw, bool wide, F &&go) {
  auto w = [&](auto B, auto R, auto D) {
    constexpr bool b = decltype(B)::value;
    go(k_score_s<b, b ? 4 : 8, decltype(R)::value, decltype(D)::value>);
  };
  auto d = [&](auto B, auto R) {
    if (wide) w(B, R, std::true_type{});
    else w(B, R, std::false_type{});
  };
  auto r = [&](auto B) {
    if (raw) d(B, std::true_type{});
    else d(B, std::false_type{});
  };
  if (bf16) r(std::true_type{});
  else r(std::false_type{});
}

hipError_t launch_score_s(const PlanDev &P, bool bf16, int max_entries, int tiles_per_run, const int64_t *src_off,
                          const int64_t *tgt_off, const uint2 *merged, const int32_t *mcnt, const uint16_t *list,
                          const uint2 *rec, const float *tlen, nwm_scorer sc, float *S, float *S_raw, int g0,
                          int G, hipStream_t st) {
  if (G <= 0) return hipSuccess;
  const int cap = sparse_cap(max_entries), es = bf16 ? 2 : 4;
  // BF16: four waves, four workgroups a compute unit.  FP32's table leaves
  // room for two, of eight waves; the narrow kind's staging for one where the
  // vocabulary is large.  A workgroup per tile keeps all its waves busy on
  // short runs, a wave per tile needs no barriers: measured (score alone, 20 M
  // cells of square pairs, V = 16384, narrow / wide): BF16 122 / 124 us at 128
  // sentences a side, 98 / 79 at 256, 80 / 65 at 1000; FP32 153 / 229 at 128,
  // 117 / 127 at 256, 107 / 93 at 512.
  const int waves = bf16 ? 4 : 8;
  const bool wide = tiles_per_run >= (bf16 ? 4 : 8) ||
                    (!bf16 && sparse_lds(P.nch, cap, es, waves, false).bytes > 80 * 1024);
  const int lds = sparse_lds(P.nch, cap, es, waves, wide).bytes;
  sparse_kernel(bf16, S_raw != nullptr, wide, [&](auto k) {
    hipLaunchKernelGGL(k, dim3(G), dim3(64 * waves), lds, st, P, src_off, tgt_off, merged, mcnt, list, rec, tlen, sc, S,
                       S_raw, g0, cap);
  });
  return hipGetLastError();
}

// Column tiles [c0, c0 + n).
hipError_t launch_tgt_lists(const PlanDev &P, const int64_t *tgt_off, const int32_t *tgt_tok, uint16_t *list,
                            uint2 *rec, float *tlen, int c0, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const size_t lds = 4 * (size_t)TL_WAVES * (size_t)P.nch;
  hipLaunchKernelGGL(k_tgt_lists, dim3(n), dim3(64 * TL_WAVES), lds, st, P.ct_meta, c0, tgt_off, tgt_tok, P.V, list,
                     rec, tlen);
  return hipGetLastError();
}

// More than the default dynamic LDS, up to what a workgroup can have.
hipError_t sparse_set_attrs() {
  hipError_t e = hipSuccess;
  for (int v = 0; v < 8; ++v)
    sparse_kernel(v & 1, v & 2, v & 4, [&](auto k) {
      if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
  return e;
}

}  // namespace nwm
