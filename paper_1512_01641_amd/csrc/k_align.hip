// Needleman-Wunsch global alignment of the sentence sequences of every
// document pair (Sec. 5.1, Figs. 1-2, eq. (1)) and the threshold filter
// (Sec. 4).
//
// k_nw_fill   persistent work-queue kernel, four strip waves and two row waves
//             per workgroup.  A strip is 64 rows of one pair's DP lattice; a
//             task is four strips, one per strip wave: consecutive strips of
//             one pair (fewer at its end) or strips of several pairs, in queue
//             order (longest chains first).  Lane r owns row r of the strip
//             and at step t computes column j = t - r + 1, so each step is one
//             anti-diagonal of the strip, computed by all lanes at once
//             (Sec. 5.1, Fig. 2).  Per cell, in FP32 without contraction:
//                up = H[i-1][j] + g, left = H[i][j-1] + g, diag = H[i-1][j-1] + S
//                first maximum of (up, left, diag) with '>' (UP > LEFT > DIAG)
//             The value from the row above moves one lane per step by a DPP
//             wave shift.  The row above the strip comes from an LDS row ring,
//             16 columns at a time (lane 0 uses them; the other lanes read
//             zeros); the strip's own last row leaves lane 63 into the next row
//             ring every 16 steps, with a count of columns put and taken.  So a
//             strip trails the one above it by 80 steps.  What does not come
//             from or go to a strip of the same task is the row waves' work:
//             one fills row rings with a pair's first row (j g) or with a row
//             another workgroup publishes, the other publishes the task's last
//             row, as tagged 64-bit agent-coherent stores (no counters, no
//             cache flushes).  A wave that gives up waiting (its poll limit)
//             sets the error flag, marks its own last row failed (tag TAG_FAIL
//             in memory, count -1 in LDS, so the strips below give up at once
//             instead of waiting out their own limits) and, in a pair's last
//             strip, writes NaN as the score; the walk then leaves the pair
//             empty.  S is staged through an LDS ring of two 64-step groups
//             per strip (16 KiB each: 64 rows x 256 bytes), filled a group
//             ahead by 16-byte LDS-direct buffer loads (no register holds S);
//             each lane reads the four steps of one 16-byte piece of its own
//             row with one ds_read_b128, placed so that the lanes of a
//             quarter-wave hit different banks.  Each lane collects its
//             directions in two bit planes, and every 64 steps the wave writes
//             one coalesced 1 KiB block.  H never reaches HBM.
//             What bounds it is a strip wave's issue: one wave per SIMD, about
//             190 instructions per 16 steps (144 of them the cells') at about
//             5 clocks.  Measured: one strip of 64 x 20000 511 us (774 with
//             the row above shifted through a register window, directions
//             packed by selects and S waits spread over the chunk), 256 x
//             20000 611 us (981), 2000 x 2000 169 us (260), 64 pairs of 5000 x
//             5000 1.63 ms (1.66: S from HBM, 3.9 TB/s).
// k_nw_reset  clears the rows that pass through memory and the queue; scores
//             of empty pairs.
// k_nw_walk   traceback from (n, m) over the stored directions: k_nw_walk_map
//             and k_nw_walk_chain find where the path enters every strip of the
//             longer pairs, k_nw_walk follows it through all strips at once
//             (the shorter pairs', strip by strip) and writes the aligned pairs
//             right-aligned (ascending) into the path area.
// k_keep      keeps the aligned pairs with S >= threshold, ascending.
#include "nwm_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace nwm {

constexpr int CHUNK = 16;             // steps per chunk
constexpr int GROUP = 64;             // steps per S staging group (four chunks)
constexpr int GROUP_BYTES = 64 * GROUP * 4;   // LDS bytes per group (64 rows x 256 bytes)
constexpr int RING_GROUPS = 2;        // groups in a strip's S ring: one in flight while one is read
constexpr int SPIN_LIMIT = 1 << 22;   // default polls before a wave gives up (error flag): of a row in memory
// LDS_POLLS polls of an LDS count count as one poll of the limit: one takes 0.11
// us, a poll of a row in memory 0.17 (the fill that stages S in registers) to
// 0.27 (a row wave).  So a strip waits for a row in LDS no shorter than the row
// waves wait for one in memory (4000 polls: 1.7 ms, 0.4 counted singly).
constexpr uint32_t LDS_POLLS = 4;
constexpr uint32_t TAG_FAIL = 2u;     // tag of a boundary value whose producer gave up

static __device__ __forceinline__ float dpp_shr1(float old, float src) {
  // lane l <- src of lane l-1; lane 0 keeps `old`
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src), 0x138, 0xF, 0xF, false));
}
static __device__ __forceinline__ float dpp_shl1(float old, float src) {
  // lane l <- src of lane l+1; lane 63 keeps `old`
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src), 0x130, 0xF, 0xF, false));
}

static __device__ __forceinline__ float dpp_next(float src) {
  // lane l <- src of lane l+1 (lane 63: 0)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(src), 0x130, 0xF, 0xF, true));
}

static __device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// A 64-bit value every lane holds the same value of, moved to scalar registers.
static __device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// A pointer every lane holds the same value of, moved to scalar registers.
template <typename T>
static __device__ __forceinline__ T *uniform_ptr(T *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return reinterpret_cast<T *>(((uint64_t)hi << 32) | lo);
}

// The parallelogram of S used by steps [GROUP*q, GROUP*q + GROUP): row r,
// columns GROUP*q - r + [0, GROUP), 256 bytes per row.  It goes straight
// from memory into one ring slot of 16 KiB by 16 LDS-direct 16-byte buffer
// loads; load k brings rows 4k .. 4k + 3 into the slot's k-th KiB.  Within
// that KiB, lane l of the load writes bytes 16 l .. 16 l + 15, so the lane
// that loads 16-byte piece c (steps 4c .. 4c + 3) of row 4k + rho is the
// one that puts it where the reader wants it:
//    lane = 16 rho + ((c + 4 (k & 3) + rho) & 15).
// Every lane of the reader (lane = row) then reads piece c of its own row
// with one ds_read_b128, and the 16 lanes of each quarter-wave (rows
// 16p + j) fall on 16 different 16-byte bank groups ((c + j) & 15).  The 16
// lanes of a load that share rho read one row's 256 contiguous bytes (rows
// start at any multiple of 4 bytes: shorter pieces of a row, 64 bytes per 16
// steps, touch twice the cache lines; a batch of 64 pairs of 5000 x 5000
// took 1.88 ms with them).  No register holds S in flight.
//
// Lane l of load k reads strip bytes 4 (r (m - 1) + GROUP q) + 16 c for its
// row r = 4k + rho and piece c: base_{k & 3} + (k >> 2) 64 (m - 1) + 256 q,
// with the group offset in the VGPR offset so that the range check covers it.
// A cell outside the strip's m columns (the first steps of a row, the steps
// after its last column) reads another cell of the strip, or 0 past the
// strip's end through the buffer range check: a value that no cell of the
// lattice sees.  Rows at or beyond `rows` (the last strip of a pair) lie past
// the end.
struct StripSrc {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t base[4];        // bytes, this lane's (row, piece) in loads 0..3
  uint32_t step;           // bytes from load k to load k + 4: 64 (m - 1)
};

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) const int lds_int;

typedef unsigned int u32x2v __attribute__((ext_vector_type(2)));
constexpr int CPOL_SC1 = 16;          // cache-policy bit of an agent-coherent access
constexpr int PUB_NONE = 0x40000000;  // buffer offset past any boundary row: the store is dropped

// The strip's last row: one tagged 64-bit agent-coherent store per lane into
// the boundary row `rs` (slot j at byte 8 j).  A lane with nothing to
// publish stores at PUB_NONE, past the buffer's range, and the range check
// drops it without a memory access.
static __device__ __forceinline__ void publish(__amdgpu_buffer_rsrc_t rs, bool pub, int j, uint64_t v) {
  const u32x2v d = {(uint32_t)v, (uint32_t)(v >> 32)};
  __builtin_amdgcn_raw_buffer_store_b64(d, rs, pub ? 8 * j : PUB_NONE, 0, CPOL_SC1);
}

// The lane's byte base for load j < 4 (see StripSrc): row rho of the load
// and piece c, inverting lane = 16 rho + ((c + 4 j + rho) & 15).
static __device__ __forceinline__ uint32_t s_lane_base(int lane, int j, int m) {
  const int rho = lane >> 4;
  const int c = ((lane & 15) - 4 * j - rho) & 15;
  return (uint32_t)(4 * j + rho) * (uint32_t)(m - 1) * 4u + 16u * (uint32_t)c;
}

#define NWM_S_LOAD(A)                               \
  "buffer_load_dwordx4 " A ", %8, 0 offen lds\n\t"  \
  "s_add_u32 m0, m0, 1024\n\t"                      \
  "v_add_u32 " A ", %9, " A "\n\t"
#define NWM_S_LOAD4 NWM_S_LOAD("%0") NWM_S_LOAD("%1") NWM_S_LOAD("%2") NWM_S_LOAD("%3")

// The 16 loads of the group at byte offset goff = 256 q into the ring slot at
// `slot`, in one asm statement so that the compiler neither reorders them with
// other memory accesses nor adds waits for them: every read of the ring waits
// for them with an explicit vmcnt (below).  M0 (the LDS address of a load)
// steps by 1 KiB per load; a VALU instruction separates each M0 write from the
// load that uses it.
static __device__ __forceinline__ void load_group(uint32_t slot, const StripSrc &src, uint32_t goff) {
  uint32_t a0, a1, a2, a3;
  asm volatile(
      "s_mov_b32 m0, %4\n\t"
      "v_add_u32 %0, %7, %5\n\t"
      "v_add_u32 %1, %7, %6\n\t"
      "v_add_u32 %2, %7, %10\n\t"
      "v_add_u32 %3, %7, %11\n\t"
      NWM_S_LOAD4 NWM_S_LOAD4 NWM_S_LOAD4 NWM_S_LOAD4
      : "=&v"(a0), "=&v"(a1), "=&v"(a2), "=&v"(a3)
      : "s"(slot), "v"(src.base[0]), "v"(src.base[1]), "s"(goff), "s"(src.rs), "s"(src.step), "v"(src.base[2]),
        "v"(src.base[3])
      : "memory", "scc", "m0");
}
#undef NWM_S_LOAD4
#undef NWM_S_LOAD

struct StripState {
  float H, diag, pw, col;
};

// Directions, one bit per step and plane, first step in the high bits: into U
// goes 1 where the cell's maximum is the value from above, into L where it is
// the value from the left (UP wins where both are, DIAG is neither).
template <bool MAX3>
static __device__ __forceinline__ float cell(float up, float left, float dg, uint32_t &U, uint32_t &L) {
  if constexpr (MAX3) {
    const float best = __builtin_fmaxf(__builtin_fmaxf(up, left), dg);
    U = (U << 1) | (up == best ? 1u : 0u);
    L = (L << 1) | (left == best ? 1u : 0u);
    return best;
  } else {
    const bool c1 = left > up;
    const float b1 = c1 ? left : up;
    const bool c2 = dg > b1;
    U = (U << 1) | (!c1 && !c2 ? 1u : 0u);
    L = (L << 1) | (c1 && !c2 ? 1u : 0u);
    return c2 ? dg : b1;
  }
}

// Eight steps with a gap of -0 (see run8_chain).  In the first 64 of a strip (EARLY: their first, a multiple of
// 8; else -1) H is updated only in the lanes 0 .. t whose first column has come
// at step t, so a lane keeps H[i][0] until then.  A lane that is past its last
// column goes on with values no lattice cell sees: a lane's cell of column j
// uses the lane above at columns j - 1 and j only, and what leaves the strip
// (its last row, the score) is taken at the step of its column.  row: the row
// above the strip at the columns of lane 0, 0 in the other lanes; hs receives H
// after every step.
template <int EARLY>
static __device__ __forceinline__ void run8(StripState &st, const float4 *sv, const float4 *row, float g, uint32_t &U,
                                            uint32_t &L, float *hs) {
  float H = st.H, diag = st.diag;
  uint64_t begun = EARLY >= 0 ? (2ull << (EARLY & 63)) - 1ull : 0ull;   // lanes at column 1 or past it
  asm volatile("" : "+s"(begun));   // (constants here would be kept in scalar registers over the whole kernel)
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const float4 v4 = sv[u >> 2], b4 = row[u >> 2];
    const float s = (u & 3) == 0 ? v4.x : (u & 3) == 1 ? v4.y : (u & 3) == 2 ? v4.z : v4.w;
    const float above = (u & 3) == 0 ? b4.x : (u & 3) == 1 ? b4.y : (u & 3) == 2 ? b4.z : b4.w;
    const float x = dpp_shr1(above, H);   // H[i-1][j]: lane r-1, or the row above the strip for lane 0
    const float best = cell<false>(x + g, H + g, diag + s, U, L);
    if constexpr (EARLY >= 0) {
      H = __builtin_amdgcn_inverse_ballot_w64(begun) ? best : H;
      begun = (begun << 1) | 1ull;
    } else {
      H = best;
    }
    diag = x;
    hs[u] = H;
  }
  st.H = H;
  st.diag = diag;
}

// The same eight steps (gap not -0) as one block, in the order a lone wave
// needs.  A chain of strips runs one wave per SIMD, where every vector
// instruction costs about 4.7 clocks whatever it is: nine per step (an add that
// shifts lanes: H of the lane above plus the row above the strip, which is 0 in
// every lane but 0, where there is no lane above; three adds, one max3, and
// compare + add-with-carry per direction plane; two-bit codes packed by selects
// took 16).  The chain of a step (shift, add, max3) has other instructions
// behind each of its own, which cover their latency and the two wait states
// that a lane shift needs after the write of its source and an add-with-carry
// after the write of its carry; the directions of a step are taken in the steps
// after it.  Left to itself the compiler moves the directions of all steps
// behind the chain, 50 clocks a step against 42.
//
// The new H is max(up, left, diag) in one instruction: the first maximum with
// '>' bit for bit whenever no operand is NaN or -0.  A finite S and a gap that
// is not -0 never produce either (H starts at +0 or i*gap != 0, and a sum is
// -0 only when both terms are); a gap of -0 takes the compare chain.
#define NWM_CMP(a, H) "v_cmp_eq_f32_e32 vcc, %[" a "], " H "\n\t"
#define NWM_ADDC(P) "v_addc_co_u32_e32 %[" P "], vcc, %[" P "], %[" P "], vcc\n\t"
// step k from H, x of the step before (Hp, Xp), temporaries u and l number u;
// A: the step before that one's L; B, C, D: the step before's
#define NWM_STEP(k, Hp, Xp, u, A, B, C, D)                                     \
  "v_add_f32 %[h" k "], " Xp ", %[s" k "]\n\t" A B                             \
  "v_add_f32_dpp %[b" k "], " Hp ", %[a" k "] wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"  \
  "v_add_f32 %[l" u "], %[g], " Hp "\n\t"                                      \
  "v_add_f32 %[u" u "], %[g], %[b" k "]\n\t" C D                               \
  "v_max3_f32 %[h" k "], %[u" u "], %[l" u "], %[h" k "]\n\t"
#define NWM_FIRST(k, Hp, Xp, u) NWM_STEP(k, Hp, Xp, u, "s_nop 0\n\t", "", "", "")
#define NWM_NEXT(k, p, u, v, A)                                                                              \
  NWM_STEP(k, "%[h" p "]", "%[b" p "]", u, A, NWM_CMP("u" v, "%[h" p "]"), NWM_ADDC("U"),                    \
           NWM_CMP("l" v, "%[h" p "]"))
// (two wait states between a compare and the add-with-carry that takes it)
#define NWM_LAST                                                                                    \
  "v_cmp_eq_f32_e64 %[m], %[l1], %[h7]\n\t" NWM_ADDC("L") NWM_CMP("u1", "%[h7]") "s_nop 1\n\t" \
  NWM_ADDC("U") "v_addc_co_u32_e64 %[L], %[m], %[L], %[L], %[m]"
// lanes past lane t keep H
#define NWM_KEEP(k, Hp, T) "s_bfm_b64 %[m], " T "+%[t], 0\n\tv_cndmask_b32_e64 %[h" k "], " Hp ", %[h" k "], %[m]\n\t"
template <int EARLY>
static __device__ __forceinline__ void run8_chain(StripState &st, const float4 *sv, const float4 *row, float g,
                                                  uint32_t &U, uint32_t &L, float *hs) {
  float x[8], u0, u1, l0, l1;
  uint64_t m;
#define NWM_OPERANDS                                                                                                  \
  : [h0] "=&v"(hs[0]), [h1] "=&v"(hs[1]), [h2] "=&v"(hs[2]), [h3] "=&v"(hs[3]), [h4] "=&v"(hs[4]), [h5] "=&v"(hs[5]), \
    [h6] "=&v"(hs[6]), [h7] "=&v"(hs[7]), [b0] "=&v"(x[0]), [b1] "=&v"(x[1]), [b2] "=&v"(x[2]), [b3] "=&v"(x[3]),          \
    [b4] "=&v"(x[4]), [b5] "=&v"(x[5]), [b6] "=&v"(x[6]), [b7] "=&v"(x[7]), [U] "+v"(U), [L] "+v"(L), [u0] "=&v"(u0),      \
    [u1] "=&v"(u1), [l0] "=&v"(l0), [l1] "=&v"(l1), [m] "=&s"(m)                                                      \
  : [s0] "v"(sv[0].x), [s1] "v"(sv[0].y), [s2] "v"(sv[0].z), [s3] "v"(sv[0].w), [s4] "v"(sv[1].x), [s5] "v"(sv[1].y), \
    [s6] "v"(sv[1].z), [s7] "v"(sv[1].w), [a0] "v"(row[0].x), [a1] "v"(row[0].y), [a2] "v"(row[0].z),                   \
    [a3] "v"(row[0].w), [a4] "v"(row[1].x), [a5] "v"(row[1].y), [a6] "v"(row[1].z), [a7] "v"(row[1].w), [H] "v"(st.H), [X] "v"(st.diag), [g] "s"(g), [t] "n"(EARLY)                 \
  : "vcc"
  if constexpr (EARLY < 0) {
    asm volatile(NWM_FIRST("0", "%[H]", "%[X]", "0")
                 NWM_NEXT("1", "0", "1", "0", "") NWM_NEXT("2", "1", "0", "1", NWM_ADDC("L"))
                 NWM_NEXT("3", "2", "1", "0", NWM_ADDC("L")) NWM_NEXT("4", "3", "0", "1", NWM_ADDC("L"))
                 NWM_NEXT("5", "4", "1", "0", NWM_ADDC("L")) NWM_NEXT("6", "5", "0", "1", NWM_ADDC("L"))
                 NWM_NEXT("7", "6", "1", "0", NWM_ADDC("L")) NWM_LAST NWM_OPERANDS);
  } else {
    asm volatile(NWM_FIRST("0", "%[H]", "%[X]", "0") NWM_KEEP("0", "%[H]", "1")
                 NWM_NEXT("1", "0", "1", "0", "") NWM_KEEP("1", "%[h0]", "2")
                 NWM_NEXT("2", "1", "0", "1", NWM_ADDC("L")) NWM_KEEP("2", "%[h1]", "3")
                 NWM_NEXT("3", "2", "1", "0", NWM_ADDC("L")) NWM_KEEP("3", "%[h2]", "4")
                 NWM_NEXT("4", "3", "0", "1", NWM_ADDC("L")) NWM_KEEP("4", "%[h3]", "5")
                 NWM_NEXT("5", "4", "1", "0", NWM_ADDC("L")) NWM_KEEP("5", "%[h4]", "6")
                 NWM_NEXT("6", "5", "0", "1", NWM_ADDC("L")) NWM_KEEP("6", "%[h5]", "7")
                 NWM_NEXT("7", "6", "1", "0", NWM_ADDC("L"))
                 ".if %[t]+8 < 64\n\t" NWM_KEEP("7", "%[h6]", "8") ".endif\n\t" NWM_LAST NWM_OPERANDS);
  }
#undef NWM_OPERANDS
  st.H = hs[7];
  st.diag = x[7];
}
#undef NWM_KEEP
#undef NWM_LAST
#undef NWM_NEXT
#undef NWM_FIRST
#undef NWM_STEP
#undef NWM_ADDC
#undef NWM_CMP

typedef float f4v __attribute__((ext_vector_type(4)));

// Lane 63's 16 columns (the carry, then H after the chunk's first 15 steps) to
// LDS bytes `to` + OFFSET, then the count of columns `col` to `count`.
// Written in asm: the one lane is picked and all are back in two instructions
// (every lane is active here).
template <int OFFSET>
static __device__ __forceinline__ void put_row(uint32_t to, float carry, const float (&hs)[CHUNK], uint32_t count,
                                               int col) {
  const f4v h0 = {carry, hs[0], hs[1], hs[2]}, h1 = {hs[3], hs[4], hs[5], hs[6]}, h2 = {hs[7], hs[8], hs[9], hs[10]},
            h3 = {hs[11], hs[12], hs[13], hs[14]};
  asm volatile(
      "s_brev_b64 exec, 1\n\t"
      "ds_write_b128 %0, %1 offset:%7\n\t"
      "ds_write_b128 %0, %2 offset:%8\n\t"
      "ds_write_b128 %0, %3 offset:%9\n\t"
      "ds_write_b128 %0, %4 offset:%10\n\t"
      "ds_write_b32 %5, %6\n\t"
      "s_mov_b64 exec, -1"
      :
      : "v"(to), "v"(h0), "v"(h1), "v"(h2), "v"(h3), "v"(count), "v"(col), "n"(OFFSET), "n"(OFFSET + 16),
        "n"(OFFSET + 32), "n"(OFFSET + 48)
      : "memory");
}

// 16 steps starting at t0 (a multiple of 16) for the fill that stages S in
// registers.  MASKED chunks (the first 64 steps and the steps past column m)
// update H only where 1 <= j <= m, so a lane keeps H[i][0] until its column
// starts and keeps H[i][m] after it ends; in between every lane is active.
// Every step shifts the last-row collector st.col (lane 63 enters).
template <bool MASKED, bool MAX3>
static __device__ __forceinline__ void run16v(StripState &st, const float4 (&sv)[4], int t0, int m, float g,
                                              int lane, uint32_t &U, uint32_t &L) {
  float H = st.H, diag = st.diag, pw = st.pw, col = st.col;
  int d = t0 - lane;   // column - 1 of this lane at the current step
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const float4 v4 = sv[u >> 2];
    const float s = (u & 3) == 0 ? v4.x : (u & 3) == 1 ? v4.y : (u & 3) == 2 ? v4.z : v4.w;
    const float next = dpp_next(pw);
    const float x = dpp_shr1(pw, H);   // H[i-1][j]: lane r-1, or the boundary row for lane 0
    pw = next;
    const float best = cell<MAX3>(x + g, H + g, diag + s, U, L);
    if (MASKED) {
      H = ((unsigned)d < (unsigned)m) ? best : H;
      ++d;
    } else {
      H = best;
    }
    diag = x;
    col = dpp_shl1(H, col);
  }
  st.H = H;
  st.diag = diag;
  st.pw = pw;
  st.col = col;
}

struct FillArgs {
  int n_items, B;
  int item0;        // first work item of this launch (its queue counts from 0)
  int n_tasks;      // tasks of this launch (the LDS-ring fill)
  int task0;        // its first task
  int spin_limit;   // polls of a boundary window before the wave gives up
  int hold;         // testing: the first strip of a pair publishes nothing
  const int32_t *it_pair, *it_strip, *n, *m;
  const int32_t *tk_pair, *tk_slot;
  const int64_t *s_off, *tb_off, *bnd_off;
};

// LDS of the LDS-ring fill, per workgroup of SLOTS strips: each strip's S
// ring, then SLOTS + 1 row rings (ring k holds the row above strip k, ring
// SLOTS the last strip's last row on its way to memory; LINK_COLS columns,
// column j in slot (j - 1) % LINK_COLS), then ZERO_BYTES of zeros (what the
// lanes but 0 read as the row above), then the counters: [k] columns put into
// row ring k (-1: its writer gave up), [SLOTS + 1 + k] columns taken from it,
// [2 SLOTS + 2] the task.
constexpr int LINK_COLS = 512;
constexpr int ZERO_BYTES = 512;
constexpr int fill_lds_bytes(int slots) {
  return slots * RING_GROUPS * GROUP_BYTES + (slots + 1) * LINK_COLS * 4 + ZERO_BYTES + 4 * (2 * slots + 3);
}
constexpr int FILL_HELPERS = 2;   // waves per workgroup that move boundary rows from and to memory
constexpr int ALL_COLS = 0x3fffffff;   // columns put of a row that is complete; columns taken by a reader that gave up
static_assert((LINK_COLS & (LINK_COLS - 1)) == 0 && LINK_COLS >= 256, "row ring");

// Published boundary values carry tag 1; clearing them every launch means a
// value left by an earlier launch is never taken as ready.  Only the rows that
// go through memory are cleared, those above a task's first strip: `slots`
// strips a task (1 where no row stays in LDS).  A workgroup takes the rows of
// one DP item after another.  Bound by its stores: 256
// pairs of 5000 x 5000 168 -> 45 us, 4096 pairs of median 60 6.5 -> 5.8 us.
__global__ __launch_bounds__(256) void k_nw_reset(FillArgs A, int slots, uint64_t *__restrict__ bnd,
                                                  int32_t *__restrict__ ctl, float g, float *__restrict__ score) {
  const int64_t tid = blockIdx.x * (int64_t)256 + threadIdx.x;
  const int64_t nthr = (int64_t)gridDim.x * 256;
  for (int k = blockIdx.x; k < A.n_items; k += gridDim.x) {
    const int st = A.it_strip[k] & ITEM_STRIP;
    if (st == 0 || st % slots != 0) continue;
    const int b = A.it_pair[k];
    const int64_t stride = bnd_stride(A.m[b]);   // (even: the rows are 16-byte aligned)
    uint4 *row = reinterpret_cast<uint4 *>(bnd + A.bnd_off[b] + (st - 1) * stride);
    for (int64_t x = threadIdx.x; x < stride / 2; x += 256) row[x] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (tid < 4) ctl[tid] = 0;   // [0] queue head, [1] error flag, [2] queue head of a second launch
  for (int64_t b = tid; b < A.B; b += nthr) {
    const int n = A.n[b], m = A.m[b];
    // H[n][0] = fl32(n*g), H[0][m] = fl32(m*g), H[0][0] = +0
    if (n == 0 || m == 0) score[b] = (n + m == 0) ? 0.0f : (float)(n + m) * g;
  }
}

template <bool MAX3, int SLOTS>
__global__ __launch_bounds__(64 * (SLOTS + FILL_HELPERS)) void k_nw_fill(
    FillArgs A, const float *__restrict__ S, float g, float *__restrict__ score, char *__restrict__ tb,
    uint64_t *__restrict__ bnd, int32_t *__restrict__ head, int32_t *__restrict__ err) {
  constexpr uint32_t epoch = 1u;   // tag of a published value (the reset clears to 0)
  extern __shared__ __align__(16) char fill_lds[];   // fill_lds_bytes(SLOTS) bytes
  const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  float *const rows_lds = reinterpret_cast<float *>(fill_lds + SLOTS * RING_GROUPS * GROUP_BYTES);
  float *const zeros = rows_lds + (SLOTS + 1) * LINK_COLS;
  int *const put = reinterpret_cast<int *>(zeros + ZERO_BYTES / 4);
  int *const taken = put + SLOTS + 1;
  int *const task_lds = taken + SLOTS + 1;
  // LDS operations of one wave are performed in order, so a count written
  // after its values (or after the reads of the slots it frees) is never seen
  // before them; only the compiler is kept from reordering.
  auto count = [](const int *c) -> int {
    return uniform(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
  };
  auto set_count = [](int *c, int v) { __hip_atomic_store(c, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };

  for (int k = threadIdx.x; k < ZERO_BYTES / 4; k += 64 * (SLOTS + FILL_HELPERS)) zeros[k] = 0.0f;
  // One task (SLOTS strips, one per wave) at a time: the whole workgroup
  // takes the next task once every wave is done with the last one, so the row
  // rings and counters start clear.  Every wave passes both barriers of every
  // task and leaves the loop at the same task.
  for (;;) {
    __syncthreads();
    if (threadIdx.x < 2 * SLOTS + 2) put[threadIdx.x] = 0;
    if (threadIdx.x == 0) *task_lds = atomicAdd(head, 1);
    __syncthreads();
    const int task = uniform(*task_lds);
    if (task >= A.n_tasks) break;

    if (wave == SLOTS) {
      // ---- rows above, into the row rings: a pair's first row (j g), or the
      // last row of a strip of another task, from memory.  Every published
      // value is one 64-bit agent-coherent (sc1) store of (value, tag 1) into
      // memory the reset kernel cleared, so a value is there when its tag is
      // set: no counters, no store drains and no cache flushes.  64 columns of
      // each strip's row are read per poll; the ready ones at their start go on.
      __amdgpu_buffer_rsrc_t rs[SLOTS];
      int at[SLOTS], m[SLOTS];   // columns handed on; columns of the row (at == m: done)
      bool first[SLOTS];         // a pair's first strip
      int left = 0;              // strips not done
      bool polls = false;        // some row comes from memory
      // lane w reads slot w's records: two dependent loads for all slots instead
      // of a chain of them each, on the way to the strips' first cells (16293
      // pairs of median 8, 91 -> 76 us; 20000 of median 60, 803 -> 747)
      const int tl = (A.task0 + task) * SLOTS + (lane & (SLOTS - 1));
      const int vb = A.tk_pair[tl], vword = A.tk_slot[tl];
      const int vm = A.m[max(vb, 0)];
      const int64_t voff = A.bnd_off[max(vb, 0)];
#pragma unroll
      for (int w = 0; w < SLOTS; ++w) {
        const int b = __builtin_amdgcn_readlane(vb, w), word = __builtin_amdgcn_readlane(vword, w);
        const int s = word & ITEM_STRIP;
        const bool on = b >= 0 && !(word & ITEM_LINK_IN);
        first[w] = s == 0;
        m[w] = on ? __builtin_amdgcn_readlane(vm, w) : 0;
        at[w] = 0;
        const int64_t off = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(voff >> 32), w) << 32 |
                                      (uint32_t)__builtin_amdgcn_readlane((int)voff, w));
        const uint64_t *row = on && s > 0 ? bnd + off + (int64_t)(s - 1) * bnd_stride(m[w]) : bnd;
        rs[w] = __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr(row), (short)0, uniform(on && s > 0 ? 8 * (m[w] + 1) : 0),
                                                  0x00020000);
        left += on;
        polls |= on && s > 0;
      }
      int spins = 0;
      while (left > 0) {
        u32x2v v[SLOTS];
#pragma unroll
        for (int w = 0; w < SLOTS; ++w)   // past the row's end: 0 (not ready), no memory access
          v[w] = __builtin_amdgcn_raw_buffer_load_b64(rs[w], 8 * (at[w] + 1 + lane), 0, CPOL_SC1);
        bool moved = false;
#pragma unroll
        for (int w = 0; w < SLOTS; ++w) {
          if (at[w] == m[w]) continue;
          const int tk = count(&taken[w]);
          const int room = tk + LINK_COLS - at[w];   // the ring's free slots
          const uint64_t wait = __ballot(first[w] ? at[w] + 1 + lane > m[w] : v[w].y != epoch);
          const int ready = wait ? __builtin_ctzll(wait) : 64;
          const int n = room < 64 && first[w] ? 0 : min(ready, room);   // (no row dribbles)
          if (tk == ALL_COLS) {   // the strip gave up
            at[w] = m[w];
            --left;
          } else if (n > 0) {
            const float x = first[w] ? (float)(at[w] + 1 + lane) * g : __uint_as_float(v[w].x);
            if (lane < n) rows_lds[w * LINK_COLS + ((at[w] + lane) & (LINK_COLS - 1))] = x;
            asm volatile("" ::: "memory");
            at[w] += n;
            set_count(&put[w], at[w] == m[w] ? ALL_COLS : at[w]);
            moved = true;
            left -= at[w] == m[w];
          } else if (ready == 0 && (spins >= A.spin_limit || uniform((int)v[w].y) == (int)TAG_FAIL)) {
            // this wave gives up, or the row's writer did
            set_count(&put[w], -1);
            at[w] = m[w];
            --left;
          }
        }
        // (a first row's ring holds some thousand clocks of work)
        if (moved) spins = 0;
        else if (++spins, polls) __builtin_amdgcn_s_sleep(1);
        else __builtin_amdgcn_s_sleep(16);
      }
      continue;
    }

    if (wave == SLOTS + 1) {
      // ---- the last strip's last row, from its row ring to memory
      const int ts = (A.task0 + task) * SLOTS + SLOTS - 1;
      const int b = uniform(A.tk_pair[ts]);
      const int s = b < 0 ? 0 : uniform(A.tk_slot[ts]) & ITEM_STRIP;
      if (b < 0 || s == ((uniform(A.n[b]) + 63) >> 6) - 1 || (A.hold && s == 0)) continue;
      const int m = uniform(A.m[b]);
      uint64_t *row = bnd + A.bnd_off[b] + (int64_t)s * bnd_stride(m);
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr(row), (short)0, uniform(8 * (m + 1)), 0x00020000);
      const float *ring = rows_lds + SLOTS * LINK_COLS;
      int at = 0;
      uint32_t poll = 0;
      for (int spins = 0; at < m;) {
        const int have = min(count(&put[SLOTS]), m);
        if (have > at) {
          const int n = min(have - at, 64);
          asm volatile("" ::: "memory");
          const float v = ring[(at + lane) & (LINK_COLS - 1)];
          publish(rs, lane < n, at + 1 + lane, ((uint64_t)epoch << 32) | __float_as_uint(v));
          asm volatile("" ::: "memory");
          at += n;
          set_count(&taken[SLOTS], at);
          spins = 0;
        } else if (spins += ++poll % LDS_POLLS == 0, have < 0 || spins > std::max(A.spin_limit, SPIN_LIMIT)) {
          // the strip gave up: the one below must not wait for values that
          // will never come
          for (int j = at + 1 + lane; j <= m; j += 64)
            __hip_atomic_store(row + j, (uint64_t)TAG_FAIL << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          set_count(&taken[SLOTS], ALL_COLS);
          break;
        } else {
          __builtin_amdgcn_s_sleep(1);
        }
      }
      continue;
    }

    // ---- one strip
    const int ts = (A.task0 + task) * SLOTS + wave;   // this wave's task slot
    const int b = uniform(A.tk_pair[ts]), s_tag = uniform(A.tk_slot[ts]);
    asm volatile("" ::"s"(b), "s"(s_tag));   // (loaded together)
    if (b < 0) continue;   // an empty slot
    const int s = s_tag & ITEM_STRIP;
    const bool hot = (s_tag & ITEM_HOT) != 0;
    if (hot) __builtin_amdgcn_s_setprio(2);
    const int n = uniform(A.n[b]), m = uniform(A.m[b]);
    const int nstrips = (n + 63) >> 6;
    const bool last = s == nstrips - 1;
    const int i0 = 64 * s;
    const int rows = min(64, n - i0);
    const float *Sb = S + A.s_off[b];
    const int64_t tb_off = uniform64(A.tb_off[b]);
    const int nG = (m + 63 + 63) >> 6;
    uint4 *tbs = reinterpret_cast<uint4 *>(tb + tb_off) + (int64_t)s * nG * 64 + lane;
    const int T_end = m + rows - 1;
    // column m of a row that goes on leaves with the step after its own
    const int nC = (T_end + (last ? 0 : 1) + CHUNK - 1) / CHUNK;
    const char *ring = fill_lds + wave * RING_GROUPS * GROUP_BYTES;
    const uint32_t ring_la = (uint32_t)uniform((int)(uint32_t)(uintptr_t)(lds_void *)(fill_lds)) +
                             wave * RING_GROUPS * GROUP_BYTES;
    const float *row_in = rows_lds + wave * LINK_COLS;
    float *row_out = rows_lds + (wave + 1) * LINK_COLS;
    bool puts = !last && !(A.hold && s == 0);

    StripSrc src;
    src.rs = __builtin_amdgcn_make_buffer_rsrc((void *)uniform_ptr(Sb + (int64_t)i0 * m), (short)0,
                                               uniform(rows * m * 4), 0x00020000);
#pragma unroll
    for (int j = 0; j < 4; ++j) src.base[j] = s_lane_base(lane, j, m);
    src.step = (uint32_t)uniform(64 * (m - 1));
    // this lane's LDS place of piece c of its row in slot 0
    const char *piece[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
      piece[c] = ring + 1024 * (lane >> 2) + 16 * (16 * (lane & 3) + ((c + 4 * ((lane >> 2) & 3) + (lane & 3)) & 15));

    StripState st;
    const int i = i0 + 1 + lane;
    st.H = (float)i * g;                                    // H[i][0]
    st.diag = (i0 == 0) ? 0.0f : (float)i0 * g;             // lane 0: H[i0][0]
    st.pw = st.col = 0.0f;
    bool failed = false;
    // The pair's offsets are pinned in scalar registers before the S
    // prologue: a wait for them placed after it would also wait for its loads.
    asm volatile("" ::"s"(tb_off));
    const int n_groups = (nC + 3) >> 2;
    load_group(ring_la, src, 0u);
    if (n_groups > 1) load_group(ring_la + GROUP_BYTES, src, 4u * GROUP);

    // Chunk c: the values of chunk c + 1 are read, then 16 steps run on cur.
    // With the last chunk of a group its ring slot (whose values are in
    // registers by now) takes the group after next; the next group, issued
    // four chunks ago, has landed (vmcnt 0).  The row above (columns 16 c + 1
    // .. 16 c + 16, in lane 0; the others read zeros) comes from row ring
    // `wave`; its count is read in the middle of the chunk before, and again
    // while it says that they are not there yet.  A lone wave issues an
    // instruction about every five clocks whatever it is, so what a chunk does
    // besides its steps counts as much as they do: the chunks run in blocks of
    // eight with every LDS address a constant offset, and room in the ring
    // below is checked once per block.
    uint32_t U0 = 0u, U1 = 0u, L0 = 0u, L1 = 0u;   // 64 steps of directions
    int in_have = 0;            // columns put into the row ring above, as last read
    int out_free = LINK_COLS;   // columns the row ring below has room for, as last read
    float4 va[4], vb[4];
    float hs[CHUNK], carry = 0.0f;   // carry: lane 63's H after the chunk before
    uint32_t put_in = (uint32_t)(uintptr_t)(lds_void *)&put[wave];
    asm volatile("" : "+v"(put_in));   // (kept in a vector register, where it is used)
    auto read_have = [&]() {
      in_have = __hip_atomic_load((lds_int *)(uintptr_t)put_in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      asm volatile("" ::: "memory");
    };
    // the sweep ends with the chunk it is in, whose values go nowhere
    int end = nC;
    auto give_up = [&]() {
      failed = true;
      puts = false;
      end = 0;
    };
    // until the row above has `need` columns, or its writer gave up, or the
    // poll limit passed
    auto wait_in = [&](int need) {
      int spins = 0;
#pragma nounroll
      for (uint32_t poll = 1;; ++poll) {
        if (poll > 5) __builtin_amdgcn_s_sleep(1);
        read_have();
        const int have = uniform(in_have);
        if (have >= need) break;
        spins += poll % LDS_POLLS == 0;
        if (have < 0 || spins > A.spin_limit) {
          give_up();
          break;
        }
      }
    };
    // until the row ring below has room for columns up to `col` (columns past
    // m too: its reader runs on past them)
    auto wait_out = [&](int col) {
      int spins = 0;
#pragma nounroll
      for (uint32_t poll = 1; col > out_free; ++poll) {
        spins += poll % LDS_POLLS == 0;
        if (spins > SPIN_LIMIT) {
          give_up();
          break;
        }
        if (poll > 1) __builtin_amdgcn_s_sleep(1);
        const int tk = count(&taken[wave + 1]);
        out_free = tk == ALL_COLS ? tk : tk + LINK_COLS;
      }
    };
    // the values of chunk K of two groups
    auto read_s = [&](float4 (&v)[4], auto k) {
#pragma unroll
      for (int p = 0; p < 4; ++p)
        v[p] = *reinterpret_cast<const float4 *>(piece[4 * (k.value & 3) + p] + (k.value >> 2) * GROUP_BYTES);
    };
    const uint32_t out_la = (uint32_t)(uintptr_t)(lds_void *)row_out;
    uint32_t out_cnt = (uint32_t)(uintptr_t)(lds_void *)&put[wave + 1];
    asm volatile("" : "+v"(out_cnt));
    // Chunk c, in place K of the ring's eight, its row `from` columns after in,
    // its output ((K + 4) & 7) * 64 bytes after out; false if it was the
    // strip's last one
    auto chunk = [&](auto early, auto k, auto from, int c, const float *in, uint32_t out, float4 (&cur)[4],
                     float4 (&nxt)[4]) -> bool {
      constexpr int K = k.value;
      constexpr bool E = early.value;
      if (__builtin_expect(uniform(in_have) < CHUNK * c + CHUNK, 0)) wait_in(CHUNK * c + CHUNK);
      float4 row[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) row[q] = reinterpret_cast<const float4 *>(in + from.value)[q];
      asm volatile("" ::: "memory");
      if ((K & 3) == 3 && lane == 0) set_count(&taken[wave], CHUNK * c + CHUNK);
      if ((K & 3) == 3) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      read_s(nxt, std::integral_constant<int, ((K + 1) & 7)>{});
      asm volatile("" ::: "memory");
      if ((K & 3) == 3 && (c >> 2) + RING_GROUPS < n_groups)
        load_group(ring_la + (K >> 2) * GROUP_BYTES, src, 4u * GROUP * ((c >> 2) + RING_GROUPS));
      U0 = (U0 << 16) | (U1 >> 16);
      L0 = (L0 << 16) | (L1 >> 16);
      if constexpr (MAX3) run8_chain<E ? CHUNK * K : -1>(st, cur, row, g, U1, L1, hs);
      else run8<E ? CHUNK * K : -1>(st, cur, row, g, U1, L1, hs);
      read_have();
      if constexpr (MAX3) run8_chain<E ? CHUNK * K + 8 : -1>(st, cur + 2, row + 2, g, U1, L1, hs + 8);
      else run8<E ? CHUNK * K + 8 : -1>(st, cur + 2, row + 2, g, U1, L1, hs + 8);
      // lgkmcnt(0): nxt and the row above have been read (before the writes
      // below join the queue, and before nxt's slot is refilled)
      __builtin_amdgcn_s_waitcnt(0xc07f);
      // the strip's last row, columns 16 c - 63 .. 16 c - 48 (it starts at step 63)
      if (!E && puts) {
        const int col = CHUNK * c - 48;
        put_row<((K + 4) & 7) * 64>(out, carry, hs, out_cnt, col < m ? col : ALL_COLS);
      }
      carry = hs[15];
      if ((K & 3) == 3) tbs[(c >> 2) * 64] = make_uint4(U0, U1, L0, L1);
      return c + 1 < end;
    };
    auto seg = [&](int q) -> int { return 128 * q & (LINK_COLS - 1); };
    auto lane0 = [&](const float *p) { return lane == 0 ? p : zeros; };
    auto sweep = [&]() {
      const float *const in0 = lane0(row_in);
      using std::integral_constant;
      constexpr std::true_type early{};
      constexpr std::false_type late{};
      if (!(chunk(early, integral_constant<int, 0>{}, integral_constant<int, 0>{}, 0, in0, 0u, va, vb) &&
            chunk(early, integral_constant<int, 1>{}, integral_constant<int, 16>{}, 1, in0, 0u, vb, va) &&
            chunk(early, integral_constant<int, 2>{}, integral_constant<int, 32>{}, 2, in0, 0u, va, vb) &&
            chunk(early, integral_constant<int, 3>{}, integral_constant<int, 48>{}, 3, in0, 0u, vb, va)))
        return;
      for (int q = 0;; ++q) {
        const int c = 4 + 8 * q;
        const float *in = lane0(row_in + seg(q)), *in2 = lane0(row_in + seg(q + 1));
        uint32_t out = out_la + 4 * seg(q);
        asm volatile("" : "+v"(out));
        if (puts && __builtin_expect(128 * q + 128 > out_free, 0)) wait_out(128 * q + 128);
        if (!(chunk(late, integral_constant<int, 4>{}, integral_constant<int, 64>{}, c, in, out, va, vb) &&
              chunk(late, integral_constant<int, 5>{}, integral_constant<int, 80>{}, c + 1, in, out, vb, va) &&
              chunk(late, integral_constant<int, 6>{}, integral_constant<int, 96>{}, c + 2, in, out, va, vb) &&
              chunk(late, integral_constant<int, 7>{}, integral_constant<int, 112>{}, c + 3, in, out, vb, va) &&
              chunk(late, integral_constant<int, 0>{}, integral_constant<int, 0>{}, c + 4, in2, out, va, vb) &&
              chunk(late, integral_constant<int, 1>{}, integral_constant<int, 16>{}, c + 5, in2, out, vb, va) &&
              chunk(late, integral_constant<int, 2>{}, integral_constant<int, 32>{}, c + 6, in2, out, va, vb) &&
              chunk(late, integral_constant<int, 3>{}, integral_constant<int, 48>{}, c + 7, in2, out, vb, va)))
          return;
      }
    };
    if (n_groups > 1) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    read_s(va, std::integral_constant<int, 0>{});
    read_have();
    sweep();
    // the steps of a last block of fewer than four chunks, to the high bits (not
    // of a block that holds none but the step after column m's)
    if (!failed && (nC & 3) != 0 && (nC >> 2) < nG) {
      const int sh = 16 * (4 - (nC & 3));
      const uint64_t u = (((uint64_t)U0 << 32) | U1) << sh, l = (((uint64_t)L0 << 32) | L1) << sh;
      tbs[(nC >> 2) * 64] = make_uint4((uint32_t)(u >> 32), (uint32_t)u, (uint32_t)(l >> 32), (uint32_t)l);
    }
    // no LDS-direct load may still be writing LDS when the next task starts
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (last) {
      // H[n][m]: row n's lane after step T_end - 1
      const int u_last = (T_end - 1) & (CHUNK - 1);
      float v = hs[0];
#pragma unroll
      for (int u = 1; u < CHUNK; ++u) v = u == u_last ? hs[u] : v;
      if (lane == n - 1 - i0) score[b] = failed ? __builtin_nanf("") : v;
    }
    if (failed) {
      // neither neighbour waits for this strip
      if (lane == 0) {
        set_count(&taken[wave], ALL_COLS);
        if (!last) set_count(&put[wave + 1], -1);
        __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (hot) __builtin_amdgcn_s_setprio(0);
  }
}

// ---- the fill with S staged in registers -----------------------------------------
// The same strip sweep, the same cells, hand-off and publication as k_nw_fill,
// with every memory access an ordinary compiler-tracked load or store: no LDS
// ring and no hand-counted waits.  Lane r loads the 16 cells of its row that
// a 16-step chunk uses (four 16-byte buffer loads of consecutive columns: the
// cell of step t is (r, t - r), byte 4 (r (m - 1) + t) of the strip) two
// chunks ahead into one of three register sets; lanes 0..15 load that chunk's
// boundary window the same way (agent-coherent 8-byte loads).  A cell outside
// the strip's columns reads another cell of the strip, or 0 past its end (the
// buffer range check): only masked steps see it.  Without the 17 KiB ring a
// wave needs registers only, so more waves fit on a compute unit.
typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ void load_s16(float4 (&d)[4], __amdgpu_buffer_rsrc_t rs, uint32_t off) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const u32x4v v = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16u * q, 0, 0);
    d[q] = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
  }
}

template <bool MAX3>
__global__ __launch_bounds__(64) void k_nw_fill_r(FillArgs A, const float *__restrict__ S, float g,
                                                  float *__restrict__ score, char *__restrict__ tb,
                                                  uint64_t *__restrict__ bnd, int32_t *__restrict__ head,
                                                  int32_t *__restrict__ err) {
  constexpr uint32_t epoch = 1u;   // tag of a published value (the reset clears to 0)
  const int lane = threadIdx.x;
  for (;;) {
    int item = 0;
    if (lane == 0) item = atomicAdd(head, 1);
    item = uniform(item);
    if (item >= A.n_items) break;
    item += A.item0;
    const int b = uniform(A.it_pair[item]);
    const int s_tag = uniform(A.it_strip[item]);
    const int s = s_tag & ~ITEM_HOT;
    const bool hot = (s_tag & ITEM_HOT) != 0;
    if (hot) __builtin_amdgcn_s_setprio(2);
    const int n = uniform(A.n[b]), m = uniform(A.m[b]);
    const int nstrips = (n + 63) >> 6;
    const bool last = s == nstrips - 1;
    const int i0 = 64 * s;
    const int rows = min(64, n - i0);
    const float *Sb = S + A.s_off[b];
    const int64_t mstride = bnd_stride(m);
    const uint64_t *in_row = bnd + A.bnd_off[b] + (int64_t)(s - 1) * mstride;   // used when s > 0
    uint64_t *out_row = bnd + A.bnd_off[b] + (int64_t)s * mstride;               // used when !last
    const int nG = (m + 63 + 63) >> 6;
    uint16_t *tbw = reinterpret_cast<uint16_t *>(reinterpret_cast<uint4 *>(tb + A.tb_off[b]) + (int64_t)s * nG * 64);
    const int T_end = m + rows - 1;
    const int T_pad = (T_end + 15) & ~15;
    const int r_last = n - 1 - i0;   // lane of row n in the last strip
    bool failed = false;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)uniform_ptr(Sb + (int64_t)i0 * m), (short)0, uniform(rows * m * 4), 0x00020000);
    const uint32_t lo = (uint32_t)lane * (uint32_t)(m - 1) * 4u;
    const __amdgpu_buffer_rsrc_t pub_rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)uniform_ptr(out_row), (short)0, last ? 0 : uniform((m + 1) * 8), 0x00020000);

    StripState st;
    const int i = i0 + 1 + lane;
    st.H = (float)i * g;                                    // H[i][0]
    st.diag = (i0 == 0) ? 0.0f : (float)i0 * g;             // lane 0: H[i0][0]
    st.col = 0.0f;
    st.pw = 0.0f;

    // the row above: lanes 0..15 hold slots tw + 1 .. tw + 16 (see k_nw_fill)
    auto wload = [&](int tw) -> uint64_t {
      return (s > 0 && lane < 16)
                 ? __hip_atomic_load(in_row + tw + 1 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                 : 0ull;
    };
    auto window_need = [&](int tw) -> bool { return lane < 16 && tw + 1 + lane <= m; };
    auto wait_window = [&](int tw, uint64_t v) -> uint64_t {
      int spins = 0;
      for (;;) {
        const uint32_t tag = (uint32_t)(v >> 32);
        if (__ballot(window_need(tw) && tag == TAG_FAIL) != 0) {
          failed = true;
          break;
        }
        if (__ballot(window_need(tw) && tag != epoch) == 0) break;
        if (++spins > A.spin_limit) {
          failed = true;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        v = wload(tw);
      }
      return v;
    };

    float4 SA[4], SB[4], SC[4];
    load_s16(SA, rs, lo);
    uint64_t WA = wload(0);
    load_s16(SB, rs, lo + 64u);
    uint64_t WB = wload(16), WC = 0ull;
    int t0 = 0;
    // one 16-step chunk from register set CUR while chunk t0 + 32 loads into NXT
#define NWM_FILL_RCHUNK(CUR, WCUR, NXT, WNXT)                                                       \
  {                                                                                                \
    if (t0 >= T_pad) break;                                                                        \
    load_s16(NXT, rs, lo + 4u * (uint32_t)(t0 + 32));                                              \
    WNXT = wload(t0 + 32);                                                                         \
    uint64_t win = WCUR;                                                                           \
    if (s > 0 && __ballot(window_need(t0) && (uint32_t)(win >> 32) != epoch) != 0) {               \
      win = wait_window(t0, win);                                                                  \
      if (failed) break;                                                                           \
    }                                                                                              \
    st.pw = s > 0 ? __uint_as_float((uint32_t)win) : (float)(t0 + 1 + lane) * g;                  \
    uint32_t U = 0u, L = 0u;                                                                       \
    if (t0 < 64 || t0 + 16 > m) run16v<true, MAX3>(st, CUR, t0, m, g, lane, U, L);      \
    else run16v<false, MAX3>(st, CUR, t0, m, g, lane, U, L);                             \
    {                                                                                              \
      const int j = t0 - 110 + lane;                                                               \
      const bool pub = !last && lane >= 48 && j >= 1 && j <= m && !(A.hold && s == 0);             \
      publish(pub_rs, pub, j, ((uint64_t)epoch << 32) | __float_as_uint(st.col));                  \
    }                                                                                              \
    /* 16-bit places of chunk c in a block row's planes: c ^ 1 of each (first step high) */        \
    tbw[((t0 >> 6) * 64 + lane) * 8 + (((t0 >> 4) & 3) ^ 1)] = (uint16_t)U;                        \
    tbw[((t0 >> 6) * 64 + lane) * 8 + 4 + (((t0 >> 4) & 3) ^ 1)] = (uint16_t)L;                    \
    t0 += 16;                                                                                      \
  }
    for (;;) {
      NWM_FILL_RCHUNK(SA, WA, SC, WC)
      NWM_FILL_RCHUNK(SB, WB, SA, WA)
      NWM_FILL_RCHUNK(SC, WC, SB, WB)
    }
#undef NWM_FILL_RCHUNK
    if (last) {
      // lane r_last stopped updating after column m: it holds H[n][m]
      const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st.H), r_last));
      if (lane == 0) score[b] = failed ? __builtin_nanf("") : v;
    } else if (failed) {
      for (int j = 1 + lane; j <= m; j += 64)
        __hip_atomic_store(out_row + j, (uint64_t)TAG_FAIL << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (failed && lane == 0) __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (hot) __builtin_amdgcn_s_setprio(0);
  }
}

// ---- traceback (Sec. 5.1): from (n, m) back to the first row or column ------------
// following the stored directions; every DIAG step emits the aligned pair.
// Position: strip s, row r of the strip, anti-diagonal step t = j - 1 + r.  From
// step t of row r the path goes LEFT to the first direction that is not LEFT
// at or before t and leaves the row there by DIAG (step - 2) or UP (step - 1);
// it ends with a step below r (column 0) or above strip 0.
//
// A walk is a chain of table lookups, one per row: a pair of 5000 sentences a
// side took 0.4 ms of one wave.  So tall pairs (by_strips) are walked by all
// their strips at once.  k_nw_walk_map climbs each strip from every step of its
// bottom row that the path may enter it at (MAP_COLS steps around the line from
// (0, 0) to (n, m)) and keeps where each leaves it and after how many DIAG
// steps; k_nw_walk_chain composes these maps from the bottom strip up, one
// lookup per strip (strips the path enters outside their maps are climbed on the
// spot, several at once); k_nw_walk then climbs each strip from its known entry and writes its
// aligned pairs at their known place.  The other pairs (chains no longer than
// the three launches) are walked strip by strip by one wave of k_nw_walk.  The
// maps and entries lie in the pair's published boundary rows, which are done
// with: every one holds at least BND_PAD slots, and a pair of n_s strips has
// n_s - 1 of them, one for each strip but the bottom one, whose entry is known.
// Measured (us, all launches; one wave per pair before): six pairs of about 3000
// sentences 420 -> 43, 100 pairs of 20 to 2000 160 -> 40, 64 pairs of 5000 394
// -> 101; far off the line: 5000 x 3000 with a preface of 2000 86 -> 78, with an
// appendix of 2000 99 -> 111, 6400 x 400 along a side 118 -> 116.
constexpr int MAP_COLS = 256;               // entry steps a strip's map covers
constexpr int MAP_BLOCKS = 2 * MAP_COLS / 64;   // blocks of directions it may read: as many steps to the left again
constexpr int WALK_BLOCKS = 5;              // blocks one climbing wave holds
constexpr uint32_t MAP_NONE = 0xFFFFFFFFu;  // the map does not know
constexpr uint32_t MAP_END = 0x80000000u;   // the path ends in the strip (| DIAG steps)
// else (step of the strip above) << 7 | DIAG steps
static_assert(8 * BND_PAD >= 4 * MAP_COLS + 32, "a strip's map, its entry and the bottom strip's exit fit a boundary row");

// first step of strip s's map (s above the bottom strip): a multiple of 64.  The
// path enters at steps 63 .. m + 62, so the map ends no later than it has to
// and starts at 64 rather than 0 where it can: up to 193 columns it holds all
// of them, up to 257 all but the first.
static __device__ __forceinline__ int map_base(int s, int n, int m) {
  const int t = (int)((int64_t)m * (64 * s + 64) / n) + 62;
  const int last = max(0, (m + 62 - MAP_COLS + 64) & ~63);
  return min(max((t - MAP_COLS / 2 + 32) & ~63, 64), last);
}

// strip s's boundary row as 32-bit words: the map, then {step, pairs before it}
// of the strip's entry (step -1: the path ends below it) and, in the last row,
// the bottom strip's exit
static __device__ __forceinline__ uint32_t *map_row(const PlanDev &P, uint64_t *bnd, int b, int m, int s) {
  return reinterpret_cast<uint32_t *>(bnd + P.bnd_off[b] + (int64_t)s * bnd_stride(m));
}
constexpr int MAP_ENTRY = MAP_COLS, MAP_BOTTOM = MAP_COLS + 4;

// A row's 64 steps of one block as masks, bit 63 - p for step 64 G + p: not
// LEFT (nl), and UP (u).  Column 0 (step r - 1 of row r) goes UP, so a climb
// needs no check for it: a path there leaves the strip without another cell.
struct RowMasks {
  uint64_t nl, u;
};
static __device__ __forceinline__ RowMasks row_masks(const uint4 &w, int G, int r) {
  const uint64_t u = ((uint64_t)w.x << 32) | w.y, l = ((uint64_t)w.z << 32) | w.w;
  const uint64_t col0 = G == 0 && r > 0 ? 1ull << (64 - r) : 0ull;
  return {u | ~l | col0, u | col0};
}

// Every lane of the wave climbs one strip from step t of row r0, over the blocks
// from step t0 on held in wnd (t lies in them); returns what a map holds.  Bound
// by the lookups' latency: one 16-byte LDS read and some 20 instructions per row.
// A lane that leaves the blocks held goes on over the first and is dropped at
// the end (its step only decreases).
static __device__ __forceinline__ uint32_t climb_lanes(const RowMasks *wnd, int t0, int r0, int t) {
  int cnt = 0;
  bool ended = false;
  for (int r = r0; r >= 0; --r) {
    uint64_t x, u;
    for (;;) {
      const RowMasks w = wnd[(max(t - t0, 0) >> 6) * 64 + r];
      const int q = ~t & 63;
      x = w.nl >> q, u = w.u >> q;
      // LEFT past the first step of the block, in any lane: on in the block
      // before it (the other lanes look the same masks up again)
      const bool on = x == 0ull && t >= t0;
      if (__ballot(on) == 0ull) break;
      if (on) t = (t & ~63) - 1;
    }
    // (only in row 0: column 0 is step -1 there, and no mask has it)
    ended = t < 0;
    const int k = __builtin_ctzll(x | (1ull << 63));
    const int diag = 1 - (int)((u >> k) & 1ull);
    if (!ended) t -= k + 1 + diag, cnt += diag;
  }
  if (t < t0 && t0 > 0) return MAP_NONE;
  return ended ? MAP_END | (uint32_t)cnt : (uint32_t)(t + 64) << 7 | (uint32_t)cnt;
}

// One workgroup per strip, one lane per entry step.
__global__ __launch_bounds__(MAP_COLS) void k_nw_walk_map(PlanDev P, const char *__restrict__ tb_bits,
                                                          const float *__restrict__ score, uint64_t *__restrict__ bnd,
                                                          int k0) {
  __shared__ RowMasks wnd[MAP_BLOCKS * 64];
  const int b = P.wk_pair[k0 + blockIdx.x], s = P.wk_strip[k0 + blockIdx.x];
  if (__builtin_isnan(score[b])) return;   // a fill that gave up
  const int n = P.n[b], m = P.m[b];
  const int nS = (n + 63) >> 6, nG = (m + 63 + 63) >> 6;
  const bool bottom = s == nS - 1;
  const int r0 = bottom ? (n - 1) & 63 : 63;
  const int t_last = m - 1 + r0;   // the step of column m
  const int w0 = bottom ? max(0, (t_last >> 6 << 6) - (MAP_COLS - 64)) : map_base(s, n, m);
  const int g0 = max((w0 >> 6) - MAP_BLOCKS / 2, 0);
  const uint4 *tbs = reinterpret_cast<const uint4 *>(tb_bits + P.tb_off[b]) + (int64_t)s * nG * 64;
#pragma unroll
  for (int k = threadIdx.x; k < MAP_BLOCKS * 64; k += MAP_COLS) {
    const int G = min(g0 + (k >> 6), nG - 1);   // (blocks past the last step: never read)
    wnd[k] = row_masks(tbs[(int64_t)G * 64 + (k & 63)], G, k & 63);
  }
  __syncthreads();
  const uint32_t out = climb_lanes(wnd, 64 * g0, r0, bottom ? t_last : min(w0 + (int)threadIdx.x, t_last));
  if (!bottom) map_row(P, bnd, b, m, s)[threadIdx.x] = w0 + (int)threadIdx.x > t_last ? MAP_NONE : out;
  else if (threadIdx.x == 0) map_row(P, bnd, b, m, nS - 2)[MAP_BOTTOM] = out;
}

// One 1 KiB row of a map into LDS (lane l: bytes 16 l .. 16 l + 15),
// LDS-direct so that no register is written while the load is in flight (the
// compiler takes an asm load's outputs as written at issue and may copy them).
// Readers wait with an explicit vmcnt.
static __device__ __forceinline__ void load_map_lds(uint32_t *to, const uint4 *src) {
  const uint32_t la = (uint32_t)uniform((int)(uint32_t)(uintptr_t)(lds_void *)to);
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off"
      :
      : "s"(la), "v"(src)
      : "memory", "m0");
}

// The wave climbs one strip (directions tbs, nG blocks) from step t of row r0.
// wnd: WALK_BLOCKS KiB of LDS of the wave's own.  cell: this lane's row's
// column step of its DIAG cell, -1 if it has none.  Returns what a map holds.
static __device__ __forceinline__ uint32_t climb_strip(const uint4 *__restrict__ tbs, uint4 *wnd, int r0, int t,
                                                       int lane, int &cell) {
  cell = -1;
  int r = uniform(r0);
  t = uniform(t);
  int g0 = 0x7fffffff;   // the lowest block in wnd
  // the WALK_BLOCKS blocks up to G (block 0 again for those below it)
  u32x4v n0, n1, n2, n3, n4;
  static_assert(WALK_BLOCKS == 5, "fetch, keep");
  auto at = [&](int G) { return *reinterpret_cast<const u32x4v *>(tbs + (int64_t)max(G, 0) * 64 + lane); };
  for (;;) {             // one block of 64 steps at a time
    if (t < r) return MAP_END | (uint32_t)__popcll(__ballot(cell >= 0));
    const int G = t >> 6;
    if (G < g0) {
      if (G != g0 - 1) n0 = at(G - 4), n1 = at(G - 3), n2 = at(G - 2), n3 = at(G - 1), n4 = at(G);   // (the first)
      g0 = G - (WALK_BLOCKS - 1);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      u32x4v *const to = reinterpret_cast<u32x4v *>(wnd) + lane;
      to[0] = n0, to[64] = n1, to[128] = n2, to[192] = n3, to[256] = n4;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      // the ones to the left of these, while these are climbed
      n0 = at(g0 - 5), n1 = at(g0 - 4), n2 = at(g0 - 3), n3 = at(g0 - 2), n4 = at(g0 - 1);
    }
    const RowMasks w = row_masks(wnd[(G - g0) * 64 + lane], G, lane);
    const int nl1 = (int)(uint32_t)(w.nl >> 32), nl0 = (int)(uint32_t)w.nl;
    const int u1 = (int)(uint32_t)(w.u >> 32), u0 = (int)(uint32_t)w.u;
    // One row per iteration, on the scalar unit, some 120 clocks (180 as the
    // compiler orders it).  q: bit of the step in the block; past 63 the block
    // is done with (the move before left it, or no bit is left in the row).
    // The row's lane gets the step of its DIAG cell, -1 after UP.
    int q = ~t & 63;
    asm("0:\n\t"
        "v_readlane_b32 s88, %[nl0], %[r]\n\t"
        "v_readlane_b32 s89, %[nl1], %[r]\n\t"
        "v_readlane_b32 s90, %[u0], %[r]\n\t"
        "v_readlane_b32 s91, %[u1], %[r]\n\t"
        "s_mov_b32 m0, %[r]\n\t"
        "s_lshr_b64 s[88:89], s[88:89], %[q]\n\t"
        "s_ff1_i32_b64 s92, s[88:89]\n\t"   // (-1 without a bit)
        "s_min_u32 s92, s92, 64\n\t"
        "s_add_i32 s92, s92, %[q]\n\t"
        "s_cmp_gt_i32 s92, 63\n\t"
        "s_cbranch_scc1 1f\n\t"
        "s_sub_i32 s93, %[end], s92\n\t"
        "s_add_i32 %[q], s92, 2\n\t"
        "s_bitcmp1_b64 s[90:91], s92\n\t"
        "s_cselect_b32 s93, -1, s93\n\t"
        "s_subb_u32 %[q], %[q], 0\n\t"
        "v_writelane_b32 %[cell], s93, m0\n\t"
        "s_sub_u32 %[r], %[r], 1\n\t"
        "s_cbranch_scc0 0b\n\t"
        "1:"
        : [cell] "+v"(cell), [r] "+s"(r), [q] "+s"(q)
        : [nl0] "v"(nl0), [nl1] "v"(nl1), [u0] "v"(u0), [u1] "v"(u1), [end] "s"(64 * G + 63)
        : "s88", "s89", "s90", "s91", "s92", "s93", "m0", "scc");
    t = 64 * G + 63 - (r < 0 ? q : max(q, 64));
    if (r < 0) return (uint32_t)(t + 64) << 7 | (uint32_t)__popcll(__ballot(cell >= 0));
  }
}

// The strip's DIAG cells to the path, `before` of the pair's being emitted
// already: cell number q of the walk (rows descending) at pa[cap - 1 - q].
static __device__ __forceinline__ void emit_strip(int2 *__restrict__ pa, int cap, int s, int before, int lane, int cell) {
  const uint64_t has = __ballot(cell >= 0);
  if (cell < 0) return;
  const int q = before + __popcll(lane == 63 ? 0ull : has >> (lane + 1));
  if (q < cap) pa[cap - 1 - q] = make_int2(64 * s + lane, cell - lane);
}

// One workgroup per pair; its first wave looks one strip up after another, in the
// maps, which come into LDS CHAIN_AHEAD strips ahead; the entries leave 64
// strips at a time.  Where the path is off the maps (a preface without a
// counterpart shifts it by the preface's length) all waves climb ahead: wave w
// climbs w strips up, from the 64 entry steps around where the path comes if it
// goes on as in the strip before, and the first wave follows the path through
// these for as far as they hold it.  Without this the strips were climbed one
// by one, 3.7 us each (5000 x 3000 sentences with a preface of 2000, the whole
// traceback: 78 us, 237 so and 86 by one wave in LDS; a pair on the line 37).
constexpr int CHAIN_AHEAD = 16;
constexpr int AHEAD_BLOCKS = 4;   // blocks held of a strip climbed ahead
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_nw_walk_chain(PlanDev P, const char *__restrict__ tb_bits,
                                                      const float *__restrict__ score, uint64_t *__restrict__ bnd,
                                                      int32_t *__restrict__ n_diag, int k0) {
  __shared__ __align__(16) uint32_t maps[CHAIN_AHEAD * MAP_COLS];
  // climbing ahead, then its results (each wave's over the blocks it held); or
  // the strip that wave 0 climbs alone
  __shared__ RowMasks held[WAVES][AHEAD_BLOCKS * 64];
  __shared__ int order[3];   // strip (-1: no more), entry step, how far the entry moves per strip
  const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int b = uniform(P.wp_pair[k0 + blockIdx.x]);
  if (__builtin_isnan(score[b])) {   // a fill that gave up: no aligned pairs
    if (threadIdx.x == 0) n_diag[b] = 0;
    return;
  }
  const int n = uniform(P.n[b]), m = uniform(P.m[b]);
  const int nS = (n + 63) >> 6, nG = (m + 63 + 63) >> 6;
  const uint4 *tbw = reinterpret_cast<const uint4 *>(tb_bits + P.tb_off[b]);
  // first entry step of the strip w above strip s, entered at step t
  auto ahead_base = [&](int w, int t, int move) { return min(max(t - w * move - 32, 0), max(m + 62 - 63, 0)); };
  auto climb_ahead = [&](int s, int t, int move) {
    const int strip = s - wave;
    if (strip < 0) return;
    const int first = ahead_base(wave, t, move);
    const int g0 = max(((first + 63) >> 6) - (AHEAD_BLOCKS - 1), 0);
    const uint4 *tbs = tbw + (int64_t)strip * nG * 64;
    uint4 w[AHEAD_BLOCKS];
#pragma unroll
    for (int k = 0; k < AHEAD_BLOCKS; ++k) w[k] = tbs[(int64_t)min(g0 + k, nG - 1) * 64 + lane];
    RowMasks *mine = held[wave];
#pragma unroll
    for (int k = 0; k < AHEAD_BLOCKS; ++k) mine[64 * k + lane] = row_masks(w[k], g0 + k, lane);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int t_in = first + lane;
    uint32_t out = climb_lanes(mine, 64 * g0, 63, min(t_in, m + 62));
    if (t_in > m + 62) out = MAP_NONE;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    reinterpret_cast<uint32_t *>(mine)[lane] = out;
  };
  if (wave > 0) {   // climbs when wave 0 says so
    for (;;) {
      __syncthreads();
      const int s = order[0], t = order[1], move = order[2];
      if (s < 0) return;
      climb_ahead(s, t, move);
      __syncthreads();
    }
  }
  uint32_t *rows = uniform_ptr(map_row(P, bnd, b, m, 0));
  const int64_t stride = 2 * bnd_stride(m);   // words per row
  uint4 *const wnd = reinterpret_cast<uint4 *>(held);
  uint32_t out = (uint32_t)uniform((int)rows[(int64_t)(nS - 2) * stride + MAP_BOTTOM]);
  int cell;
  if (out == MAP_NONE)
    out = climb_strip(tbw + (int64_t)(nS - 1) * nG * 64, wnd, (n - 1) & 63, m - 1 + ((n - 1) & 63), lane, cell);
  int before = (int)(out & 127u);
  const uint4 *next = reinterpret_cast<const uint4 *>(rows + (int64_t)(nS - 2) * stride) + lane;   // the next map to load
  auto load = [&](int s) {   // (strip 0 again below it, so that every strip issues one load: never read)
    load_map_lds(&maps[(s & (CHAIN_AHEAD - 1)) * MAP_COLS], next);
    if (s > 0) next -= stride / 4;
  };
  for (int k = 0; k < CHAIN_AHEAD; ++k) load(nS - 2 - k);
  int climbed = -1, c_t = 0, c_move = 0;   // the strips climbed ahead: from this one up
  int t_below = -1;                        // entry of the strip below s1
  // strip s entered at step t, outside its map
  auto off_map = [&](int s, int t, int below) {
    auto look = [&]() {
      const int w = climbed - s, x = t - ahead_base(w, c_t, c_move);
      if (climbed < 0 || w >= WAVES || (unsigned)x >= 64u) return MAP_NONE;
      return (uint32_t)uniform((int)reinterpret_cast<const uint32_t *>(held[w])[x]);
    };
    uint32_t to = look();
    if (to != MAP_NONE) return to;
    // how far the entry moves per strip: as it just did
    climbed = s, c_t = t, c_move = below < 0 ? 64 : below - t;
    if (lane == 0) order[0] = s, order[1] = t, order[2] = c_move;
    __syncthreads();
    climb_ahead(s, t, c_move);
    __syncthreads();
    to = look();
    if (to != MAP_NONE) return to;
    climbed = -1;   // farther to the left than the blocks held: alone, in their space
    to = climb_strip(tbw + (int64_t)s * nG * 64, wnd, 63, t, lane, cell);
    // vmcnt(0) here, or the compiler puts it where the strips on their maps come
    // by, and they wait for the maps ahead (14 -> 27 us for 79 strips)
    __builtin_amdgcn_s_waitcnt(0x0f70);
    return to;
  };
  for (int s1 = nS - 2; s1 >= 0; s1 -= 64) {   // lane k: strip s1 - k
    const int base = map_base(max(s1 - lane, 0), n, m);
    int2 entry = make_int2(-1, 0);
    for (int k = 0; k < 64 && k <= s1; ++k) {
      const int s = s1 - k;
      if ((out & MAP_END) != 0u) break;
      const int t = (int)(out >> 7);
      if (lane == k) entry = make_int2(t, before);
      const int idx = t - __builtin_amdgcn_readlane(base, k);
      // every strip loads one map, this one CHAIN_AHEAD strips ago
      asm volatile("s_waitcnt vmcnt(15)" ::: "memory");
      static_assert(CHAIN_AHEAD == 16, "the wait above");
      out = (uint32_t)uniform((int)maps[(s & (CHAIN_AHEAD - 1)) * MAP_COLS + (idx & (MAP_COLS - 1))]);
      if ((unsigned)idx >= (unsigned)MAP_COLS) out = MAP_NONE;
      if (__builtin_expect(out == MAP_NONE, 0))
        out = off_map(s, t, k > 0 ? __builtin_amdgcn_readlane(entry.x, max(k - 1, 0)) : t_below);
      before += (int)(out & 127u);
      load(s - CHAIN_AHEAD);
    }
    t_below = __builtin_amdgcn_readlane(entry.x, 63);
    if (s1 - lane >= 0) *reinterpret_cast<int2 *>(rows + (int64_t)(s1 - lane) * stride + MAP_ENTRY) = entry;
  }
  if (lane == 0) order[0] = -1;
  // no LDS-direct load may still be writing LDS when the wave ends
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (lane == 0) n_diag[b] = before;
  __syncthreads();
}

// One wave per strip of the longer pairs (blocks below n_strips), then one per
// pair of dp_order[o0 ...]: the others, strip by strip.
__global__ __launch_bounds__(64) void k_nw_walk(PlanDev P, const char *__restrict__ tb_bits,
                                                  const float *__restrict__ score, uint64_t *__restrict__ bnd,
                                                  int2 *__restrict__ path, int32_t *__restrict__ n_diag, int k0,
                                                  int n_strips, int o0) {
  __shared__ uint4 wnd[WALK_BLOCKS * 64];
  const int lane = threadIdx.x;
  const bool strip = (int)blockIdx.x < n_strips;
  const int b = uniform(strip ? P.wk_pair[k0 + blockIdx.x] : P.dp_order[o0 + blockIdx.x - n_strips]);
  const int n = uniform(P.n[b]), m = uniform(P.m[b]);
  const int nS = (n + 63) >> 6, nG = (m + 63 + 63) >> 6;
  const int cap = min(n, m);
  // an empty side, or a fill that gave up (NaN score): no aligned pairs
  const bool none = n <= 0 || m <= 0 || __builtin_isnan(score[b]);
  int s = nS - 1, r = (n - 1) & 63, t = m - 1 + r, before = 0;
  if (strip) {
    if (none) return;
    s = uniform(P.wk_strip[k0 + blockIdx.x]);
    if (s < nS - 1) {
      const int2 entry = *reinterpret_cast<const int2 *>(map_row(P, bnd, b, m, s) + MAP_ENTRY);
      r = 63, t = uniform(entry.x), before = uniform(entry.y);
    }
    if (t < 0) return;   // the path ends below
  } else if (P.by_strips[b]) {
    return;   // by its strips
  } else if (none) {
    if (lane == 0) n_diag[b] = 0;
    return;
  }
  const uint4 *tbw = reinterpret_cast<const uint4 *>(tb_bits + P.tb_off[b]);
  int2 *pa = path + P.p_off[b];
  for (;;) {
    int cell;
    const uint32_t out = (uint32_t)uniform((int)climb_strip(tbw + (int64_t)s * nG * 64, wnd, r, t, lane, cell));
    emit_strip(pa, cap, s, before, lane, cell);
    if (strip) return;
    before += (int)(out & 127u);
    if ((out & MAP_END) != 0u || s == 0) break;
    --s, r = 63, t = (int)(out >> 7);
  }
  if (lane == 0) n_diag[b] = before;
}

// The aligned pairs with S >= thr, in path order.  KEEP_WAVES waves per
// workgroup: all of them on one of the n_long longer pairs wp_pair[q0 ...]
// (what one wave does alone in rounds of 256 cells is a chain of two memory
// latencies a round: 36 us for 5000 cells, 12 so), then one each on pairs of
// dp_order[o0 ...].  A launch without longer pairs has KEEP_ALONE waves per
// workgroup: the sixteen of one leave their places only together (16293 pairs
// of median 8, 14.4 -> 10.5 us).
constexpr int KEEP_WAVES = 16, KEEP_ALONE = 1, KEEP_CELLS = 4;   // cells per lane and round
__global__ __launch_bounds__(64 * KEEP_WAVES) void k_keep(PlanDev P, const float *__restrict__ S, float thr,
                                                          const int2 *__restrict__ path,
                                                          const int32_t *__restrict__ n_diag, int2 *__restrict__ kept,
                                                          int32_t *__restrict__ n_kept, int q0, int n_long, int o0,
                                                          int n_pairs) {
  __shared__ int found[2][KEEP_WAVES];   // kept cells of each wave in a round (two, so that one barrier a round does)
  const int wave = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const bool together = (int)blockIdx.x < n_long;
  int b;
  if (together) {
    b = uniform(P.wp_pair[q0 + blockIdx.x]);
  } else {
    const int o = ((int)blockIdx.x - n_long) * (int)(blockDim.x >> 6) + wave;
    if (o >= n_pairs) return;
    b = uniform(P.dp_order[o0 + o]);
  }
  const int n = uniform(P.n[b]), m = uniform(P.m[b]);
  if (!together && n_long > 0 && P.by_strips[b]) return;   // by a workgroup
  const int cap = min(n, m);
  const int k = min(uniform(n_diag[b]), cap);
  const int2 *pa = path + P.p_off[b] + (cap - k);
  int2 *kp = kept + P.p_off[b];
  const float *Sb = S + P.s_off[b];
  const int first = together ? 64 * KEEP_CELLS * wave : 0, step = 64 * KEEP_CELLS * (together ? KEEP_WAVES : 1);
  int nk = 0;
  // the path loads, then the S loads that depend on them, are each in flight
  // together
  for (int q0 = 0, round = 0; q0 < k; q0 += step, ++round) {
    const int at = q0 + first + lane;
    int2 c[KEEP_CELLS];
    float sv[KEEP_CELLS];
#pragma unroll
    for (int u = 0; u < KEEP_CELLS; ++u) c[u] = at + 64 * u < k ? pa[at + 64 * u] : make_int2(0, 0);
#pragma unroll
    for (int u = 0; u < KEEP_CELLS; ++u) sv[u] = at + 64 * u < k ? Sb[(int64_t)c[u].x * m + c[u].y] : 0.0f;
    uint64_t km[KEEP_CELLS];
    int mine = 0;
#pragma unroll
    for (int u = 0; u < KEEP_CELLS; ++u) {
      km[u] = __ballot(at + 64 * u < k && sv[u] >= thr);
      mine += __popcll(km[u]);
    }
    int to = nk;
    if (together) {
      if (lane == 0) found[round & 1][wave] = mine;
      __syncthreads();
      const int f = lane < KEEP_WAVES ? found[round & 1][lane] : 0;
      for (int w = 0; w < KEEP_WAVES; ++w) {
        const int c = __builtin_amdgcn_readlane(f, w);
        if (w < wave) to += c;
        nk += c;
      }
    } else {
      nk += mine;
    }
#pragma unroll
    for (int u = 0; u < KEEP_CELLS; ++u) {
      if ((km[u] >> lane) & 1ull) kp[to + __popcll(km[u] & ((1ull << lane) - 1ull))] = c[u];
      to += __popcll(km[u]);
    }
  }
  if (lane == 0 && (!together || wave == 0)) n_kept[b] = nk;
}

// compute units; resident fill workgroups per unit for the LDS-ring fill
// with tasks of FILL_SLOTS strips and with single strips, and resident waves
// for the register staging
static int g_fill_cus = 0, g_fill_per = 0, g_fill_per1 = 0, g_fill_per_r = 0;

template <int SLOTS>
static hipError_t fill_ring_attrs(int &per) {
  int a = 0, c = 0;
  hipError_t e = hipFuncSetAttribute((const void *)k_nw_fill<false, SLOTS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     fill_lds_bytes(SLOTS));
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void *)k_nw_fill<true, SLOTS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            fill_lds_bytes(SLOTS));
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_nw_fill<false, SLOTS>, 64 * (SLOTS + FILL_HELPERS), fill_lds_bytes(SLOTS));
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&c, k_nw_fill<true, SLOTS>, 64 * (SLOTS + FILL_HELPERS), fill_lds_bytes(SLOTS));
  per = a < c ? a : c;   // either variant's grid is resident at once
  if (per < 1) per = 1;
  return e;
}

hipError_t fill_set_attrs(int) {
  if (g_fill_cus == 0) {
    int dev = 0, cus = 0, per = 0, per1 = 0, pr = 0, pr3 = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    // the four-strip fill takes more than the default 64 KiB of LDS per workgroup
    if (e == hipSuccess) e = fill_ring_attrs<FILL_SLOTS>(per);
    if (e == hipSuccess) e = fill_ring_attrs<1>(per1);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&pr, k_nw_fill_r<false>, 64, 0);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&pr3, k_nw_fill_r<true>, 64, 0);
    if (e != hipSuccess) return e;
    pr = pr < pr3 ? pr : pr3;   // either variant's grid is resident at once
    g_fill_per = per;
    g_fill_per1 = per1;
    g_fill_per_r = pr > 0 ? pr : 1;
    g_fill_cus = cus > 0 ? cus : 1;
  }
  return hipSuccess;
}

static FillArgs fill_args(const PlanDev &P) {
  FillArgs A;
  A.n_items = P.n_items;
  A.B = P.B;
  A.item0 = 0;
  A.n_tasks = P.n_tasks;
  A.task0 = 0;
  A.spin_limit = SPIN_LIMIT;
  A.hold = 0;
  A.it_pair = P.it_pair;
  A.it_strip = P.it_strip;
  A.tk_pair = P.tk_pair;
  A.tk_slot = P.tk_slot;
  A.n = P.n;
  A.m = P.m;
  A.s_off = P.s_off;
  A.tb_off = P.tb_off;
  A.bnd_off = P.bnd_off;
  return A;
}

// Clears the rows that a fill of this staging publishes and the queue heads;
// scores of empty pairs.
hipError_t launch_nw_reset(const PlanDev &P, float g, float *score, uint64_t *bnd, int32_t *ctl, int staging,
                           hipStream_t st) {
  if (P.B <= 0) return hipSuccess;
  const int blocks = std::min(std::max(P.n_items, (P.B + 255) / 256), 2048);
  hipLaunchKernelGGL(k_nw_reset, dim3((unsigned)blocks), dim3(256), 0, st, fill_args(P),
                     staging == 0 ? FILL_SLOTS : 1, bnd, ctl, g, score);
  return hipGetLastError();
}

// DP items [item0, item0 + n) of the plan (the register staging) or the same
// strips as tasks [task0, task0 + nt) (the LDS ring), popped from the queue
// head `head` (cleared by the reset).  Strips of one pair must all be in one
// launch.
hipError_t launch_nw_fill_items(const PlanDev &P, const float *S, float g, float *score, char *tb, uint64_t *bnd,
                                int32_t *head, int32_t *err, int item0, int n, int task0, int nt,
                                int waves_per_cu, int spin_limit, int hold, int staging, hipStream_t st) {
  if (P.B <= 0 || n <= 0) return hipSuccess;
  if (g_fill_cus == 0) {
    hipError_t e = fill_set_attrs(0);
    if (e != hipSuccess) return e;
  }
  FillArgs A = fill_args(P);
  A.item0 = item0;
  A.n_items = n;
  A.task0 = task0;
  A.n_tasks = nt;
  A.spin_limit = spin_limit > 0 ? spin_limit : SPIN_LIMIT;
  A.hold = hold;
  // every wave of the grid is resident at once (the hand-off between strips
  // waits on other waves), so the grid never exceeds the occupancy; for the
  // LDS ring, waves_per_cu counts the waves of whole workgroups.  Staging 0:
  // LDS ring, tasks of FILL_SLOTS strips; 2: LDS ring, one strip per
  // workgroup (the plan's items as tasks of one); 1: registers.
  const bool max3 = !(g == 0.0f && std::signbit(g));   // a gap of -0 keeps the compare chain (see run16v)
  if (staging == 1) {
    const int per = (waves_per_cu > 0 && waves_per_cu < g_fill_per_r) ? waves_per_cu : g_fill_per_r;
    const int grid = std::min(n, g_fill_cus * per);
    if (max3)
      hipLaunchKernelGGL(k_nw_fill_r<true>, dim3(grid), dim3(64), 0, st, A, S, g, score, tb, bnd, head, err);
    else
      hipLaunchKernelGGL(k_nw_fill_r<false>, dim3(grid), dim3(64), 0, st, A, S, g, score, tb, bnd, head, err);
  } else if (staging == 2) {
    A.tk_pair = P.it_pair;
    A.tk_slot = P.it_strip;
    A.task0 = item0;
    A.n_tasks = n;
    int per = g_fill_per1;
    if (waves_per_cu > 0 && waves_per_cu < per) per = waves_per_cu;
    const int grid = std::min(n, g_fill_cus * per);
    constexpr int lds = fill_lds_bytes(1);
    if (max3)
      hipLaunchKernelGGL((k_nw_fill<true, 1>), dim3(grid), dim3(64 * (1 + FILL_HELPERS)), lds, st, A, S, g, score, tb, bnd, head, err);
    else
      hipLaunchKernelGGL((k_nw_fill<false, 1>), dim3(grid), dim3(64 * (1 + FILL_HELPERS)), lds, st, A, S, g, score, tb, bnd, head, err);
  } else {
    int groups = g_fill_cus * g_fill_per;
    if (waves_per_cu > 0) groups = std::min(groups, std::max(1, g_fill_cus * waves_per_cu / FILL_SLOTS));
    const int grid = std::min(nt, groups);
    constexpr int lds = fill_lds_bytes(FILL_SLOTS);
    if (max3)
      hipLaunchKernelGGL((k_nw_fill<true, FILL_SLOTS>), dim3(grid), dim3(64 * (FILL_SLOTS + FILL_HELPERS)), lds, st, A, S, g, score, tb,
                         bnd, head, err);
    else
      hipLaunchKernelGGL((k_nw_fill<false, FILL_SLOTS>), dim3(grid), dim3(64 * (FILL_SLOTS + FILL_HELPERS)), lds, st, A, S, g, score,
                         tb, bnd, head, err);
  }
  return hipGetLastError();
}

hipError_t launch_nw_fill(const PlanDev &P, const float *S, float g, float *score, char *tb, uint64_t *bnd,
                          int32_t *ctl, int waves_per_cu, int spin_limit, int hold, int staging,
                          hipStream_t st) {
  hipError_t e = launch_nw_reset(P, g, score, bnd, ctl, staging, st);
  if (e != hipSuccess) return e;
  return launch_nw_fill_items(P, S, g, score, tb, bnd, ctl, ctl + 1, 0, P.n_items, 0, P.n_tasks, waves_per_cu,
                              spin_limit, hold, staging, st);
}

// Pairs dp_order[o0 .. o0 + n), among them the longer pairs wp_pair[q0 .. q0 +
// nq) with the strips wk_*[k0 .. k0 + nk).
hipError_t launch_nw_walk(const PlanDev &P, const char *tb, const float *score, uint64_t *bnd, int2 *path,
                          int32_t *n_diag, int o0, int n, int q0, int nq, int k0, int nk, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (nq > 0) {
    hipLaunchKernelGGL(k_nw_walk_map, dim3(nk), dim3(MAP_COLS), 0, st, P, tb, score, bnd, k0);
    // sixteen waves' blocks leave room for one workgroup per compute unit, eight
    // waves' for three
    if (nq <= g_fill_cus)
      hipLaunchKernelGGL(k_nw_walk_chain<16>, dim3(nq), dim3(64 * 16), 0, st, P, tb, score, bnd, n_diag, q0);
    else
      hipLaunchKernelGGL(k_nw_walk_chain<8>, dim3(nq), dim3(64 * 8), 0, st, P, tb, score, bnd, n_diag, q0);
  }
  // (with no other pairs in the range, the strips alone)
  hipLaunchKernelGGL(k_nw_walk, dim3(nk + (nq < n ? n : 0)), dim3(64), 0, st, P, tb, score, bnd, path, n_diag, k0, nk,
                     o0);
  return hipGetLastError();
}

hipError_t launch_keep(const PlanDev &P, const float *S, float thr, const int2 *path, const int32_t *n_diag,
                       int2 *kept, int32_t *n_kept, int o0, int n, int q0, int nq, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int waves = nq > 0 ? KEEP_WAVES : KEEP_ALONE;
  const int others = nq < n ? (n + waves - 1) / waves : 0;
  hipLaunchKernelGGL(k_keep, dim3(nq + others), dim3(64 * waves), 0, st, P, S, thr, path, n_diag, kept, n_kept, q0,
                     nq, o0, n);
  return hipGetLastError();
}

}  // namespace nwm
