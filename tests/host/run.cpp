// One job: a batch from a file, through the library's C entry points on the wave
// machine, results to a file.  The alignment fill (inline assembly) is plain code
// here, and does nothing in nwm_mine.
#include <hip/hip_runtime.h>
#include <sanitizer/asan_interface.h>

#include "libnwmine.h"
#include "nwm_internal.h"

// what lies between the pieces of the workspace of the plan made last
static std::vector<std::pair<size_t, size_t>> gaps;
void host_gap(size_t from, size_t to) { gaps.push_back({from, to}); }

namespace nwm {
hipError_t fill_set_attrs(int) { return 0; }
hipError_t launch_nw_reset(const PlanDev &, float, float *, uint64_t *, int32_t *, int, hipStream_t) { return 0; }
hipError_t launch_nw_fill_items(const PlanDev &, const float *, float, float *, char *, uint64_t *, int32_t *, int32_t *,
                                int, int, int, int, int, int, int, int, hipStream_t) {
  return 0;
}

// The fill in plain code: scores and the traceback's bit planes (what lies
// outside the lattice is noise).
hipError_t launch_nw_fill(const PlanDev &P, const float *S, float g, float *score, char *tb, uint64_t *, int32_t *, int, int, int, int,
                          hipStream_t) {
  uint64_t noise = 88172645463325252ull;
  for (int b = 0; b < P.B; ++b) {
    const int n = P.n[b], m = P.m[b], nG = (m + 126) >> 6;
    std::vector<float> H(m + 1), above(m + 1);
    for (int j = 0; j <= m; ++j) H[j] = (float)j * g;
    uint4 *blocks = reinterpret_cast<uint4 *>(tb + P.tb_off[b]);
    for (int i = 1; i <= n && m > 0; ++i) {
      above = H;
      H[0] = (float)i * g;
      const int s = (i - 1) >> 6, r = (i - 1) & 63;
      std::vector<uint64_t> U(nG), L(nG);
      for (int k = 0; k < nG; ++k)
        for (uint64_t *w : {&U[k], &L[k]}) noise ^= noise << 13, noise ^= noise >> 7, noise ^= noise << 17, *w = noise;
      for (int j = 1; j <= m; ++j) {
        const float up = above[j] + g, left = H[j - 1] + g, diag = above[j - 1] + S[P.s_off[b] + (int64_t)(i - 1) * m + j - 1];
        const float best = std::max(std::max(up, left), diag);
        H[j] = best;
        const int t = j - 1 + r;
        const uint64_t bit = 1ull << (63 - (t & 63));
        U[t >> 6] = up == best ? U[t >> 6] | bit : U[t >> 6] & ~bit;
        L[t >> 6] = left == best ? L[t >> 6] | bit : L[t >> 6] & ~bit;
      }
      for (int k = 0; k < nG; ++k)
        blocks[((int64_t)s * nG + k) * 64 + r] =
            make_uint4((uint32_t)(U[k] >> 32), (uint32_t)U[k], (uint32_t)(L[k] >> 32), (uint32_t)L[k]);
    }
    score[b] = n == 0 || m == 0 ? (n + m == 0 ? 0.0f : (float)(n + m) * g) : H[m];
  }
  return 0;
}
}  // namespace nwm

static FILE *in;
template <typename T>
static T *take(size_t n) {   // exactly as long as its contents
  T *p = (T *)std::malloc(std::max<size_t>(n, 1) * sizeof(T));
  if (std::fread(p, sizeof(T), n, in) != n) std::abort();
  return p;
}
static void check(nwm_status s) {
  if (s != NWM_OK) std::fprintf(stderr, "%s\n", nwm_strerror(s)), std::exit(3);
}

int main(int, char **argv) {
  in = std::fopen(argv[1], "rb");
  const int64_t *h = take<int64_t>(12);
  const int64_t op = h[0], B = h[1], V = h[2], deg = h[3], prec = h[4], bound = h[5], raw = h[6], n_par = h[7];
  const int64_t n_src = h[8], n_tgt = h[9], nnz = h[10], passes = h[11];
  const int64_t *par = take<int64_t>(2 * n_par);
  nwm_batch b{};
  b.B = (int32_t)B;
  b.V = (int32_t)V;
  b.n_host = take<int32_t>(B);
  b.m_host = take<int32_t>(B);
  b.src_off = take<int64_t>(n_src + 1);
  b.src_tokens = b.src_off[n_src];
  b.src_tok = take<int32_t>(b.src_tokens);
  b.tgt_off = take<int64_t>(n_tgt + 1);
  b.tgt_tokens = b.tgt_off[n_tgt];
  b.tgt_tok = take<int32_t>(b.tgt_tokens);
  b.max_sent_tokens = (int32_t)bound;
  nwm_dict d{};
  d.V = (int32_t)V;
  d.max_deg = (int32_t)deg;
  d.row_off = take<int32_t>(V + 1);
  d.col = take<int32_t>(nnz);
  d.val = take<float>(nnz);
  const float *w = take<float>(3);
  const nwm_scorer sc{w[0], w[1], w[2]};
  nwm_ctx *ctx = nullptr;
  check(nwm_create(&ctx, 0));
  nwm_plan *p = nullptr;
  check(nwm_plan_create(ctx, &b, (int32_t)deg, (nwm_prec)prec, &p));
  nwm_sizes z;
  check(nwm_plan_sizes(p, &z));
  for (int64_t k = 0; k < n_par; ++k) check(nwm_plan_set_param(p, (nwm_param)par[2 * k], (int32_t)par[2 * k + 1]));
  check(nwm_plan_set_timing(p, op != 1));
  char *ws = (char *)aligned_alloc(256, (z.ws_bytes + 255) / 256 * 256);
  std::memset(ws, 0xA5, z.ws_bytes);
  for (auto &g : gaps) __asan_poison_memory_region(ws + (g.first + 7) / 8 * 8, g.second - (g.first + 7) / 8 * 8);
  float *S = (float *)std::malloc(4 * z.S_elems + 1), *R = (float *)std::malloc(4 * z.S_elems + 1);
  for (size_t k = 0; k < z.S_elems; ++k) S[k] = R[k] = NAN;
  double wb[3] = {};
  if (op == 2) {   // the dense chain of the backward
    const float *E = take<float>(z.S_elems);
    float *S0 = take<float>(z.S_elems), *R0 = take<float>(z.S_elems);
    check(nwm_align_backward(p, &b, nullptr, nullptr, nullptr, E, S, nullptr, S0, R0, sc, wb, ws, nullptr));
  }
  std::vector<float> f(B + 1, NAN);
  std::vector<int32_t> i(B + 1), j(B + 1), kept(2 * z.kept_cap + 1);
  char *tb = (char *)aligned_alloc(16, (z.tb_bytes + 31) / 16 * 16);
  if (op == 3) {
    const float *gt = take<float>(2);
    float *S0 = take<float>(z.S_elems);
    for (int64_t k = 0; k < passes; ++k)
      check(nwm_align_batch(p, S0, gt[0], gt[1], f.data(), i.data(), kept.data(), j.data(), tb, ws, nullptr));
  }
  for (int64_t k = 0; k < passes; ++k) {
    if (op == 0) check(nwm_score_pairs(p, &b, &d, sc, S, raw ? R : nullptr, ws, nullptr));
    if (op == 1)
      check(nwm_mine(p, &b, &d, sc, -0.2f, 0.5f, S, raw ? R : nullptr, f.data(), i.data(), kept.data(), j.data(), tb, ws, nullptr));
  }
  double ms[NWM_N_KCLASSES];
  int32_t launches[NWM_N_KCLASSES];
  check(nwm_plan_kernel_ms(p, ms, launches, 1));
  FILE *out = std::fopen(argv[2], "wb");
  std::fwrite(launches, 4, NWM_N_KCLASSES, out);
  std::fwrite(wb, 8, 3, out);
  std::fwrite(S, 4, z.S_elems, out);
  std::fwrite(R, 4, z.S_elems, out);
  if (op == 3) {
    std::fwrite(f.data(), 4, B, out);
    std::fwrite(i.data(), 4, B, out);
    std::fwrite(j.data(), 4, B, out);
    std::fwrite(kept.data(), 8, z.kept_cap, out);
  }
  std::fclose(out);
  nwm_destroy(ctx);   // (a plan may outlive its context)
  nwm_plan_destroy(p);
  return 0;
}
