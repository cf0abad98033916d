"""Runs the scoring, traceback and backward kernels' own sources on the host (tests/host: a
wave64 machine of fibers) under the address and undefined-behaviour sanitizers,
behind the library's C entry points.  Every input, the workspace's pieces and
the dynamic LDS are exactly as long as their contents.

The sources are compiled as they are but for LDS declarations, inline assembly
(a compare-and-swap) and a rendezvous wherever a kernel relies on the order in
which the LDS operations of one wave are performed."""
from __future__ import annotations

import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np

from paper_1512_01641_amd import _abi
from paper_1512_01641_amd import build as B

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")
CLANG = "/opt/rocm/llvm/bin/clang++"
SOURCES = ["k_expand", "k_score", "k_sparse", "k_align", "k_backward", "k_bidir", "nwm_abi"]
CHECKS = ["-fsanitize=address,undefined", "-fno-sanitize=alignment,vptr,function", "-fno-sanitize-recover=undefined"]
FLAGS = ["-std=c++17", "-O1", "-w", "-ffp-contract=off", "-I" + HERE, "-I" + B.CSRC, "-I" + os.path.join(B.ROOT, "include")]

SYNC = "wave_sync();"
SWAP = """template <int NQ>
static void cas_round(uint32_t (&old)[NQ], uint32_t *key, const uint32_t (&h)[NQ], uint32_t HS, uint32_t junk,
                      const uint32_t (&w)[MERGE_ROUNDS]) {
  for (int q = 0; q < NQ; ++q) old[q] = atomicCAS(&key[h[q] < HS ? h[q] : junk], HEMPTY, h[q] < HS ? w[q] : HEMPTY);
}
"""
# per source: (pattern, replacement, matches)
EDITS = {
    "k_sparse": [
        # (read of another lane where lanes diverge: taken before)
        (r"const uint32_t alast = half \? \(uint32_t\)(\S+\(\(int\)a, 63\))\s*: \(uint32_t\)(\S+\(\(int\)a, 31\));",
         r"const uint32_t a63 = (uint32_t)\1, a31 = (uint32_t)\2, alast = half ? a63 : a31;", 1),
        (r"const int c = row_cnt\(k\);", r"const int c = row_cnt(k); const int64_t rbk = row_base(k);", 1),
        (r"merged\[row_base\(k\) \+ x\]", "merged[rbk + x]", 1)],
    "k_expand": [
        (r"template <int NQ>\nstatic __device__ __forceinline__ void cas_round.*?\n}\n", SWAP, 1),
        (r"const uint32_t base = [^;]*key;", "uint32_t *const base = key;", 1),
        (r"(?=#pragma unroll\n  for \(int q = 0; q < NQ; \+\+q\)\n    if \(h\[q\] & EXA_JOIN\))", SYNC + "\n", 1),
        (r"(?=#pragma unroll\n  for \(int q = 0; q < NQ; \+\+q\) \{\n    uint2 o =)", SYNC + "\n", 1)],
    "k_score": [
        (r"(scatter_set_regs<BF16>\(nxt, Ao_, Ao_ \+ TB, lane, junk\);)", SYNC + r" \1 " + SYNC, 1),
        (r"(mfma_frags<BF16>\(Fc, acc\);)", SYNC + r" \1", 1),
        (r"(read_frags<BF16>\(F, At1?, Bt1?, lane\);)", r"\1 " + SYNC, 3),
        (r"(mfma_frags<BF16>\(F, acc\);)", SYNC + r" \1", 3)],
    "k_align": [
        # the traceback and the filter only; the fill is plain code (run.cpp)
        (r"// The parallelogram of S used by steps.*?(?=// ---- traceback \(Sec\. 5\.1\))",
         "typedef unsigned int u32x4v __attribute__((ext_vector_type(4)));\n", 1),
        (r"// compute units; resident fill workgroups.*?(?=// Pairs dp_order\[o0)", "static int g_fill_cus = 4;\n", 1),
        (r"const uint32_t la = [^;]*;\n\s*asm volatile\(.*?\"m0\"\);", "std::memcpy(to + 4 * (threadIdx.x & 63), src, 16);", 1),
        (r'asm volatile\("s_waitcnt vmcnt\(\d+\)" ::: "memory"\);', "", 2),
        (r'asm\("0:\\n\\t".*?"scc"\);', """for (;;) {
      const uint64_t nl = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(nl1, r) << 32 | (uint32_t)__builtin_amdgcn_readlane(nl0, r);
      const uint64_t up = (uint64_t)(uint32_t)__builtin_amdgcn_readlane(u1, r) << 32 | (uint32_t)__builtin_amdgcn_readlane(u0, r);
      const int b = q < 64 && nl >> q ? q + __builtin_ctzll(nl >> q) : 64;
      if (b > 63) break;
      const int is_up = (int)(up >> b & 1);
      if (lane == r) cell = is_up ? -1 : 64 * G + 63 - b;
      q = b + 2 - is_up;
      if (--r < 0) break;
    }""", 1)],
    "nwm_abi": [
        # the workspace's pieces stand apart
        (r"size_t r = o;\n\s*o = (align_up\(o \+ std::max<size_t>\(bytes, 1\), 256\));",
         r"size_t r = o; o = \1 + 4096; host_gap(r + bytes, o);", 1),
        (r"constexpr int64_t SPLIT_TILES = 8192;",
         'static const int64_t SPLIT_TILES = getenv("HOST_SPLIT") ? atoll(getenv("HOST_SPLIT")) : 8192;', 1),
        (r"in <= W\.a_choff", "in + 4096 <= W.a_choff", 1),
        (r"const bool shared = ", 'const bool shared = !getenv("HOST_APART") && ', 1),
        (r"^", "#include <stddef.h>\nvoid host_gap(size_t, size_t);\n", 1)],
}


def _source(name):
    with open(os.path.join(B.CSRC, name + ".hip")) as f:
        t = f.read()
    t = re.sub(r"extern __shared__ (?:__align__\(16\) )?(\w+) (\w+)\[\]", r"\1 *const \2 = (\1 *)nwm::host_lds", t)
    t = t.replace("__shared__", "static").replace('asm volatile("" ::: "memory");', "")
    for pattern, to, count in EDITS.get(name, []):
        t, k = re.subn(pattern, (lambda _, to=to: to) if "\n" in to else to, t, count=0 if pattern != r"^" else 1, flags=re.S)
        assert k == count, (name, pattern, k)
    return "#include <hip/hip_runtime.h>\nnamespace nwm { extern char host_lds[]; }\n" + t


def build(folder) -> str:
    """Compiles the machine and the library for it; returns the program."""
    files = [os.path.join(HERE, "machine.cpp"), os.path.join(HERE, "run.cpp")]
    for name in SOURCES:
        files.append(os.path.join(str(folder), name + ".cpp"))
        with open(files[-1], "w") as f:
            f.write(_source(name))

    def one(path):
        obj = os.path.join(str(folder), os.path.basename(path)[:-4] + ".o")
        subprocess.run([CLANG, *FLAGS, *CHECKS, "-c", path, "-o", obj], check=True)
        return obj
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        objs = list(ex.map(one, files))
    out = os.path.join(str(folder), "run")
    subprocess.run([CLANG, *CHECKS, *objs, "-o", out], check=True)
    return out


def run(program, batch, op="score", prec=0, params=None, raw=True, bound=None, passes=1, E=None, S=None, S_raw=None,
        apart=False, split=None, order=None, gap=-0.2, threshold=0.5):
    """One job ("score", "mine", the dense "backward" or "align" over S); a sanitizer report
    ends the program and raises.  apart: no two lists share space; split: tiles
    from which a batch's parts choose their contraction each; order: a seed for the
    order in which waves and lanes run.  Returns S, S_raw, the launches per kernel
    class and the backward's weight gradient."""
    n, m = np.asarray(batch.n, np.int64), np.asarray(batch.m, np.int64)
    bound = int(np.diff(batch.src_off).max(initial=0)) if bound is None else bound
    params = params or {}
    head = [("score", "mine", "backward", "align").index(op), len(n), batch.V, batch.d_deg, prec, bound, int(raw), len(params),
            int(n.sum()), int(m.sum()), len(batch.d_col), passes]
    parts = [np.asarray(head, np.int64), np.asarray([x for k, v in params.items() for x in (_abi.PARAMS[k], v)], np.int64),
             np.asarray(batch.n, np.int32), np.asarray(batch.m, np.int32), batch.src_off, batch.src_tok, batch.tgt_off,
             batch.tgt_tok, batch.d_row_off, batch.d_col, batch.d_val, np.asarray(batch.scorer, np.float32)]
    if op == "backward":
        parts += [np.asarray(x, np.float32) for x in (E, S, S_raw)]
    if op == "align":
        parts += [np.asarray([gap, threshold], np.float32), np.asarray(S, np.float32)]
    folder = os.path.dirname(program)
    job, res = os.path.join(folder, "job"), os.path.join(folder, "result")
    with open(job, "wb") as f:
        for a in parts:
            f.write(np.ascontiguousarray(a).tobytes())
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:detect_stack_use_after_return=0:halt_on_error=1",
               UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
    if apart:
        env["HOST_APART"] = "1"
    if order is not None:
        env["HOST_ORDER"] = str(order)
    if split is not None:
        env["HOST_SPLIT"] = str(split)
    r = subprocess.run([program, job, res], capture_output=True, text=True, env=env)
    if r.returncode != 0:
        raise RuntimeError("exit %d\n%s" % (r.returncode, r.stderr[-4000:]))
    cells = int((n * m).sum())
    with open(res, "rb") as f:
        k = len(LAUNCHES)
        launches = np.frombuffer(f.read(4 * k), np.int32)
        wb = np.frombuffer(f.read(24), np.float64)
        out = [np.frombuffer(f.read(4 * cells), np.float32) for _ in range(2)]
        if op == "align":
            k = len(n)
            return dict(score=np.frombuffer(f.read(4 * k), np.float32), n_diag=np.frombuffer(f.read(4 * k), np.int32),
                        n_kept=np.frombuffer(f.read(4 * k), np.int32),
                        kept=np.frombuffer(f.read(), np.int32).reshape(-1, 2))
    return dict(S=out[0], S_raw=out[1], launches=dict(zip(LAUNCHES, launches.tolist())), grad_wb=wb)


LAUNCHES = ("merge", "build_a", "build_b", "score", "nw_fill", "walk", "keep", "backward", "expand_a")
