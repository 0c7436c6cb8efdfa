"""The table of GEMM schedules (no GPU needed): every entry holds for every token count that it serves."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_07609_amd", "csrc")

# Walks a table as the scheduler step does, one token count after the other. A launch that cuts K has one item per workgroup and one
# workgroup per compute unit, and its sums and counters have room for that many, so more items than that are never run,
# or leave the buffers. Returns the first token count that breaks a rule, 0 if none does.
HARNESS = r"""
#include <cstdint>
typedef uint32_t u32;
#include "gemm_plan.h"
static bool holds(u32 plan, int epi, u32 N, u32 K, u32 T, bool experts, u32 ncu) {
  static const u32 rows[8] = {0, 64, 128, 128, 256, 0, 256, 256}, toks[8] = {0, 64, 64, 128, 128, 0, 192, 256};
  const u32 shape = plan & 7u, slices = plan >> 3;
  if (shape == PLAN_STREAM) return slices == 0 && (T <= 64 || (experts && T <= 256));
  if (shape == PLAN_TALL) return slices == 0 && T <= 64;
  if (slices == 0) return true;
  if (experts || shape > 4 || (epi != EPI_QKV_ROPE && epi != EPI_RESIDUAL) || slices * 2 > gemm_k_tiles(K)) return false;
  return (uint64_t)((N + rows[shape] - 1) / rows[shape]) * ((T + toks[shape] - 1) / toks[shape]) * slices <= ncu;
}
extern "C" u32 first_that_fails(u32 max_tokens, u32 d, u32 nq, u32 nkv, u32 hd, u32 F, u32 V, u32 experts, u32 ncu, u32 tune, u32* in_slices) {
  const u32 qkv = (nq + 2 * nkv) * hd;
  const std::vector<GemmPlan> plan = gemm_plan_table(max_tokens, qkv, d, nq * hd, F, V, experts, ncu, tune);
  *in_slices = 0;
  for (u32 T = 1; T <= max_tokens; ++T) {
    if (gemm_plan_entry(T) >= plan.size()) return T;
    const GemmPlan& p = plan[gemm_plan_entry(T)];
    if (!holds(p.qkv, EPI_QKV_ROPE, qkv, d, T, experts, ncu) || !holds(p.oproj, EPI_RESIDUAL, d, nq * hd, T, experts, ncu) ||
        !holds(p.gateup, EPI_SILU_GATE, 2 * F, d, T, false, ncu) || (!experts && !holds(p.down, EPI_RESIDUAL, d, F, T, false, ncu)) ||
        !holds(p.lm_head, EPI_SCALED_STORE, V, d, T, false, ncu)) return T;
    *in_slices = (p.qkv >> 3) | (p.oproj >> 3) | (experts ? 0u : p.down >> 3) ? T : *in_slices;
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    (tmp / "plan.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, "-o", str(tmp / "plan.so"), str(tmp / "plan.cpp")], check=True)
    return ctypes.CDLL(str(tmp / "plan.so")).first_that_fails


@pytest.mark.parametrize("ncu", [256, 304, 64])
@pytest.mark.parametrize("experts", [0, 1])
def test_every_schedule_holds_for_the_token_counts_it_serves(table, ncu, experts):
    """Widths from 32 to 4096, most of them narrow: their matrices still have K in slices at 16 k tokens, where one more block of tokens is
    too many items (d_model 160 with d_ffn 9216 at 16385 tokens). Iterations of up to 40000 tokens, the automatic choice and every
    shape and number of slices forced."""
    n = ctypes.c_uint32()
    reach = 0
    for d, nq, nkv, hd in ((32, 1, 1, 64), (96, 2, 1, 64), (128, 1, 1, 128), (160, 4, 4, 64), (256, 8, 2, 64), (1024, 16, 16, 64), (4096, 32, 8, 128)):
        for F in (96, 2048, 4704, 9216, 14336):
            assert table(40000, d, nq, nkv, hd, F, 1003, experts, ncu, 0, ctypes.byref(n)) == 0, (d, F)
            reach = max(reach, n.value)
        for shape in range(1, 8):
            for slices in (0, 2, 3, 5, 8, 15):
                assert table(3000, d, nq, nkv, hd, 4704, 1003, experts, ncu, shape << 12 | slices << 24, ctypes.byref(n)) == 0, (d, shape, slices)
    assert (reach > 10000) == (not experts and ncu >= 256), reach        # (narrow matrices are in slices that far)
