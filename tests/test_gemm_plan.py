"""Host-side plans.  Every tile plan of the skinny GEMM names a kernel that
exists, and prefill chunks are even: the planner
(csrc/gemm_plan.h, plain C++) is compiled for the host and walked over weight
shapes and row tiles; launch_gemm instantiates exactly the (epilogue, row tiles,
strips) of gemm_instance and refuses what gemm_launchable does."""
import ctypes
import os
import shutil
import subprocess

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_18583_amd")
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpard.so")

PROGRAM = r"""
#include <cstdio>
#include "gemm_plan.h"
using namespace pard;

// As the engine's run_gemm launches a pass of mt row tiles.
static int check(const char* name, int epi, const GemmPlan& p, int mt) {
  const int S = pick_S(epi, p.n_strips, mt);
  if (gemm_launchable(epi, mt, S, p.nw, p.n_strips, p.kb_total, ceil_div(p.n_strips, S), p.ksplit,
                      ceil_div(p.kb_total, p.ksplit)) && (epi != EPI_RESID || resid_ss_tiles(p) * S == p.n_strips))
    return 0;
  printf("%s: %d strips x %d k-blocks, %d row tiles -> %d strips, %d wavefronts, %d ranges\n", name, p.n_strips,
         p.kb_total, mt, S, p.nw, p.ksplit);
  return 1;
}

// Prefill chunks of n rows: the whole prompt in order, none longer than
// pass_rows, whole units of 128 rows but the last, none of a few rows.
static int check_chunks(int n, int pass_rows) {
  const int m = prefill_chunks(n, pass_rows);
  int at = 0, bad = m != ceil_div(n, pass_rows);
  for (int i = 0; i < m; ++i) {
    const int b = prefill_chunk_begin(n, m, i), e = prefill_chunk_begin(n, m, i + 1);
    bad |= b != at || b % 128 != 0 || e <= b || e - b > pass_rows || (m > 1 && e - b <= 128);
    at = e;
  }
  bad |= at != n;
  if (bad) printf("chunks: %d rows in passes of %d\n", n, pass_rows);
  return bad;
}

int main() {
  int bad = 0;
  for (int pass_rows = 512; pass_rows <= 4096; pass_rows += 256) {
    for (int n = 1; n <= 40000; ++n) bad += check_chunks(n, pass_rows);
    for (int n = 126900; n <= 127100; ++n) bad += check_chunks(n, pass_rows);
    for (int n = (1 << 24) - 400; n <= (1 << 24); n += 7) bad += check_chunks(n, pass_rows);
  }
  // gate/up of 17 to 64 rows: no wider tile than fills its rounds
  for (int mt = 2; mt <= 4; ++mt) {
    bad += pick_S(EPI_SWIGLU, 512, mt) != 2 || pick_S(EPI_SWIGLU, 516, mt) != 4 || pick_S(EPI_SWIGLU, 1344, mt) != 7;
    bad += pick_S(EPI_SWIGLU, 1376, mt) != (mt == 2 ? 2 : 4) || pick_S(EPI_SWIGLU, 1664, mt) != 4;
  }
  if (bad) printf("gate/up tiles\n");
  for (int mt = 1; mt <= 3; ++mt)   // lm_head: eight strips from 1536 on
    bad += pick_S(EPI_LOGITS, 1536, mt) != 8 || pick_S(EPI_LOGITS, 2000, mt) != 8 || pick_S(EPI_LOGITS, 1024, mt) != 4;
  if (bad) printf("lm_head tiles\n");
  const int kbs[] = {1, 2, 3, 4, 7, 8, 28, 64, 128, 255, 256, 383, 384, 448, 592, 1000, 2048};
  for (int mt = 1; mt <= 4; ++mt)
    for (int kb : kbs) {
      for (int n = 1; n <= 2400; ++n) {
        bad += check("qkv", EPI_QKV, plan_gemm(EPI_QKV, n * 16, kb * 32), mt);
        bad += check("o", EPI_RESID, plan_o(n * 16, kb * 32), mt);
        bad += check("down", EPI_RESID, plan_gemm(EPI_RESID, n * 16, kb * 32), mt);
        if (n % 2 == 0) bad += check("gate/up", EPI_SWIGLU, plan_gemm(EPI_SWIGLU, n * 16, kb * 32), mt);
        bad += check("lm_head", EPI_LOGITS, plan_gemm(EPI_LOGITS, n * 16, kb * 32), mt);
      }
      for (int n = 2402; n <= 20000; n += 34) {
        bad += check("gate/up", EPI_SWIGLU, plan_gemm(EPI_SWIGLU, n * 16, kb * 32), mt);
        bad += check("lm_head", EPI_LOGITS, plan_gemm(EPI_LOGITS, n * 16, kb * 32), mt);
      }
    }
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_every_plan_has_its_kernel_and_chunks_are_even(tmp_path):
    src, exe = tmp_path / "plans.cpp", tmp_path / "plans"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, f"wrong plans:\n{res.stdout[:2000]}"


class _RowsPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("variant", "n_tiles", "m_blocks", "ksplit", "ent_strips", "entries")]


# row tiles, wavefronts and strips per wavefront of gemm_rows.hip's kVariants
ROWS_TILES = [(8, 8, 2), (9, 8, 2), (9, 4, 2), (8, 4, 2), (6, 4, 2)]
ROWS_PART = 18 << 20


@pytest.mark.skipif(not os.path.exists(LIB), reason="libpard.so not built")
def test_row_block_plans_cover_their_weight():
    """Row-block plans over weight shapes and row counts: the tiles cover the
    strips and the row bound once, every input split has k-blocks, the partial
    tiles fit their buffer, and the row pieces fit the row-sum and argmax
    buffers (one per two strips)."""
    plan_rows = ctypes.CDLL(LIB)._ZN4pard9plan_rowsEiiii
    plan_rows.restype, plan_rows.argtypes = _RowsPlan, [ctypes.c_int] * 4
    for n_strips in [*range(1, 40), 64, 96, 128, 160, 192, 256, 288, 384, 512, 608, 640, 768, 960, 1024, 1280, 1792, 2368, 3584, 8016, 9504]:
        for kb in (1, 2, 7, 8, 9, 28, 64, 128, 448, 896):
            for rows, typ in ((65, 65), (96, 80), (144, 144), (288, 288), (512, 100), (517, 517), (2048, 2048), (4096, 4096)):
                p = plan_rows(n_strips, kb, rows, typ)
                where = (n_strips, kb, rows, typ, [getattr(p, f) for f, _ in p._fields_])
                mb, cg, ns = ROWS_TILES[p.variant]
                assert p.n_tiles * cg * ns >= n_strips > (p.n_tiles - 1) * cg * ns, where
                assert p.m_blocks * mb * 16 >= rows > (p.m_blocks - 1) * mb * 16, where
                assert 1 <= p.ksplit <= max(1, kb // 8), where
                assert p.ksplit == 1 or p.ksplit * p.m_blocks * mb * n_strips * 256 <= ROWS_PART, where
                assert p.ent_strips == (4 if p.ksplit > 1 else ns), where
                assert p.entries == -(-n_strips // p.ent_strips) <= -(-n_strips // 2), where
