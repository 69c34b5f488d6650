"""Slots of a workgroup's tile beyond the last product of a batch have empty
operands, but a masked load still reads one limb: at an operand of the tile's
first product and not at the start of the caller's arrays, which a batch whose
offsets begin further up does not own.  The descriptor code itself, compiled for
the host."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_11621_amd", "csrc")

PROGRAM = r"""
#include "common.hpp"
#include <cstdio>
static int check(const DescView& dv, uint64_t nmul, uint64_t per) {
  for (uint64_t first = 0; first < nmul; first += per)
    for (uint64_t i = first; i < first + per; i++) {
      const MulDesc d = dv.slot(i, first, nmul), o = dv.get(i < nmul ? i : first);
      if (d.a_off != o.a_off || d.b_off != o.b_off || d.c_off != o.c_off || d.r_off != o.r_off) return 1;
      if (i < nmul ? d.la != o.la || d.lb != o.lb : d.la || d.lb) return 2;
    }
  return 0;
}
int main() {
  for (uint64_t nmul = 1; nmul <= CAT_INLINE_DESC; nmul++)
    for (uint64_t per = 1; per <= 64; per *= 2) {
      static MulDesc tab[CAT_INLINE_DESC];
      DescView in{}, tb{}, tr{}, un{};
      in.ninl = (uint32_t)nmul;
      tb.table = tab;
      for (uint64_t i = 0; i < nmul; i++)
        in.inl[i] = tab[i] = MulDesc{1000 + 300 * i, 9000 + 200 * i, 70 * i, 7 * i, (uint32_t)(200 + i), (uint32_t)(130 + i)};
      tr.tree.ngroups = 1;
      tr.tree.j = 3;
      tr.tree.base[0] = 4096;
      tr.tree.K[0] = 16 * nmul - 3;
      tr.tree.mpref[1] = nmul;
      un.uni = 1;
      un.u = UniDesc{512, 96, 64, 48, 48, 40, (uint32_t)nmul - 1, ~0u};
      const DescView* all[] = {&in, &tb, &tr, &un};
      for (int k = 0; k < 4; k++)
        if (const int r = check(*all[k], nmul, per)) {
          printf("form %d, %d products in tiles of %d: %d\n", k, (int)nmul, (int)per, r);
          return 1;
        }
    }
  return 0;
}
"""


def test_slots_without_a_product(tmp_path):
    from paper_2601_11621_amd import build

    src, exe = tmp_path / "slots.hip", tmp_path / "slots"
    src.write_text(PROGRAM)
    subprocess.check_call([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", CSRC, str(src), "-o",
                           str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_kernels_take_their_slots_from_there():
    """No kernel fills a slot with a descriptor of its own (offset zero)."""
    text = open(os.path.join(CSRC, "fntt.hip")).read()
    assert not re.search(r"MulDesc\s+\w+\s*(\{\s*\}|=\s*\{\s*\})", text)
    assert len(re.findall(r"dv\.slot\(", text)) == 3


@pytest.mark.gpu
@pytest.mark.parametrize("la,lb,count", [(200, 150, 3), (777, 301, 5), (2000, 2000, 1), (3000, 100, 7), (9000, 4000, 2)])
def test_offsets_that_begin_further_up(la, lb, count):
    import numpy as np
    import torch

    import paper_2601_11621_amd as cat

    cat.init(0)
    rng = np.random.default_rng(la)
    a, b = (rng.integers(0, 2**32, 5000 + n * count, dtype=np.uint64).astype(np.uint32) for n in (la, lb))
    a_off, b_off = (5000 + n * np.arange(count + 1, dtype=np.uint64) for n in (la, lb))
    print("slots", la, lb, count, flush=True)
    for mode in ("batched", "plain"):
        c, c_off = cat.mul_batched(cat.from_numpy(a), a_off, cat.from_numpy(b), b_off, mode=mode)
        c = cat.to_numpy(c)
        for i in range(count):
            x, y, z = (int.from_bytes(v[int(o[i]):int(o[i]) + n].tobytes(), "little")
                       for v, o, n in ((a, a_off, la), (b, b_off, lb), (c, c_off, la + lb)))
            assert x * y == z, (mode, i)
    torch.cuda.synchronize()
