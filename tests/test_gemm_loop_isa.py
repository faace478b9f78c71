"""The k-loop of the tile kernels keeps the loads of the next k-tiles in flight while it waits for one: the wait before
each barrier counts them.  A wait of the compiler's own for all of them in front of that barrier would cost the latency
these kernels are built to hide, with the same results.  This test compiles the kernel source to gfx950 assembly (no GPU
needed) and checks, for every instantiation, the counts that stand directly in front of the barriers."""
import collections
import os
import re

import pytest

from paper_2603_26498_amd import build as B

SRC = os.path.join(B.CSRC, "gemm_bf16.hip")


def test_the_barriers_of_the_k_loop_wait_for_one_tile_only(tmp_path):
    try:
        hipcc = B._hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    out = str(tmp_path / "gemm.s")
    B._run([hipcc, *B.FLAGS, "-S", "--cuda-device-only", SRC, "-o", out])
    asm = open(out).read()
    seen = collections.Counter()
    # template arguments: tile rows and columns, waves along them, waves that share the k-steps, stages, ...
    for m in re.finditer(r"^(_ZN4tcmv16gemm_bf16_kernelI((?:Li\d+E){8})EEvNS_8GemmArgsE):", asm, re.M):
        bm, bn, wm, wn, kw, stages, _, epi = map(int, re.findall(r"Li(\d+)E", m.group(2)))
        loads = (bm + bn) // 8 // (wm * wn * kw)                   # wave-wide loads of a wave and k-tile
        body = asm[m.end():asm.index(".Lfunc_end", m.end())]
        ins = [x.strip().split(";")[0].strip() for x in body.split("\n") if x.startswith("\t") and not x.startswith(("\t.", "\t;"))]
        counts = collections.Counter()
        for a, b in zip(ins, ins[1:]):
            w = re.match(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$", a)
            if w and b == "s_barrier":
                counts[int(w.group(1))] += 1
        # all stages but the first in flight before the loop; one less in the loop and in the iteration behind it; then fewer
        assert counts[(stages - 1) * loads] == 1, (m.group(1), counts)
        assert all(counts[i * loads] == (2 if i == stages - 2 else 1) for i in range(1, stages - 1)), (m.group(1), counts)
        seen[(bm, bn)] += 1
    assert len(seen) == 6 and all(n >= 6 for n in seen.values()), seen
