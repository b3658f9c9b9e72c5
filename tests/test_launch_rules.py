"""The launch rules that follow from sizes alone (csrc/rules.h), over their ranges,
from a host program compiled here."""
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]


def evaluate(tmp_path, expr, calls):
    """expr, a C++ expression in q[0], q[1], ..., for every tuple of calls."""
    src = tmp_path / "rules.cpp"
    src.write_text('#include "rules.h"\n#include <cstdio>\nusing namespace mgdwf;\nint main() {\n'
                   '  long long q[8];\n  while (scanf("%lld %lld %lld %lld", q, q + 1, q + 2, q + 3) == 4)\n'
                   f'    printf("%lld\\n", (long long)({expr}));\n}}\n')
    exe = tmp_path / "rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", str(ROOT / "paper_1205_2933_amd" / "csrc"), str(src), "-o", str(exe)],
                   check=True)
    pad = lambda c: " ".join(str(int(v)) for v in (tuple(c) + (0, 0, 0, 0))[:4])
    out = subprocess.run([str(exe)], input="\n".join(map(pad, calls)), capture_output=True, text=True, check=True)
    return [int(v) for v in out.stdout.split()]


SITES = sorted({1, 2, 9, 16, 32, 48, 85, 86, 96, 108, 127, 128, 129, 144, 162, 170, 171, 192, 240, 255, 256, 257, 512,
                1024, 2592, 4096, 65536})


def test_restriction_splits(tmp_path):
    """Every split has rows of its own beyond the first four, the workspace holds any count,
    and more than four splits stay within two workgroups per CU (eight in FP64)."""
    calls = [(vc, rows, n, f64) for vc in SITES for rows in (1, 80, 96, 255, 256, 1024, 1279, 1280, 1792, 4096, 5775, 65536)
             for n in (1, 2, 3, 12, 300) for f64 in (0, 1)]
    got = evaluate(tmp_path, "restrict_splits_general(q[0], q[1], q[2], q[3])", calls)
    most = evaluate(tmp_path, "restrict_splits(q[0])", calls)
    for (vc, rows, n, f64), s, m in zip(calls, got, most):
        assert 4 <= s <= m <= 16, (vc, rows, n, f64, s, m)
        if s > 4:
            assert s * 256 <= rows and vc * n * s <= (2048 if f64 else 512), (vc, rows, n, f64, s)
    # blocks of few rows keep four (they took up to 3.6 times as long with 16)
    assert set(evaluate(tmp_path, "restrict_splits_general(q[0], q[1], q[2], q[3])",
                        [(16, 80, 12, 0), (256, 256, 1, 1), (256, 96, 1, 0), (16, 128, 1, 1)])) == {4}


def test_ordered_apply_groups(tmp_path):
    """No workgroup without right-hand sides, and where the matrix is too large for the
    caches one pass over it per four right-hand sides at most, or the general kernel (0)."""
    calls = [(vc, n2, n) for vc in SITES for n2 in (16, 32, 48, 64) for n in range(1, 41)]
    for (vc, n2, n), g in zip(calls, evaluate(tmp_path, "sq_ordered_group(q[0], (int)q[1], (int)q[2])", calls)):
        assert 0 <= g <= min(n, 4), (vc, n2, n, g)
        if g:
            groups = -(-n // g)
            assert (groups - 1) * g < n, (vc, n2, n, g)
            if vc >= 256:
                assert groups == -(-n // 4), (vc, n2, n, g)  # one right-hand side is not worked on twice, nor four in two
        if n <= 4:
            assert g or (n, n2) == (1, 64), (vc, n2, n)
        elif vc > 160 and not (n2 == 16 and vc >= 1024):
            assert g == 0, (vc, n2, n)


def test_row_split_rounds(tmp_path):
    """The split form takes at most two rounds of 256 workgroups, and only where the sites
    alone are no full round."""
    calls = [(v, mt, f64, cg) for v in SITES for mt in (2, 3, 4) for f64 in (0, 1) for cg in (0, 1)]
    for (v, mt, f64, cg), split in zip(calls, evaluate(tmp_path, "sq_split_rows(q[0], (int)q[1], q[2], q[3])", calls)):
        rounds = -(-v * mt // 256)
        assert not split or (rounds <= 2 and v < 256), (v, mt, f64, cg)
        assert split or rounds > 1, (v, mt, f64, cg)
    # 162 sites x 64 dof, one right-hand side: 73 us split, 61 with whole sites
    assert evaluate(tmp_path, "sq_split_rows(q[0], (int)q[1], q[2], q[3])", [(162, 4, 1, 0), (162, 4, 0, 0)]) == [0, 0]


def test_coarse_build_memory(tmp_path):
    """Three columns at a time only where their fields leave half of the free memory."""
    field = 12 * 16 * 16 * 4096 * 32  # bytes of an FP64 field on 16^3x32x16
    calls = [(field, free) for free in (0, 9 * field, 27 * field, 53 * field, 54 * field, 10**12)]
    calls += [(16 * 10**9 // 27, 10**12), (16 * 10**9 // 27 + 1, 10**12)]
    assert evaluate(tmp_path, "coarse_build_columns((double)q[0], (double)q[1])", calls) == [1, 1, 1, 1, 3, 3, 3, 1]
