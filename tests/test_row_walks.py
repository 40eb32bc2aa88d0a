"""The index arithmetic of walks over rows (csrc/hg_rows.h), on the host at
positions up to 2^31 - 1: more entries than a test builds a graph of."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")


def run_cpp(tmp_path, body):
    """Compiles and runs a program with `body` in main; its output lines as lists of ints."""
    src = tmp_path / "t.cpp"
    src.write_text('#include "hg_rows.h"\n#include <cstdio>\nusing namespace hg;\nint main() {\n' + body + "\n}\n")
    exe = tmp_path / "t"
    subprocess.run([CXX, "-std=c++17", "-O1", "-fwrapv", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2608_02168_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


pytestmark = pytest.mark.skipif(CXX is None, reason="no host compiler")

# strides of the kernels' walks: 4 x 1024 neighbours, a block's and a wave's width
WALKS = [(beg, end, step) for step in (4096, 256, 64) for end in (2**31 - 1, 2**31 - 64, 2**31 - 4096, 5000)
         for beg in (end - 1, end - step, end - step - 1, end - 3 * step, end) if 0 <= beg]


def test_walks_end(tmp_path):
    body = "".join(f"{{ int n = 0; row_pos last = 0; HG_ROW_WALK(p, {b}, {e}, {s}) {{ last = p; if (++n > 8) break; }}"
                   f' printf("%d %u\\n", n, (unsigned)last); }}\n' for b, e, s in WALKS)
    for (b, e, s), (n, last) in zip(WALKS, run_cpp(tmp_path, body)):
        steps = list(range(b, e, s))
        assert (n, last) == (len(steps), steps[-1] if steps else 0), (b, e, s)


@pytest.mark.parametrize("lo,hi", [(2**31 - 1 - 65, 2**31 - 1), (2**31 - 1 - 16_384, 2**31 - 1),
                                   (2**31 - 1 - 40_000, 2**31 - 1), (2**31 - 300, 2**31 - 1), (7, 7 + 16_385)])
def test_gap_rows_written_once(tmp_path, lo, hi):
    """The threads of the blocks that fill a gap write each of its rows once and no other."""
    (row,) = run_cpp(tmp_path, f"""
  long long n = 0, sum = 0, out = 0;
  for (int i = 0; i < gap_pieces({lo}, {hi}); ++i) {{
    const RowRange g = gap_piece({lo}, {hi}, i);
    for (unsigned t = 0; t < 256; ++t) {{
      HG_ROW_WALK(q, g.beg + t, g.end, 256) {{
        if ((long long)(int32_t)q < {lo} || (long long)(int32_t)q >= {hi}) {{ ++out; break; }}
        ++n;
        sum += q;
      }}
    }}
  }}
  printf("%lld %lld %lld\\n", n, sum, out);""")
    assert row == [hi - lo, (lo + hi - 1) * (hi - lo) // 2, 0]
