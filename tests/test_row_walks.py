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


@pytest.mark.parametrize("beg,end", [(2**31 - 66, 2**31 - 1), (2**31 - 65, 2**31 - 1), (2**31 - 2, 2**31 - 1), (5, 200)])
def test_wave_takes_each_entry_once(tmp_path, beg, end):
    """The gathers of a row by a wave: lane l at base + l, 64 entries a round."""
    (row,) = run_cpp(tmp_path, f"""
  long long n = 0, sum = 0, cnt = 0;
  int rounds = 0;
  HG_ROW_WALK(base, {beg}, {end}, 64) {{
    cnt += wave_entries(base, {end});
    for (int l = 0; l < 64; ++l) {{
      const row_pos pos = base + l;
      if (pos < (row_pos){end}) {{
        ++n;
        sum += pos;
      }}
    }}
    if (++rounds > 9) break;
  }}
  printf("%lld %lld %lld\\n", n, sum, cnt);""")
    assert row == [end - beg, (beg + end - 1) * (end - beg) // 2, end - beg]


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


LENGTHS = [0, 1, 23, 24, 47, 48, 64, 65, 256, 257, 1_024, 1_025, 2_048, 2_049, 32_768, 33_280, 100_003, 524_288,
           600_001, 2**31 - 131_072, 2**31 - 2_049, 2**31 - 1_024, 2**31 - 1]


@pytest.mark.parametrize("edges,nodes", [(10**5, 10**4), (2**31 - 1, 10**4), (2**31 - 1, 10**6), (2**31 - 1, 2**31 - 2)])
def test_pieces_cover_long_rows(tmp_path, edges, nodes):
    """A row's pieces per block and the chunks of a destination row, up to the longest row, and the row
    covered once by pieces of at most a chunk."""
    body = f"const PlanCut k = plan_cut({edges}, {nodes});\n"
    body += 'printf("%d %d %d\\n", k.chunk, k.blocks, k.whole);\n'
    for n in LENGTHS:
        body += f"""{{ const int m = cuts_of({n}, k), p = m * k.blocks;
  int at = 0, most = 0, holes = 0;
  for (int c = 0; c < p; ++c) {{
    const RowRange r = row_piece(0, {n}, c, p);
    holes += r.beg != at || r.end <= r.beg;
    at = r.end;
    most = r.end - r.beg > most ? r.end - r.beg : most;
  }}
  printf("%d %d %d %d %d\\n", m, fwd_chunks_of({n}), at, most, holes); }}
"""
    (chunk, blocks, whole), *rows = run_cpp(tmp_path, body)
    for n, (m, fwd, at, most, holes) in zip(LENGTHS, rows):
        size = max(chunk, min(1_024, n // 512))  # a row of more than 512 chunks takes longer ones
        assert m == (-(-n // (size * blocks)) if n > whole else 0), n
        assert fwd == (-(-n // 2_048) if n > 2_048 else 0), n
        assert (at, holes) == (n if m else 0, 0) and most <= size, n
