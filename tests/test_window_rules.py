"""The rules of the windowed sweeps (window_rules.hpp), compiled for the CPU and run through every small case:
which arrivals a set's windows read, which buffer of admitted sums is free to be cleared, in how many ticks nothing
completes, and the longest windows that a wavefront with the instances in its lanes takes."""
import shutil
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2509_06362_amd" / "csrc"


def run_rules(tmp_path, body):
    """Compiles `body` behind the header and returns the integers it prints."""
    if shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "window_rules.hpp"\nusing namespace maaso;\n'
                   "int main() {\n" + body + "\n  return 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


def test_arrivals_are_read_between_windows_only(tmp_path):
    """A set that is one window (a static score) may come without arrivals: none is read.  With more
    windows every request that a window can end at has the arrival behind it, and none past the set."""
    rows = run_rules(tmp_path, """
  for (uint32_t n = 0; n <= 70; ++n)
    for (uint32_t w = 1; w <= 72; ++w)
      for (uint32_t r = 0; r < 130; ++r)
        if (reads_arrival_behind(r, n, w)) printf("%u %u %u\\n", n, w, r);
  const uint32_t most = 1u << 31;
  if (reads_arrival_behind(most - 1u, most, 1u) || !reads_arrival_behind(most - 2u, most, 1u)) printf("0 0 0\\n");""")
    read = {tuple(row) for row in rows}
    expected = {(n, w, r) for n in range(71) for w in range(1, 73) if w < n for r in range(n - 1)}
    assert read == expected


def test_sum_buffers_are_cleared_while_nobody_uses_them(tmp_path):
    """Wavefronts that share a candidate meet at one barrier per window and are otherwise in any order, so
    in the interval that ends at window w's barrier anyone may be reading the sums of window w - 1, adding
    to those of window w or clearing.  No two of these touch one buffer, and a buffer that is added to has
    been cleared, in an earlier interval, since it was last read."""
    rows = run_rules(tmp_path, """
  for (uint32_t w = 0, buf = 0; w < 40; ++w, buf = next_sum_buffer(buf))
    printf("%u %u\\n", buf, cleared_sum_buffer(buf));
  printf("%u %u\\n", kSumBuffers, kSumBuffers);""")
    n = rows.pop()[0]
    clean = {b: True for b in range(n)}       # as the kernel starts
    for w, (added, cleared) in enumerate(rows):
        used = [added, cleared] + ([rows[w - 1][0]] if w else [])
        assert len(set(used)) == len(used), f"window {w}: {used}"
        assert all(0 <= b < n for b in used)
        assert clean[added], f"window {w} adds to what an earlier one left"
        clean[added] = False                  # read behind this interval's barrier
        clean[cleared] = True


def test_nothing_completes_in_safe_ticks(tmp_path):
    """One tick less than row_safe_ticks: the binary32 comparison that the windowed kernels make says that nothing
    completes, over service times, batch rows and window lengths of all sizes; and the bound is not idle: within
    1 % of the exact one where it is above some thousand ticks."""
    rows = run_rules(tmp_path, """
  uint64_t seed = 88172645463325252ull;
  auto next = [&]() { seed ^= seed << 13; seed ^= seed >> 7; seed ^= seed << 17; return seed; };
  auto unit = [&]() { return (float)(next() >> 40) * 0x1p-24f; };
  int wrong = 0, loose = 0, tight = 0;
  for (int k = 0; k < 2000000; ++k) {
    const float s_bar = __builtin_exp2f(unit() * 24.0f - 2.0f), tbt = __builtin_exp2f(unit() * 16.0f - 14.0f);
    const uint32_t w = 1u + (uint32_t)(next() % (k % 2 ? 300u : 65535u)), window = 1u + (uint32_t)(next() % 24u);
    const float pen = k % 3 ? 1.0f : 1.0f + unit();
    const uint32_t safe = row_safe_ticks(s_bar, tbt, w, window);
    if (safe == 0u) continue;
    const int run = (int)(w - 1u + window);
    const float svc = s_bar * (tbt * pen);
    const float served = (float)run * ((float)(safe - 1u) * 0x1p-20f);
    wrong += !(served < svc);
    const double exact = (double)s_bar * tbt / run * 1048576.0;
    if (exact > 4000.0 && exact < 3.9e9) { ++tight; loose += (double)safe < 0.99 * exact; }
  }
  printf("%d %d %d\\n", wrong, loose, tight);
  printf("%u %u %u\\n", row_safe_ticks(1e30f, 1e30f, 1u, 1u), row_safe_ticks(1e-30f, 1e-20f, 1u, 1u), row_safe_ticks(1.0f, 1.0f, 1u, 1u));""")
    assert rows[0][0] == 0 and rows[0][1] == 0 and rows[0][2] > 100000
    assert rows[1] == [4000000000, 0, 1048576 - 1024]


def test_longest_short_windows(tmp_path):
    """The general form, which runs where queues do not fit 32 bits, is slower per request: its windows are never longer
    than the 32-bit form's, never where it was measured slower than the kernel it would replace by 10 % and more, and a window of
    one request is always short."""
    rows = run_rules(tmp_path, """
  for (uint32_t i = 1; i <= 256; ++i)
    printf("%u %u %u %u %u %u %u\\n", i, sweep_short_window(i, false, true), sweep_short_window(i, false, false),
           sweep_short_window(i, true, true), sweep_short_window(i, true, false), assign_short_window(i, true),
           assign_short_window(i, false));""")
    slower = {4: 8, 8: 11, 16: 15, 24: 16, 32: 18, 40: 20, 64: 20, 100: 24, 128: 24, 136: 24, 200: 28, 256: 28}  # windows, sweep
    assert [r[0] for r in rows] == list(range(1, 257))
    for i, sweep, sweep_general, score, score_general, assign, assign_general in rows:
        assert 1 <= sweep_general <= sweep and 1 <= score_general <= score <= sweep and 1 <= assign_general <= assign
        if i in slower:
            assert sweep_general < slower[i] and score_general < slower[i]
        assert assign_general < (9 if i <= 64 else 7 if i <= 128 else 6)
