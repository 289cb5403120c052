"""The rules of the windowed sweeps (window_rules.hpp), compiled for the CPU and run through every small case:
which arrivals a set's windows read, which buffer of admitted sums is free to be cleared, in how many ticks nothing
completes, the longest windows that a wavefront with the instances in its lanes takes, and which shapes are laid out."""
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


def lays_out(tmp_path, sweeps=(), assigns=(), sums=()):
    """What the rules say of (units, sets, slots, requests of a window, windows, shortest queue), (slots, requests of a window, windows,
    shortest queue) and (slots, requests of a window, windows)."""
    body = ""
    for name, rows in (("sweep_lays_out", sweeps), ("assign_lays_out", assigns), ("sweep_sums_batches", sums)):
        for r in rows:
            args = ", ".join(str(int(x)) for x in r)
            body += f'  printf("%d\\n", (int){name}({args}));\n'
    return [row[0] for row in run_rules(tmp_path, body)]


def test_shapes_that_were_measured_slower_are_not_laid_out(tmp_path):
    """Few windows do not earn the launches, and a distributor's single block is slow where many different instances admit; the shapes that
    were measured several times as fast stay laid out."""
    slow_sweeps = [(64, 1, 4, 4096, 1, 0), (64, 1, 64, 4096, 2, 0), (1024, 1, 64, 512, 1, 0), (911, 1, 41, 517, 1, 0), (4096, 1, 4, 512, 2, 0),
                   (8192, 1, 64, 256, 1, 0), (512, 1, 64, 2048, 2, 0), (558, 3, 16, 4096, 16, 0), (1134, 3, 32, 4096, 4, 0), (1000, 1, 4, 4096, 1, 0),
                   (300, 1, 4, 65_536, 1, 0), (500, 1, 16, 16_000, 1, 0), (500, 1, 3, 16_000, 3, 0),
                   (1080, 3, 32, 257, 4, 0)]
    slow_assigns = [(256, 8192, 64, 0), (16, 11, 64, 1), (256, 20, 64, 1), (13, 13_263, 14, 0), (64, 16_384, 32, 0), (43, 10_639, 17, 0),
                    (17, 29, 58, 1), (35, 26, 42, 1), (64, 32_768, 64, 0)]
    slow_sums = [(64, 2048, 4), (256, 2048, 1), (4, 2048, 64), (64, 4096, 2), (64, 300, 1000)]
    assert lays_out(tmp_path, slow_sweeps, slow_assigns, slow_sums) == [0] * (len(slow_sweeps) + len(slow_assigns) + len(slow_sums))
    fast_sweeps = [(8192, 1, 128, 4096, 32, 0), (2160, 3, 64, 256, 512, 0), (4096, 1, 64, 4096, 1, 0), (1024, 1, 64, 16_384, 8, 0),
                   (512, 1, 64, 4096, 16, 0), (1024, 1, 64, 4096, 1, 1), (4096, 1, 256, 2048, 1, 0), (64, 1, 64, 16_384, 4, 0),
                   (1080, 3, 32, 257, 11, 0), (1620, 3, 48, 400, 7, 0),
                   (105, 1, 35, 10_637, 10, 0), (1125, 1, 113, 1333, 4, 0), (2020, 1, 6, 7847, 1, 0), (1626, 1, 123, 1459, 1, 0), (1278, 3, 39, 645, 14, 0)]
    fast_assigns = [(64, 4096, 1024, 0), (8, 512, 1024, 1), (2, 11, 1, 0), (16, 2048, 256, 0), (128, 8192, 512, 0), (256, 4096, 64, 1),
                    (64, 1024, 64, 1), (4, 4096, 1, 0), (64, 16_384, 256, 0),
                    (24, 14_162, 110, 0), (55, 23, 958, 1), (91, 1160, 1, 1), (61, 4187, 1, 0), (31, 14_911, 39, 1)]
    fast_sums = [(128, 4096, 32), (64, 2048, 16), (4, 16_384, 4), (64, 16_384, 1)]
    assert lays_out(tmp_path, fast_sweeps, fast_assigns, fast_sums) == [1] * (len(fast_sweeps) + len(fast_assigns) + len(fast_sums))


def test_longer_streams_stay_laid_out(tmp_path):
    """With more windows of one length the sweep gains, so no shape leaves the form again, and nor does a distributor's beyond four windows."""
    rows = run_rules(tmp_path, """
  const uint32_t units[] = {64, 400, 720, 1000, 2160, 4096, 9000}, lengths[] = {11, 48, 64, 128, 256, 300, 512, 1024, 2048, 4096, 8192, 16384, 65536};
  int left = 0, laid = 0;
  for (uint32_t sq = 0; sq < 2; ++sq)
    for (uint32_t i = 1; i <= 256; ++i)
      for (uint32_t w : lengths) {
        bool a = false;
        for (uint32_t n = 8; n <= 1024; n *= 2) { const bool b = assign_lays_out(i, w, n, sq); left += a && !b; laid += b; a = b; }
        for (uint32_t u : units)
          for (uint32_t sets = 1; sets <= 3; sets += 2) {
            a = false;
            for (uint32_t n = 1; n <= 1024; n *= 2) { const bool b = sweep_lays_out(u, sets, i, w, n, sq); left += a && !b; laid += b; a = b; }
          }
      }
  printf("%d %d\\n", left, laid);""")
    assert rows[0][0] == 0 and rows[0][1] > 10000


def test_shapes_of_the_laid_out_tests_are_laid_out(tmp_path):
    from tests import test_gpu_ordered_windows as T
    windows = lambda n_req, window: (min(window, n_req), -(-n_req // window))
    sweeps = [(c, 1, i, *windows(r, w), sq) for c, i, _, w, r, _, _ in T.SWEEPS for sq in (0, 1) if c >= 400 or not sq]
    assigns = [(i, *windows(r, w), p) for i, _, w, r, p, _ in T.DISTRIBUTORS] + [(i, *windows(r, w), p) for i, w, r, p in T.FLAGGED]
    got = lays_out(tmp_path, sweeps, assigns)
    assert all(got), [x for x, ok in zip(sweeps + assigns, got) if not ok]
    tables = [(i, *windows(r, w)) for _, i, _, w, r, _, _ in T.SWEEPS]
    assert 5 <= sum(lays_out(tmp_path, sums=tables)) <= len(tables) - 10
