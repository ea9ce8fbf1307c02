"""The division of the work (csrc/mosaic_schedule.h), which host and device evaluate alike, on the CPU: every division has
room in the partial arrays, for either of the two kernels that may do a launch's work, and the word through which a
launch tells its division to the ones behind it leads nobody outside, whatever it holds.  Which unit a workgroup begins with:
every unit has one workgroup, and the 8 XCDs, to which workgroups are dealt in turn, have equally many units (to one), also
where the launch has more workgroups than the division has units."""
import os
import subprocess

import pytest

import test_gpu_shared_bounds as shared_bounds
import test_gpu_streamed_head as streamed_head

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_06562_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <stdio.h>
#include "mosaic_internal.h"
#include "mosaic_schedule.h"
using namespace mosaic;
static long bad, divisions, differ;
static void check(bool ok, const char* what, int64_t max_rows, int rows, int d, int V, long budget, int n) {
  if (!ok && ++bad < 10) printf("%s: max_rows %ld rows %d d %d V %d budget %ld: %d\n", what, (long)max_rows, rows, d, V, budget, n);
}
int main() {
  const int shapes[][2] = {{64, 300}, {256, 2500}, {256, 50257}, {4096, 50257}, {4096, 126464}, {3584, 151936}};
  for (auto& shape : shapes) for (int64_t max_rows : {1, 40, 255, 769, 4096, 60000}) for (long budget : {0L, 20000L, 4L << 20})
    for (int sample = 0; sample < 2; ++sample) {
      const int d = shape[0], V = shape[1];
      mosaic_plan plan;
      if (mosaic_plan_workspace(131072, max_rows, d, V, budget, 256, sample, &plan) != MOSAIC_OK) { printf("no plan\n"); return 1; }
      const KernelChoice choice = choose_kernel(131072, d, d, V, plan, sample != 0);
      ScheduleInput in{};
      in.vocab_tiles = (uint32_t)((V + 255) / 256 - (choice.paired ? 1 : 0));
      in.k_tiles = (uint32_t)d / 64;
      in.sampling = (uint32_t)sample;
      in.grid = (uint32_t)plan.grid;
      in.extra = choice.paired ? 1 : 0;
      in.slots64 = (uint32_t)((int64_t)plan.vocab_splits * plan.rows_per_chunk / 64);
      const int64_t slots = (int64_t)plan.vocab_splits * plan.rows_per_chunk;
      const int most = (int)(max_rows < plan.rows_per_chunk ? max_rows : plan.rows_per_chunk);
      for (int rows = 1; rows <= most; rows += 1 + rows / 7) {
        int splits[2];
        for (int general = 0; general < 2; ++general) {
          in.widths = general ? 0x80 : 0xff;
          const Schedule s = choose_schedule(in, rows);
          ++divisions;
          splits[general] = s.splits;
          check(s.splits >= 1 && s.splits <= (int)in.vocab_tiles && s.stride == partial_stride(rows) &&
                    (int64_t)s.row_tiles * 32 * s.width >= rows && (general == 0 || s.width == 8) &&
                    ((int64_t)s.splits + in.extra) * s.stride <= slots, "division", max_rows, rows, d, V, budget, s.splits);
          check(held_splits(in, rows, s.splits) == s.splits, "a division is not taken over", max_rows, rows, d, V, budget, s.splits);
        }
        differ += splits[0] != splits[1];
        for (int found : {-2147483647 - 1, -7, 0, 1, 2, 3, 255, 256, 257, 4096, 1 << 20, 2147483647}) {
          const int held = held_splits(in, rows, found);
          check(held >= 1 && ((int64_t)held + in.extra) * partial_stride(rows) <= slots, "outside", max_rows, rows, d, V, budget, found);
        }
      }
    }
  printf("%ld divisions, %ld bad, %ld rows on which the two kernels' differ\n", divisions, bad, differ);
  return bad != 0;
}
"""


PLACES = r"""
#include <stdio.h>
#include <vector>
#include "mosaic_internal.h"
#include "mosaic_schedule.h"
using namespace mosaic;
int main() {
  long launches = 0, surplus = 0, bad = 0;
  auto check = [&](int grid, int units, int V, int rows) {
    std::vector<int> taken(units < grid ? units : grid), xcd(8);
    bool ok = true;
    for (int b = 0; b < grid; ++b) {
      const int u = first_unit(b, grid, units);
      if (u < units) ok = ok && u >= 0 && u < (int)taken.size() && ++taken[u] == 1, ++xcd[b % 8];
    }
    int least = grid, most = 0;
    for (int n : xcd) least = n < least ? n : least, most = n > most ? n : most;
    for (int n : taken) ok = ok && n == 1;
    ++launches, surplus += grid > units;
    if (!(ok && most - least <= 1) && ++bad < 10)
      printf("V %d rows %d: %d units on %d workgroups, %d to %d an XCD\n", V, rows, units, grid, least, most);
  };
  for (int grid : {1, 7, 8, 9, 64, 100, 255, 256, 304}) for (int units = 1; units <= 320; ++units) check(grid, units, 0, 0);
  const int shapes[][2] = {{512, 8192}, {1024, 32000}, {3584, 151936}, {3584, 152064}, {4096, 126464}};
  for (auto& shape : shapes) for (int max_rows : {32, 100, 256, 700}) for (int sample = 0; sample < 2; ++sample) {
    mosaic_plan plan;
    if (mosaic_plan_workspace(4096, max_rows, shape[0], shape[1], 0, 256, sample, &plan) != MOSAIC_OK) return 1;
    ScheduleInput in{};
    in.vocab_tiles = (uint32_t)(shape[1] + 255) / 256;
    in.k_tiles = (uint32_t)shape[0] / 64;
    in.sampling = (uint32_t)sample;
    in.grid = (uint32_t)plan.grid;
    in.slots64 = (uint32_t)((int64_t)plan.vocab_splits * plan.rows_per_chunk / 64);
    for (uint32_t widths : {0xffu, 0x80u}) for (int rows = 1; rows <= max_rows; ++rows) {
      in.widths = widths;
      const Schedule s = choose_schedule(in, rows);
      check(plan.grid, s.row_tiles * s.splits, shape[1], rows);
    }
  }
  printf("%ld launches, %ld with more workgroups than units, %ld bad\n", launches, surplus, bad);
  return bad != 0 || surplus == 0;
}
"""

LONE = r"""
#include <stdio.h>
#include <stdlib.h>
#include "mosaic_internal.h"
#include "mosaic_schedule.h"
using namespace mosaic;
int main(int argc, char** argv) {
  for (int a = 1; a + 3 < argc; a += 4) {
    const int d = atoi(argv[a]), V = atoi(argv[a + 1]), rows = atoi(argv[a + 2]), sample = atoi(argv[a + 3]);
    mosaic_plan plan;
    if (mosaic_plan_workspace(rows, rows, d, V, 0, 256, sample, &plan) != MOSAIC_OK) return 1;
    if (!choose_kernel(rows, d, d, V, plan, sample != 0).fast) return 1;
    ScheduleInput in{};
    in.vocab_tiles = (uint32_t)(V + 255) / 256;
    in.k_tiles = (uint32_t)d / 64;
    in.widths = 0xff;
    in.sampling = (uint32_t)sample;
    in.grid = (uint32_t)plan.grid;
    in.slots64 = (uint32_t)((int64_t)plan.vocab_splits * plan.rows_per_chunk / 64);
    const Schedule s = choose_schedule(in, rows);
    printf("%d %d\n", s.width, s.row_tiles);
  }
}
"""

SHARES = r"""
#include <stdio.h>
#include <stdlib.h>
#include "mosaic_internal.h"
#include "mosaic_schedule.h"
using namespace mosaic;
int main(int argc, char** argv) {
  for (int a = 1; a + 4 < argc; a += 5) {
    const int d = atoi(argv[a]), V = atoi(argv[a + 1]), bound = atoi(argv[a + 2]), found = atoi(argv[a + 3]);
    mosaic_plan plan;
    if (mosaic_plan_workspace(131072, bound, d, V, atol(argv[a + 4]), 256, 1, &plan) != MOSAIC_OK) return 1;
    const int rows = found < plan.rows_per_chunk ? found : plan.rows_per_chunk;
    const KernelChoice choice = choose_kernel(131072, d, d, V, plan, true);
    if (!choice.fast && !choice.paired) return 1;
    ScheduleInput in{};
    in.vocab_tiles = (uint32_t)((V + 255) / 256 - (choice.paired ? 1 : 0));
    in.k_tiles = (uint32_t)d / 64;
    in.widths = 0xff;
    in.sampling = 1;
    in.grid = (uint32_t)plan.grid;
    in.extra = choice.paired ? 1 : 0;
    in.slots64 = (uint32_t)((int64_t)plan.vocab_splits * plan.rows_per_chunk / 64);
    const Schedule s = choose_schedule(in, rows);
    printf("%d %d %d %d %d\n", s.width, (int)ceil_div(in.vocab_tiles, (uint32_t)s.splits),
           (int)ceil_div((uint32_t)(s.row_tiles * s.splits), in.grid), (int)units_share(in.vocab_tiles, s.width, s.splits),
           plan.num_chunks);
  }
}
"""


def build_and_run(tmp_path, program, *args):
    src = tmp_path / "schedule.hip"
    src.write_text(program)
    exe = str(tmp_path / "schedule")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-o",
                    exe, str(src), os.path.join(CSRC, "mosaic_plan.cpp")], check=True, stderr=subprocess.DEVNULL)
    res = subprocess.run([exe, *map(str, args)], stdout=subprocess.PIPE, text=True, timeout=120)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
    return res.stdout


def divisions_found(tmp_path, draws):
    """(width, tiles of the longest unit, rounds, whether units share, chunks), of the first chunk, of draws given as (d, V,
    bound, rows found, budget)"""
    out = build_and_run(tmp_path, SHARES, *[x for draw in draws for x in draw])
    found = [tuple(int(x) for x in line.split()) for line in out.split("\n") if line]
    assert len(found) == len(draws)
    return found


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_sharing_follows_the_rows_found(tmp_path):
    """whatever the bound: a draw shares where its units, as found, have a second tile (a third where they are narrow)"""
    heads = [(512, 8192), (1024, 32000), (2048, 65536), (3584, 152064), (3584, 151936), (4096, 126464), (512, 8130)]
    draws = [(d, V, bound, rows, 0) for d, V in heads for bound in (512, 4096, 16384)
             for rows in (1, 16, 20, 64, 65, 200, 300, 512, 1000, 4096, 9000) if rows <= bound]
    found = divisions_found(tmp_path, draws)
    for draw, (width, tiles, _, shares, _) in zip(draws, found):
        assert shares == (tiles > (1 if width >= 2 else 2)), draw
    at = {draw[:4]: f for draw, f in zip(draws, found)}
    for bound in (512, 4096, 16384):
        for rows in (16, 20, 64, 200):
            assert not at[512, 8192, bound, rows][3] and not at[1024, 32000, bound, rows][3] and not at[2048, 65536, bound, rows][3]
        assert not at[4096, 126464, bound, 20][3] and at[4096, 126464, bound, 200][3] and at[4096, 126464, bound, 300][3]
    assert all(at[d, V, 16384, 9000][3] for d, V in heads)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_the_draws_that_hold_shared_bounds_do_share(tmp_path):
    """of tests/test_gpu_shared_bounds.py and test_gpu_non_finite.py, and what those are held against does not; one round and
    several; in chunks"""
    for draw, (_, _, rounds, share, chunks) in zip(shared_bounds.SHARING, divisions_found(tmp_path, shared_bounds.SHARING)):
        assert share == 1, draw
        assert (rounds > 1) == (draw[3] > 16384) and (chunks > 1) == (draw[4] > 0), (draw, rounds, chunks)
    for draw, (_, _, _, share, _) in zip(shared_bounds.ALONE, divisions_found(tmp_path, shared_bounds.ALONE)):
        assert share == 0, draw


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_units_are_spread_over_the_xcds(tmp_path):
    build_and_run(tmp_path, PLACES)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_divisions_have_room_and_a_foreign_word_leads_nowhere(tmp_path):
    out = build_and_run(tmp_path, PROGRAM)
    assert int(out.split(" bad, ")[1].split()[0]) > 0             # else the two kernels are not told apart here


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_the_streamed_steps_are_lone_row_tiles_of_every_width(tmp_path):
    """of tests/test_gpu_streamed_head.py: the nt copies are a lone row tile's, in code of its own per width and draw"""
    steps = [(d, V, rows, drawn) for (d, V), counts in streamed_head.STEPS.items() for drawn in (0, 1) for rows in counts[drawn]]
    out = build_and_run(tmp_path, LONE, *[x for step in steps for x in step]).split("\n")
    found = [tuple(int(x) for x in line.split()) for line in out if line]
    assert len(found) == len(steps)
    shared = [s for s, f in zip(steps, found) if f[1] != 1]
    assert all(d == 1024 and drawn and rows > 224 for d, _, rows, drawn in shared), shared
    for ragged in (False, True):
        for drawn in (0, 1):
            widths = {f[0] for s, f in zip(steps, found) if f[1] == 1 and s[3] == drawn and (s[1] % 256 != 0) == ragged}
            assert widths == set(range(1, 9)), (ragged, drawn, widths)
    several = build_and_run(tmp_path, LONE, *[x for (d, V) in streamed_head.STEPS for drawn in (0, 1)
                                              for x in (d, V, streamed_head.T, drawn)]).split("\n")
    assert all(int(line.split()[1]) > 1 for line in several if line)     # what they are held against
