"""Host-side check, without a GPU, of the launches of the long-row kernels: HIP takes fewer than 2^32 threads, graphs may have
some 10^9 edges, and a workgroup of a sliced launch must keep its XCD over the stride of the grid."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r'''
#include <cstdio>
#include "bigrows.h"
int main() {
  ink_ctx c;
  const int64_t nodes[] = {1, 100, 8192, 8193, 2000000, 4000000, (1ll << 30) - 1}, per_node[] = {0, 1, 20, 220, 536};
  for (int64_t n : nodes)
    for (int64_t p : per_node) {
      const int64_t edges = n * p < (1ll << 30) - 1 ? n * p : (1ll << 30) - 1;
      c.n = (int)n; c.n_cap = n; c.n_edges = c.n_edges_now = edges;
      const int64_t every = edges / ink::kBigChunk + (n < edges / ink::kBigDeg ? n : edges / ink::kBigDeg) + 1;
      for (int64_t chunks : {int64_t(0), int64_t(1), every, 2 * every})
        for (int slices = 1; slices <= ink::big_slices(256); slices++)
          for (int latency = 0; latency < 2; latency++)
            printf("%lld %lld %d\n", (long long)chunks, (long long)ink::big_grid(&c, chunks, slices, latency != 0), latency ? 1024 : 256);
    }
}
'''


def run_program(tmp_path, text):
    src, exe = tmp_path / "sizes.cpp", tmp_path / "sizes"
    src.write_text(text)
    subprocess.check_call(["hipcc", "-std=c++17", "-O0", "--offload-arch=gfx950", "-x", "hip", "-I", os.path.join(ROOT, "paper_2309_11071_amd", "csrc"),
                           str(src), "-o", str(exe)], stderr=subprocess.DEVNULL)
    return [tuple(map(int, line.split())) for line in subprocess.check_output([str(exe)], text=True).splitlines()]


def test_grids_of_the_long_row_kernels(tmp_path):
    rows = run_program(tmp_path, PROGRAM)
    assert len(rows) > 1000
    for chunks, groups, threads in rows:
        assert 0 < groups and groups % 8 == 0 and groups * threads < 2 ** 32
        if threads == 1024:                                # a short launch has no workgroup without a chunk for each slice of each chunk
            assert groups <= max(chunks, 1024) + 8
        if chunks == 0:                                    # usually there are none: nothing but an empty launch
            assert groups * threads <= 2 ** 20
    assert max(g for _, g, _ in rows) > 2 ** 19               # the bound does not touch what graphs of usual sizes launch


SEGMENTS = r'''
#include <cstdio>
#include "longev.h"
int main() {
  const int64_t events[] = {262144, 262145, 500000, 1000000, 1100000, 2000000, 8000000, 8388609, 20000000};
  for (int64_t n : events)
    for (int64_t per : {1, 2, 5, 7, 10, 15, 17, 25, 67, 500})
      for (int64_t longest : {500, 700, 2000, 100000}) {
        if (longest < per) continue;
        const ink::LongEvents L = ink::long_events(ink::EventBounds{n, longest}, n / per);
        printf("%lld %lld %lld %d %d\n", (long long)n, (long long)(n / per), (long long)longest, L.limit, L.chunk);
      }
}
'''


def test_limits_of_long_segments(tmp_path):
    """Low limits only where few segments are above them: with many events a target, or none that is long, a list of nearly
    all segments costs more than the chains it cuts."""
    seen = set()
    for events, targets, longest, limit, chunk in run_program(tmp_path, SEGMENTS):
        seen.add((limit, chunk))
        if targets <= 8192:                                   # short launches
            assert (limit, chunk) == (128, 256)
        elif events <= 1 << 18 or events > 1 << 23 or events / targets > 16 or longest <= 700:
            assert (limit, chunk) == (256, 256), (events, targets, longest)
        elif events > 1 << 20 or events / targets > 8.1:
            assert (limit, chunk) == (128, 256), (events, targets, longest)
        else:
            assert (limit, chunk) == (64, 128), (events, targets, longest)
    assert len(seen) == 3


CHUNKS = r'''
#include <cstdio>
#include "longev.h"
int main() {
  for (int64_t n : {0, 64, 65, 129, 257, 513, 100000, 262145, 1000000, 8000000, 20000000})
    for (ink::LongEvents L : {ink::LongEvents{nullptr, nullptr, 64, 128}, ink::LongEvents{nullptr, nullptr, 128, 256}, ink::LongEvents{nullptr, nullptr, 256, 256}})
      printf("%lld %d %d %lld %lld\n", (long long)n, L.limit, L.chunk, (long long)ink::long_ev_rows(L, n), (long long)ink::long_ev_chunks(L, n));
}
'''


def test_room_for_the_chunks_of_long_segments(tmp_path):
    """Room for the chunks of any division of the events into segments, and hardly more: at 8M events and 256 columns a
    chunk too many for every 256 events is a quarter of a gigabyte of partial rows."""
    for n, limit, chunk, rows, chunks in run_program(tmp_path, CHUNKS):
        most_rows, most_chunks = n // (limit + 1), 0
        for s in range(limit + 1, min(n, 4 * chunk) + 1):          # as many segments of s events as there can be, the rest in one more
            rest = n % s
            most_chunks = max(most_chunks, n // s * -(-s // chunk) + (-(-rest // chunk) if rest > limit else 0))
        assert most_rows <= rows <= 1.02 * most_rows + 2
        assert most_chunks <= chunks <= 1.02 * most_chunks + 3, (n, limit, chunk, chunks, most_chunks)


COMBINE = r'''
#include <cstdio>
#include "bigrows.h"
int main() {
  for (int64_t chunks : {0, 1, 200, 366, 782, 1953, 3126, 5859})
    for (int wd : {4, 64, 128, 132, 256})
      for (int sums = 0; sums < 2; sums++) {
        ink::AggArgs a{};
        a.big_chunks = chunks; a.wd = wd;
        printf("%lld %d %d %d\n", (long long)chunks, wd, sums, (int)ink::combine_on_arrival(a, sums != 0));
      }
}
'''


def test_many_parts_of_long_rows_have_a_kernel_that_combines_them(tmp_path):
    for chunks, wd, sums, arrive in run_program(tmp_path, COMBINE):
        assert arrive == (chunks <= (1953 if sums and wd <= 128 else 200)), (chunks, wd, sums)
