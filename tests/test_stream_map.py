"""The memory that the streaming forward GEMM touches, enumerated on the host: its index arithmetic lives in a header without
device types, which is compiled here with the host compiler."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SUMS = r"""
#include <cstdio>
#include <vector>
#include "stream_map.hpp"
using namespace grouter;

// every form of the kernel: NB weight matrices, RB row blocks; 8 waves, 64 columns a workgroup
template <int NB, int RB>
int check() {
    constexpr int W = 8, COLS = kStreamCols;
    using Sums = StreamSums<NB, COLS>;
    for (int rows = 1; rows <= 16 * RB; ++rows)
        for (int cols = 8; cols <= 72; cols += 8) {        // columns from the workgroup's first one to the matrix's end
            const int here = cols < COLS ? cols : COLS;
            std::vector<int> stored(rows * COLS, 0);
            for (int rb = 0; rb < RB && rb * 16 < rows; ++rb)
                for (int tid = 0; tid < W * 64; ++tid) {
                    const Sums s(tid);
                    if (!s.finishes(rows - rb * 16, cols)) continue;
                    for (int w = 0; w < W; ++w)
                        for (int nb = 0; nb < NB; ++nb) {
                            const int at = s.at(w, nb), begin = w * Sums::kWaveBytes;
                            if (at < begin || at + 16 > begin + Sums::kWaveBytes || at % 16)
                                return std::printf("NB %d RB %d rows %d: thread %d reads byte %d of wave %d's area\n", NB, RB, rows, tid, at - begin, w), 1;
                        }
                    for (int c = 0; c < 4; ++c) ++stored[(rb * 16 + s.row) * COLS + s.col + c];
                }
            for (int r = 0; r < rows; ++r)
                for (int c = 0; c < COLS; ++c)
                    if (stored[r * COLS + c] != (c < here ? 1 : 0))
                        return std::printf("NB %d RB %d rows %d cols %d: row %d column %d stored %d times\n", NB, RB, rows, cols, r, c, stored[r * COLS + c]), 1;
        }
    return 0;
}
int main() { return check<1, 1>() | check<1, 2>() | check<1, 4>() | check<2, 1>() | check<2, 2>() | check<2, 4>(); }
"""


def run_host(tmp_path, source):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_06626_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_partial_sums_stay_in_their_area_and_every_output_is_stored_once(tmp_path):
    r = run_host(tmp_path, SUMS)
    assert r.returncode == 0, r.stdout


TILES = r"""
#include <cstdio>
#include <vector>
#include "stream_map.hpp"
using namespace grouter;

int main() {
    for (int bound = 1; bound <= 40; ++bound)              // row tiles the launch allows for
        for (int ncb = 1; ncb <= 20; ++ncb)
            for (const StreamOrder order : {kStreamPlain, kStreamRuns, kStreamByExpert}) {
                const int grid = stream_grid(order, bound, ncb);
                for (int n = -1; n <= bound; ++n) {        // row tiles the plan header names; -1: a plan of other dimensions
                    std::vector<int> taken(bound * ncb, 0);
                    for (int block = 0; block < grid; ++block) {
                        bool vouched = false;
                        int read = -1;
                        StreamTile t;
                        const bool ok = t.pick(block, ncb, order, [&]() { vouched = true; return n; },
                                               [&](int mt) { if (!vouched || mt < 0 || mt >= n) read = -2; else if (read == -1) read = mt; });
                        if (read == -2 || (n < 0 && ok) || (ok && read != t.mt))
                            return std::printf("bound %d, %d column blocks, %d tiles: workgroup %d reads a record nobody vouched for\n", bound, ncb, n, block), 1;
                        if (ok) ++taken[t.mt * ncb + t.cb];
                    }
                    for (int i = 0; i < bound * ncb; ++i)
                        if (taken[i] != (i < n * ncb ? 1 : 0))
                            return std::printf("bound %d, %d column blocks, %d tiles: pair %d taken %d times\n", bound, ncb, n, i, taken[i]), 1;
                }
            }
    return 0;
}
"""


def test_tile_records_are_read_after_the_header_and_every_tile_is_taken_once(tmp_path):
    r = run_host(tmp_path, TILES)
    assert r.returncode == 0, r.stdout
