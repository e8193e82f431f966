"""Launch order and routes of the compute kernels (host arithmetic, no GPU): programs built from the kernels' own header count what
each of the eight XCDs is given, and say which way a product goes."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "fs_tile.h"

// Blocks with vectors per XCD, most loaded one; position t of the launch order holds item t, the first `full` of which hold vectors.
template <int WPB>
int most(const fs_format &f, int full, bool &permutation)
{
    const fs_launch_geometry g = fs_launch_geometry_for(&f, WPB);
    int of_xcd[8] = {0}, *seen = (int *)calloc((size_t)g.nbx * WPB, sizeof(int));
    for (int bx = 0; bx < g.nbx; bx++) {
        const int t = fs_launch_turn<WPB>(bx, g.slice, g.n_swz);
        for (int w = 0; w < WPB; w++) {
            if (t + w < 0 || t + w >= g.nbx * WPB) { permutation = false; continue; }
            seen[t + w]++;
            if (t + w < full) of_xcd[bx % 8]++;
        }
    }
    for (int t = 0; t < g.nbx * WPB; t++) permutation = permutation && seen[t] == 1;
    free(seen);
    int m = 0;
    for (int x = 0; x < 8; x++) m = of_xcd[x] > m ? of_xcd[x] : m;
    return m;
}

int main(int argc, char **argv)
{
    fs_format f{};
    f.M = atoi(argv[1]); f.n_items = atoi(argv[2]); f.n_cut_items = atoi(argv[3]); f.V = 8;
    f.W = f.n_blocks = (f.M + 7) / 8;  // every window one block
    if (f.n_cut_items) f.n_blocks += 40 * f.n_cut_items;
    const int full = atoi(argv[4]);
    bool ok = true;
    const int m1 = most<1>(f, full, ok), m2 = most<2>(f, full, ok), m4 = most<4>(f, full, ok);
    printf("%d %d %d %d\n", ok, m1, m2, m4);
}
"""


ROUTES = r"""
#include <cstdio>
#include "fs_tile.h"

// The work lists that a caller's chunk makes (parts of T blocks, whole windows by min(T, 4)): the rules ask for their items as they are.
int main()
{
    long seen = 0, wrong = 0;
    for (int T = 1; T <= 32; T++)
        for (long blocks = 1; blocks < 300000; blocks += 1 + blocks / 37) {
            if (blocks < 8192 && T == fs_short_part_blocks(blocks)) continue;  // what the conversion makes by itself
            const int Ts = T < 4 ? T : 4;
            for (long items : {(blocks + Ts - 1) / Ts, (blocks + Ts - 1) / Ts * 3 / 4, (blocks + T - 1) / T})
                for (long cut : {0L, items / 9, items / 8 + 1, items / 2 + 1, items * 3 / 4 + 1, items})
                    for (long d : {8L, 32L, 40L, 128L}) {
                        fs_format f{};
                        f.V = 8; f.KB = 32; f.chunk = T * 32; f.K = 200000;
                        f.n_blocks = blocks; f.n_items = items; f.n_cut_items = cut < items ? cut : items;
                        const long n = f.n_items, c = f.n_cut_items;
                        const bool order = (n >= 4096 && c * (d <= 32 ? 2 : 8) >= n) || (d > 32 && n >= 1536 && c * 4 >= n * 3);
                        wrong += fs_spmm_wide(&f, 136) != (n >= 1024) || fs_sddmm_in_order(&f, d) != (f.K * d * 2 > 4 << 20 && order);
                        seen++;
                    }
        }
    printf("%ld %ld\n", seen, wrong);
    // and the shorter items of small matrices do not pass for many
    for (long blocks : {3000L, 4092L, 4093L, 16380L}) {
        fs_format f{};
        f.V = 8; f.KB = 32; f.K = 200000; f.n_blocks = blocks; f.chunk = 32 * (blocks < 8192 ? fs_short_part_blocks(blocks) : 8);
        f.n_items = blocks / 2; f.n_cut_items = f.n_items;
        printf("%d %d ", fs_spmm_wide(&f, 136), fs_sddmm_in_order(&f, 32));
    }
}
"""


def build(tmp, name, text):
    src, exe = tmp / (name + ".hip"), tmp / name
    src.write_text(text)
    csrc = os.path.join(ROOT, "paper_2412_11007_amd", "csrc")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I" + csrc,
                    "-I" + os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True, capture_output=True)
    return str(exe)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return build(tmp_path_factory.mktemp("launch_order"), "order", PROGRAM)


def counts(program, M, items, cut, full):
    return [int(x) for x in subprocess.run([program] + [str(x) for x in (M, items, cut, full)], check=True, text=True, capture_output=True).stdout.split()]


@pytest.mark.parametrize("M,items", [(262144, 8192), (262152, 8193), (100003, 3126), (65536, 2048), (8192, 303), (4000, 5)])
def test_rows_with_entries_on_one_side_reach_every_xcd(program, M, items):
    """Entries in the first rows only (a padded batch, isolated nodes behind a sampled block): every XCD gets its eighth of the items that
    hold any, to within a workgroup of up to four items."""
    for full in {items // 8, items // 3, items}:
        ok, *most = counts(program, M, items, 0, full)
        assert ok
        for wpb, m in zip((1, 2, 4), most):
            assert m <= full / 8 + wpb, (M, items, full, wpb, m)


@pytest.mark.parametrize("items,cut", [(8192, 8192), (9001, 5000), (20000, 12345), (4100, 4097), (515, 7)])
def test_launch_order_is_a_permutation(program, items, cut):
    """... and the parts of cut windows, which an XCD takes in runs, are each taken once."""
    assert counts(program, 500000, items, cut, items)[0]


def test_routes_ask_for_the_items_of_a_callers_chunk(tmp_path):
    """fs_spmm's wide passes and fs_sddmm's order by the number of items: a chunk of the caller's makes as many in a small matrix as it
    likes, and only the shorter items that the conversion makes there by itself are counted by their blocks."""
    first, second = subprocess.run([build(tmp_path, "routes", ROUTES)], check=True, text=True, capture_output=True).stdout.split("\n")[:2]
    seen, wrong = (int(x) for x in first.split())
    assert seen > 100000 and wrong == 0, (seen, wrong)
    assert [int(x) for x in second.split()] == [0, 0, 0, 0, 1, 0, 1, 0]
