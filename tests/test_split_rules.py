"""The rules that cut work lists (csrc/split_rules.h, plain C++) at the ends of their ranges."""
import os
import subprocess
import textwrap

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_13356_amd", "csrc")


def _run(tmp_path, body):
    src = tmp_path / "t.cpp"
    src.write_text("#include <cstdio>\n#include <initializer_list>\n#include \"split_rules.h\"\nusing namespace lss;\nint main() {\n" +
                   textwrap.dedent(body) + "\nreturn 0;\n}\n")
    exe = tmp_path / "t"
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", str(exe)])
    return subprocess.check_output([str(exe)], text=True).split()


def test_m2l_plan_ends_where_its_indices_do(tmp_path):
    """Pair indices of the M2L plan are int32: lists up to 2^31 - 1 pairs, longer ones by class."""
    assert _run(tmp_path, """
        for (int64_t n : {int64_t(0), int64_t(1), (int64_t(1) << 31) - 1, int64_t(1) << 31, int64_t(1) << 40})
            printf("%d ", m2l_plan_holds(n));
    """) == ["1", "1", "1", "0", "0"]


def test_every_piece_of_a_direct_sum_has_work(tmp_path):
    """All tile widths, target and node counts up to where the split ends: the pieces cover the nodes in order, none is
    empty where a tile walks all nodes, and targets times pieces stay below what a context allocates for, 2^19 at most
    (the workspace of the allocation-free call)."""
    assert _run(tmp_path, """
        for (int tile : {64, 128, 256})
            for (int64_t n = 1; n < 200000; n += 1 + n / 7)
                for (int64_t nodes = 1; nodes < 3000000; nodes += 1 + nodes / 9)
                    for (bool whole : {true, false}) {
                        const int64_t tiles = (n + tile - 1) / tile, chunks = (nodes + tile - 1) / tile;
                        const int s = direct_pieces(tiles, chunks, tile, whole);
                        int64_t at = 0, none = 0;
                        for (int k = 0; k < s; ++k) {
                            int64_t lo = 0, hi = nodes;
                            piece_range(tile, k, s, lo, hi);
                            if (lo != at || hi < lo || (whole && hi == lo)) ++none;
                            at = hi;
                        }
                        if (none || at != nodes || s < 1 || (s > 1 && n * s > direct_partials_kept(n, chunks, tile))) {
                            printf("%d %ld %ld: %d pieces, %ld wrong ", tile, (long)n, (long)nodes, s, (long)none);
                            return 0;
                        }
                    }
        printf("ok");
    """) == ["ok"]


def test_a_smaller_direct_sum_needs_no_more(tmp_path):
    """What a context allocates for grows with the number of targets up to where the split ends, to 2^19 at most."""
    assert _run(tmp_path, """
        for (int tile : {64, 128, 256})
            for (int64_t chunks = 1; chunks < 20000; chunks += 1 + chunks / 5) {
                int64_t before = 0;
                for (int64_t n = 1; n <= 163840 - tile; n += 1 + n / 50) {
                    const int64_t k = direct_partials_kept(n, chunks, tile);
                    if (k < before || k > (1 << 19)) {
                        printf("%d %ld %ld: %ld after %ld ", tile, (long)chunks, (long)n, (long)k, (long)before);
                        return 0;
                    }
                    before = k;
                }
            }
        printf("ok");
    """) == ["ok"]
