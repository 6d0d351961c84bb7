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
