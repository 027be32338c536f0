"""When a pass of one row takes the one launch (csrc/row_rule.h, plain arithmetic), against what was measured on both sides of
the line."""
import pathlib
import subprocess

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2603_09215_amd" / "csrc"

# MB a layer, layers, us a step gained by the one launch (the least of the contexts measured)
MEASURED = [
    (130, 8, 6), (162, 4, -11), (162, 6, -2), (162, 8, 6),
    (189, 2, -12), (189, 4, -4), (189, 8, 9), (198, 3, -3), (199, 4, -1), (198, 6, 17), (198, 8, 28),
    (209, 4, 1), (209, 8, 21), (219, 4, 3), (229, 4, 4), (229, 8, 30),
    (294, 2, -6), (294, 3, 5), (294, 4, 15), (294, 8, 54), (408, 2, -2), (408, 3, 10), (408, 4, 26), (408, 8, 77),
    (466, 2, 1), (466, 4, 26), (466, 8, 73), (466, 14, 147),
]
DRIVER = r"""
#include <cstdio>
#include "row_rule.h"
int main() {
  double mb; int layers;
  while (scanf("%lf %d", &mb, &layers) == 2) printf("%d\n", (int)spark::one_row_pays((size_t)(mb * 1e6), layers));
}
"""


def test_rule_takes_the_launch_only_where_it_was_measured_to_gain(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], input="".join(f"{mb} {layers}\n" for mb, layers, _ in MEASURED), capture_output=True, text=True, check=True)
    taken = [t == "1" for t in out.stdout.split()]
    assert len(taken) == len(MEASURED)
    for (mb, layers, gain), t in zip(MEASURED, taken):
        assert not t or gain > 0, (mb, layers, gain)
        # from 189 MB and four layers on, what gains more than 2 % of a step (0.31 us a MB and layer) is not passed over
        assert t or mb < 189 or layers < 4 or gain <= 0.02 * 0.31 * mb * layers, (mb, layers, gain)


def test_numbers_begin_again_before_they_run_out(tmp_path):
    src, exe = tmp_path / "numbers.cpp", tmp_path / "numbers"
    src.write_text("""
#include <cstdio>
#include "row_rule.h"
int main() {
  unsigned last, layers;
  while (scanf("%u %u", &last, &layers) == 2) printf("%d\\n", (int)spark::row_numbers_run_out(last, layers));
}
""")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    points = [(last, layers) for layers in (1, 4, 28) for last in (0, 1, 2 ** 31 - 1, *(2 ** 32 - 1 - layers + k for k in (-1, 0, 1)), 2 ** 32 - 1)
              if last < 2 ** 32]
    out = subprocess.run([str(exe)], input="".join(f"{a} {b}\n" for a, b in points), capture_output=True, text=True, check=True)
    for (last, layers), took in zip(points, out.stdout.split(), strict=True):
        assert (took == "1") == (last + layers > 2 ** 32 - 1), (last, layers)
