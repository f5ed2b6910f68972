"""CPU checks of host decisions of the layer that depend on where buffers lie: the code that decides, compiled for the host, with functions in the place of
the launches that tell what would be launched."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PAIR = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "ffn_common.hpp"
namespace exf {
bool exact_pair_fits(int64_t, int, int, int) { return true; }
bool exact_pair_routed_fits(int64_t, int, int, int) { return true; }
int launch_exact_pair(const StreamGemm&, const StreamGemm&, hipStream_t) { puts("one"); return 0; }
int launch_stream_gemm(const StreamGemm&, int, hipStream_t) { puts("two"); return 0; }
}
int main(int argc, char** argv)
{
    exf::StreamGemm a{}, b{};
    auto at = [&](const char* name) -> char* {
        for (int i = 1; i + 1 < argc; i += 2)
            if (strcmp(argv[i], name) == 0) return reinterpret_cast<char*>(strtoull(argv[i + 1], nullptr, 0));
        return nullptr;
    };
    auto ints = [&](const char* name) { return reinterpret_cast<int32_t*>(at(name)); };
    a.max_rows = b.max_rows = 1024, a.K = b.N = 64, a.N = b.K = 256, a.E_local = b.E_local = a.E = 8;
    a.a_div = static_cast<int>(reinterpret_cast<uintptr_t>(at("k")));
    a.act = at("x"), a.weight = at("w1"), a.sorted_act = at("x_sorted"), a.a_row = ints("src_of_sorted"), a.src_of_sorted = ints("src_of_sorted");
    a.topk_idx = ints("ids"), a.expert_map = ints("map"), a.expert_counts = ints("counts");
    b.out = at("out"), b.sorted_out = at("y_sorted"), b.out_row = a.a_div == 1 ? a.src_of_sorted : nullptr;
    return exf::launch_stream_pair(a, b, EXF_F32, nullptr);
}
"""


def _compile(tmp, name, text):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    src, exe = str(tmp / (name + ".cpp")), str(tmp / name)
    with open(src, "w") as f:
        f.write(text)
    csrc = os.path.join(ROOT, "paper_2401_08383_amd", "csrc")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, src, "-o", exe], check=True, capture_output=True)

    def run(**values):
        args = [w for k, v in values.items() for w in (k, str(v))]
        return subprocess.run([exe, *args], check=True, capture_output=True, text=True).stdout.split()

    return run


@pytest.fixture(scope="module")
def pair(tmp_path_factory):
    return _compile(tmp_path_factory.mktemp("pair"), "pair", PAIR)


# 1024 rows of 64 floats, a megabyte between buffers
ROWS, MB = 1024 * 64 * 4, 1 << 20
APART = dict(x=1 * MB, w1=2 * MB, x_sorted=4 * MB, src_of_sorted=5 * MB, ids=6 * MB, map=7 * MB, counts=8 * MB, out=9 * MB, y_sorted=10 * MB)


@pytest.mark.parametrize("k,moved,launches", [
    (1, {}, 1), (1, {"out": 4 * MB}, 2), (1, {"out": 4 * MB + ROWS - 16}, 2), (1, {"out": 4 * MB - ROWS + 16}, 2), (1, {"out": 4 * MB + ROWS}, 1), (1, {"out": 4 * MB - ROWS}, 1),
    (1, {"y_sorted": 4 * MB}, 1), (1, {"y_sorted": 4 * MB + 256}, 2), (1, {"y_sorted": 4 * MB, "out": 4 * MB}, 2), (1, {"x_sorted": 0, "y_sorted": 0}, 1),
    (1, {"x_sorted": 0, "y_sorted": 0, "out": 1 * MB + 256}, 2), (1, {"y_sorted": 1 * MB}, 2), (1, {"out": 6 * MB - 256}, 2), (1, {"out": 7 * MB}, 2), (1, {"out": 2 * MB + 64}, 2),
    (2, {"y_sorted": 0}, 1), (2, {"y_sorted": 0, "out": 4 * MB}, 1), (2, {"y_sorted": 0, "out": 4 * MB - 256}, 2), (2, {"y_sorted": 0, "out": 5 * MB}, 2),
    (2, {"y_sorted": 0, "out": 1 * MB + ROWS // 2}, 1), (2, {"y_sorted": 0, "out": 1 * MB + ROWS // 2 - 16}, 2), (1, {"out": (1 << 64) - 256}, 1)])
def test_one_launch_only_where_results_lie_apart_from_what_the_first_contraction_touches(pair, k, moved, launches):
    """fp32, both contractions and the sort as one launch: with results over the sorted copies of the rows, the ids or x it would be a race.  (k = 2: the
    second contraction leaves the sorted rows, `out` here.)"""
    at = {**APART, **moved}
    assert pair(k=k, **at) == (["one"] if launches == 1 else ["two", "two"])
