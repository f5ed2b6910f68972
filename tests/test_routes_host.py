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
bool exact_pair_routed_fits(int64_t, int, int, int, int) { return true; }
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

LAYER = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "layer.hip"
namespace exf {
int fail(int code, const char*, ...) { return code; }
int check_gate(const void*, const void*, int64_t, int, int, int, int, const int32_t*, const float*) { return 0; }
int check_dispatch(const void*, const int32_t*, int64_t, int, int, int, int, int, const void*, const int32_t*, const int32_t*, const int32_t*, const int32_t*, const void*, size_t) { return 0; }
int check_ffn(const void*, const int32_t*, const void*, const void*, int64_t, int, int, int, int, int, const void*, const void*, size_t) { return 0; }
int check_ffn_fused(const void*, const int32_t*, const int32_t*, const float*, const int32_t*, const void*, const void*, int64_t, int, int, int, int, int, int, const void*, const void*, size_t) { return 0; }
int check_combine(const void*, const int32_t*, const float*, int64_t, int, int, int, const void*) { return 0; }
bool stream_path_fits(int64_t A, int, int, int, int) { return A <= 512; }
bool routed_tiles_fit(int64_t A, int, int, int, int, int) { return A > 512; }
bool gate_joins_layer(int64_t T, int, int, int, bool) { return T <= 16; }
int ffn_combined(const void*, const int32_t*, const int32_t*, const float*, const int32_t*, const void*, const void*, int64_t, int, int, int, int, int, void*, void*, void*, void*) { puts("ffn"); return 0; }
int ffn_fused_routed(const FfnRouting& r, const void*, const float*, const void*, const void*, int64_t, int, int, int, int, int, int, void*, void*, size_t, void*)
{
    puts(r.w_gate != nullptr ? "gated" : "routed");
    return 0;
}
}
extern "C" {
size_t moe_expert_ffn_workspace_bytes(int64_t, int, int, int, int) { return 1 << 20; }
size_t moe_expert_ffn_fused_workspace_bytes(int64_t, int, int, int, int, int) { return 1 << 20; }
int moe_gate_topk(const void*, const void*, int64_t, int, int, int, int, int, float*, int32_t*, float*, void*) { puts("gate"); return 0; }
int moe_dispatch(const void*, const int32_t*, const int32_t*, int64_t, int, int, int, int, int, void*, int32_t*, int32_t*, int32_t*, int32_t*, void*, size_t, void*) { puts("dispatch"); return 0; }
int moe_expert_ffn(const void*, const int32_t*, const void*, const void*, const void*, const void*, int64_t, int, int, int, int, int, void*, void*, size_t, void*) { puts("ffn"); return 0; }
int moe_expert_ffn_fused(const void*, const int32_t*, const int32_t*, const float*, const int32_t*, const void*, const void*, const void*, const void*, int64_t, int, int, int, int, int, int, void*, void*, size_t, void*) { puts("ffn"); return 0; }
int moe_combine(const void*, const int32_t*, const float*, int64_t, int, int, int, void*, void*) { puts("combine"); return 0; }
}
int main(int argc, char** argv)
{
    auto at = [&](const char* name) -> char* {
        for (int i = 1; i + 1 < argc; i += 2)
            if (strcmp(argv[i], name) == 0) return reinterpret_cast<char*>(strtoull(argv[i + 1], nullptr, 0));
        return nullptr;
    };
    auto number = [&](const char* name) { return reinterpret_cast<uintptr_t>(at(name)); };
    exf_moe_layer l{};
    l.T = number("T"), l.k = 1, l.d = 64, l.f = 256, l.E = 8, l.E_local = 8, l.dt = number("f32") ? EXF_F32 : EXF_BF16, l.fused = number("fused");
    l.x = at("x"), l.w_gate = at("w_gate"), l.forced_idx = reinterpret_cast<int32_t*>(at("ids")), l.expert_map = reinterpret_cast<int32_t*>(at("map"));
    l.topk_idx = reinterpret_cast<int32_t*>(at("topk_idx")), l.ffn_workspace = at("ws"), l.ffn_workspace_bytes = number("ws_bytes");
    return moe_layer_forward(&l, nullptr);
}
"""

RULE = r"""
#include <stdio.h>
#include <stdlib.h>
#include "ffn_stream.hip"
int main(int, char** argv)
{
    auto n = [&](int i) { return atoi(argv[2 * i]); };
    return puts(exf::exact_pair_routed_fits(n(1), n(2), n(3), n(4), n(5)) ? "one" : "two") < 0;
}
"""


def _compile(tmp, name, text, link=()):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    src, exe = str(tmp / (name + ".cpp")), str(tmp / name)
    with open(src, "w") as f:
        f.write(text)
    csrc = os.path.join(ROOT, "paper_2401_08383_amd", "csrc")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-x", "hip", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, src, "-o", exe, *link], check=True, capture_output=True)

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


@pytest.fixture(scope="module")
def layer(tmp_path_factory):
    return _compile(tmp_path_factory.mktemp("layer"), "layer", LAYER)


# a workspace of a megabyte is needed and given; the rows are T * 64 of two bytes (four)
BUFFERS = dict(x=1 * MB, w_gate=2 * MB, topk_idx=4 * MB, ws=16 * MB, ws_bytes=MB)
SEQUENCE = ["gate", "dispatch", "ffn"]


@pytest.mark.parametrize("T,fused,moved,calls", [
    (8, 0, {}, ["gated"]), (8, 1, {}, ["gated"]), (100, 0, {}, ["gate", "routed"]), (1000, 0, {}, ["gate", "routed"]), (1000, 1, {}, SEQUENCE),
    # x in the workspace, where it ends and begins, with a workspace given larger than is needed
    (8, 0, {"x": 16 * MB}, SEQUENCE), (100, 0, {"x": 17 * MB - 16}, SEQUENCE), (100, 0, {"x": 17 * MB}, ["gate", "routed"]), (1000, 0, {"x": 16 * MB + 64}, SEQUENCE),
    (1000, 0, {"x": 16 * MB - 128000}, ["gate", "routed"]), (1000, 0, {"x": 16 * MB - 127984}, SEQUENCE), (1000, 0, {"x": 17 * MB - 16, "ws_bytes": (1 << 64) - 1}, SEQUENCE),
    (1000, 0, {"x": 17 * MB, "ws_bytes": 64 * MB}, ["gate", "routed"]), (400, 0, {"x": 16 * MB - 102400, "f32": 1}, ["gate", "routed"]), (400, 0, {"x": 16 * MB - 102384, "f32": 1}, SEQUENCE),
    # the ids, the map, the gate's weights
    (100, 1, {"ids": 16 * MB + 64}, SEQUENCE), (1000, 0, {"ids": 16 * MB + 64}, SEQUENCE), (100, 0, {"ids": 8 * MB}, ["gate", "routed"]), (100, 1, {"map": 17 * MB - 4}, SEQUENCE),
    (1000, 0, {"map": 17 * MB - 4}, SEQUENCE), (1000, 0, {"map": 8 * MB}, ["gate", "routed"]), (8, 1, {"w_gate": 16 * MB}, ["gate", "routed"])])
def test_a_layer_is_calls_in_sequence_where_what_they_read_lies_in_the_workspace(layer, T, fused, moved, calls):
    """A first contraction that sorts reads x and the ids while hidden activations are written, where the calls in sequence have read them before."""
    assert layer(T=T, fused=fused, **{**BUFFERS, **moved}) == calls


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    return _compile(tmp_path_factory.mktemp("rule"), "rule", RULE, ("-Wl,--unresolved-symbols=ignore-all",))


@pytest.mark.parametrize("A,d,f,E,E_local,launches", [
    (1024, 64, 256, 8, 8, "one"), (512, 64, 256, 8, 8, "two"), (900, 468, 564, 29, 29, "one"), (900, 468, 564, 58, 29, "two"), (1000, 64, 256, 16, 2, "one"),
    (1000, 64, 256, 16, 1, "one"), (512, 32, 128, 8, 2, "one"), (700, 44, 300, 56, 7, "one"), (900, 92, 252, 32, 16, "one"), (1025, 64, 256, 8, 8, "two")])
def test_one_launch_of_a_share_of_the_experts(rule, A, d, f, E, E_local, launches):
    """Not where the rows that are dropped shorten two launches by more than clearing them costs."""
    assert rule(A=A, d=d, f=f, E=E, E_local=E_local) == [launches]
