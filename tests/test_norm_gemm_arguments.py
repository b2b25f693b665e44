"""What the launcher of the products behind a normalisation refuses, before anything is launched (no GPU needed): it is called in the built library."""
import os
import subprocess

from paper_2305_17423_amd import build
from paper_2305_17423_amd.binding import LIB_PATH

PROGRAM = r"""
#include <cstdio>
#include "%s/igemm.h"
using namespace fise;
int main() {
    alignas(16) static char any[64];
    for (int src = 0; src < 4; ++src)
        for (int geglu = 0; geglu < 2; ++geglu)
            for (int bias = 0; bias < 2; ++bias) {
                NormGemmArgs a{};
                a.x = any; a.src = src; a.K = 320; a.G = 32; a.tile = 1; a.tiles_w = a.Ho = a.Wo = 8; a.B = 1; a.Ma = 64;
                a.w[0] = (const bf16_t*)any; a.N = a.sect_n = 320; a.geglu = geglu; a.out[0] = (bf16_t*)any; a.mode[0] = OUT_COMPACT;
                a.bias = bias ? (const bf16_t*)any : nullptr;
                const bool refused = (geglu && src != NG_ROWS_LN) || (bias && !geglu && (src == NG_ROWS_LN || src == NG_MAP_LN));
                if (refused && launch_norm_gemm(a, nullptr) != FISE_ERR_SHAPE) std::printf("accepted: src %%d geglu %%d bias %%d\n", src, geglu, bias);
                if (bias && !refused && !norm_gemm_has_bias(geglu, src)) std::printf("dropped: src %%d geglu %%d\n", src, geglu);
            }
    std::puts("done");
}
"""


def test_a_bias_that_would_not_be_added_is_refused(tmp_path):
    (tmp_path / "arguments.cpp").write_text(PROGRAM % build.CSRC)
    r = subprocess.run([build.HIPCC, "-std=c++17", "-x", "hip", "--offload-host-only", "-c", str(tmp_path / "arguments.cpp"), "-o", str(tmp_path / "arguments.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    subprocess.run([build.HIPCC, str(tmp_path / "arguments.o"), LIB_PATH, "-Wl,-rpath," + LIB_PATH.rsplit("/", 1)[0], "-o", str(tmp_path / "arguments")], check=True)
    nothing_to_launch_on = {**os.environ, "HIP_VISIBLE_DEVICES": "-1"}
    assert subprocess.run([str(tmp_path / "arguments")], env=nothing_to_launch_on, check=True, capture_output=True, text=True).stdout == "done\n"
