"""Sizes and rules that the router's launches are planned by, from the header
they stand in (host only: compiled for the CPU)."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_18410_amd", "csrc")
SOURCE = r"""
#include <algorithm>
#include "launch.hpp"
using namespace rolesub;
extern "C" {
// bytes that one launch of the two-kernel form addresses, in the larger of the
// areas that a workspace holds behind its other pieces
size_t launch_bytes(int B, int T, int d, int Hr, int G, int C, int kind, int bf16, size_t* area, size_t* ntile) {
  const int MB = route_tile_blocks(Hr, G, C, kind), S = route_tile_slices(d, MB, kind, bf16);
  const size_t sk = (route_sk_part_floats(B, T, Hr, kind) + route_sk_cnt_ints(B, T, Hr, kind)) * 4;
  *area = std::max(sk, route_tile_bytes(B, T, Hr, G, C, kind)) - route_fold_floats(Hr, G, C, kind) * 4;
  *ntile = std::min(route_tile_step(*area, S, MB), (static_cast<size_t>(B) * T + 63) / 64);
  return *ntile * S * MB * 4096;
}
// h, W1, W_r and E at the addresses given
bool uses_tiles(int B, int T, int d, int G, int C, int d_e, int Hr, int kind, int bf16, size_t h, size_t W1, size_t W_r, size_t E) {
  RouteParams p = {};
  p.B = B; p.T = T; p.d = d; p.G = G; p.C = C; p.d_e = d_e; p.Hr = Hr; p.kind = kind;
  p.h = reinterpret_cast<void*>(h); p.W1 = reinterpret_cast<void*>(W1);
  p.W_r = reinterpret_cast<void*>(W_r); p.E = reinterpret_cast<void*>(E);
  return route_uses_tiles(p, bf16);
}
bool sk_fits(int B, int T) { return route_sk_fits(B, T); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                    str(d / "plan.cpp"), "-o", str(d / "plan.so")], check=True)
    lib = ctypes.CDLL(str(d / "plan.so"))
    lib.launch_bytes.restype = ctypes.c_size_t
    lib.sk_fits.restype = lib.uses_tiles.restype = ctypes.c_bool
    return lib


@pytest.mark.parametrize("d,Hr,G,C,kind", [(256, 128, 8, 8, 0), (64, 128, 8, 17, 0), (4096, 128, 32, 64, 0), (64, 300, 8, 8, 0),
                                           (8000, 4000, 32, 64, 0), (4096, 0, 32, 6, 1), (33, 0, 1, 1, 1)])
@pytest.mark.parametrize("bf16", [0, 1])
def test_launches_stay_within_32_bit_offsets(plan, d, Hr, G, C, kind, bf16):
    area, ntile = ctypes.c_size_t(), ctypes.c_size_t()
    for B, T in ((1, 1), (2, 80), (64, 177), (1500, 177), (11000, 177), (24000, 177), (1, 1 << 20), (1 << 20, 2000)):
        n = plan.launch_bytes(B, T, d, Hr, G, C, kind, bf16, ctypes.byref(area), ctypes.byref(ntile))
        assert 1 <= ntile.value and n < 2 ** 31 and n <= area.value, (B, T, n, area.value)


def test_split_k_only_where_its_offsets_reach(plan):
    for B, T in ((1, 48), (64, 177), (10000, 177), (10531, 177), (10532, 177), (11000, 177), (24000, 177), (1 << 20, 1000)):
        tiles = -(-B * T // 96)  # two halves of six waves, nine 16-byte products a lane
        assert plan.sk_fits(B, T) == (tiles * 2 * 6 * 64 * 9 * 16 < 2 ** 31), (B, T)


def test_one_kernel_forms_take_only_what_their_dma_copies(plan):
    A = 0x7f0000001000  # 16-byte boundary

    def tiles(B=64, T=177, d=4096, G=8, C=8, d_e=128, Hr=128, kind=0, bf16=1, off=(0, 0, 0, 0)):
        return plan.uses_tiles(B, T, d, G, C, d_e, Hr, kind, bf16, *(ctypes.c_size_t(A + x) for x in off))

    assert not tiles() and not tiles(B=1, T=3073) and not tiles(off=(16, 32, 48, 64)) and not tiles(d=64, d_e=8)
    assert tiles(B=1, T=3072) and tiles(bf16=0) and tiles(kind=1) and tiles(Hr=64) and tiles(C=17) and tiles(d=4128)
    assert tiles(d_e=4) and tiles(d_e=127)
    for i in range(4):
        for x in (2, 4, 8, 14):
            off = [0] * 4
            off[i] = x
            assert tiles(off=off), off
    # language terms of 2 GiB and more
    assert tiles(B=1 << 22, T=2, d=64) and not tiles(B=(1 << 22) - 1, T=2, d=64)
