"""Where the node blocks of a wave lie in LDS, checked at compile time (host
side only): the 16-byte stores that fill them need each block on 16 bytes,
also the second to fourth of the kernels that take several elements to a wave."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
#include "newton_mfma.hpp"
using namespace fpts;
template <typename T, int D, int R, int N>
constexpr bool ok()
{
    typedef newton::NodeLds<T, D, R, N> L;
    // block u of a wave starts at u * STRIDE, the tables after the last one
    return L::STRIDE >= L::SIZE && L::STRIDE * sizeof(T) % 16 == 0 &&
           newton::Lds<T, D, R, N>::NODES == L::STRIDE;
}
template <int N>
constexpr bool all()
{
    return ok<double, 3, 3, N>() && ok<double, 3, 2, N>() && ok<double, 2, 2, N>() &&
           ok<float, 3, 3, N>() && ok<float, 3, 2, N>() && ok<float, 2, 2, N>();
}
static_assert(all<2>() && all<3>() && all<4>() && all<5>() && all<6>(), "");
static_assert(all<7>() && all<8>() && all<9>() && all<10>(), "");
"""


def test_node_blocks_start_on_16_bytes(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src = tmp_path / "layout.cpp"
    src.write_text(SRC)
    r = subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only",
                        "-fsyntax-only", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2501_12349_amd", "csrc"), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
