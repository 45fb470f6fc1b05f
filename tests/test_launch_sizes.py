"""Host arithmetic of launch sizes near and past 32 bits: csrc/sizes.hpp
compiled by itself with the host compiler (CPU only), and, from the source,
that the setup kernels with several lanes per entry are launched through it
and take strides."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_09001_amd", "csrc")


def _run(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include "sizes.hpp"\nusing namespace amg;\nint main() {\n' + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return [int(t) for t in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


def test_stride_grid(tmp_path):
    items = [0, 1, 255, 256, 257, 1 << 31, (1 << 31) + 1, 67_108_864 << 6, (67_108_864 << 6) + 64, 1 << 40]
    out = _run(tmp_path, "\n".join(f'std::printf("%u\\n", stride_grid({t}LL, 256));' for t in items))
    for t, g in zip(items, out):
        assert 1 <= g and g * 256 < 1 << 32
        if t <= 1 << 31:                      # every item its own lane
            assert g == max(1, -(-t // 256))


def test_ell_fits(tmp_path):
    M = 1 << 30
    cases = [(1, 1, 1), (2 * M // 64, M - 1, 1), (67_108_864, 80_000_000, 1_250_000), (67_108_865, M - 1, 0),
             (67_108_864 + 100, 100, 100), (33_554_431, M - 1, 0), (33_554_432, M - 1, 1 << 20), (5, 128, 2), (7, 128, 2)]
    out = _run(tmp_path, "\n".join(f'std::printf("%d\\n", (int)ell_fits({s}, {z}, {k}));' for s, z, k in cases))
    want = [int(64 * s <= 2 * z + 64 * k and 64 * s < 1 << 31) for s, z, k in cases]
    assert out == want
    # (64 times the steps of the third and fifth case is 2^32 and a little more: 0 and 6,400 in 32 bits)
    assert want[2] == 0 and want[4] == 0
    text = open(os.path.join(CSRC, "fused.hip")).read()
    assert "cnt[sl] = (w + g - 1) / g;" in text and "ell_fits(steps, nnz, E.slices)" in text


@pytest.mark.parametrize("name,kernel", [("setup.hip", k) for k in ("k_pm", "k_pm_apply", "k_p_rows", "k_p_refill",
                                                                    "k_r_fill")] + [("fused.hip", "k_dt_values")])
def test_kernels_with_lanes_per_entry_take_strides(name, kernel):
    text = open(os.path.join(CSRC, name)).read()
    at = text.index(f" {kernel}(")
    body = text[at:text.index("\n}\n", at)]
    assert re.search(r"\+= (stride|\(int64_t\)gridDim\.x \* \w+)", body), kernel
    grids = re.findall(rf"hipLaunchKernelGGL\(\(?{kernel}(?:<[^>]*>)?\)?,\s*(\w+(?:\(\w+)?)", text)
    assert grids and set(grids) <= {"dim3(sys_grid", "dim3(stride_grid", "pg", "grid"}, grids
    if kernel == "k_p_rows":
        assert "const dim3 pg(stride_grid(" in text
    if kernel == "k_pm":
        assert "const dim3 grid(stride_grid(" in text
