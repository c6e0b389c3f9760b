"""The library holds the kernel instances that its dispatch reaches, and no
others: each costs time when a process loads it."""
import os
import re
import shutil
import subprocess

import pytest

amg = pytest.importorskip("paper_1403_1649_amd")


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(amg.library_path()):
        pytest.skip("libamg_hip.so not built")
    if not shutil.which("nm"):
        pytest.skip("nm not found")
    out = subprocess.run(["nm", "-C", amg.library_path()], capture_output=True, text=True, check=True).stdout
    return sorted(set(re.findall(r"__device_stub__(k_\w+<.*>)\(", out)))


def test_corrected_iterates_of_small_levels_are_csr_alone(kernels):
    small = [k for k in kernels if re.search(r"Corr[VK]<", k) and not k.startswith(("k_elem<", "k_finalize<"))]
    assert small
    assert all(re.match(r"k_rows<\w+, \d+, .*, false>$", k) for k in small)


def test_one_lane_per_row_is_the_callers_product(kernels):
    one = [k for k in kernels if re.match(r"k_rows<\w+, 1, ", k)]
    assert len(one) == 1 and "OpSpmv" in one[0]


def test_block_kernels_take_offsets_for_the_post_smoothing_operator(kernels):
    off = [k for k in kernels if re.match(r"k_rows_m<\w+, \d+, \d+, true, ", k)]
    assert off and all("MPostT<" in k for k in off)


def test_the_combined_coarse_vectors_are_not_streamed(kernels):
    post = [k for k in kernels if "OpPostT" in k]
    assert any(k.startswith("k_stream<") for k in post)
    assert not any(k.startswith("k_stream<") and "CoarseK<" in k for k in post)
    assert all(re.match(r"k_rows<\w+, [48], ", k) for k in post if k.startswith("k_rows<"))
