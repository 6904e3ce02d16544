"""Checks on the compiler's listing of the few-row products (CPU only: hipcc cross-compiles gfx950 here): the library holds the
shapes that the dispatch can choose and no others, and none of them keeps registers in memory."""
import re
import shutil
import subprocess

import pytest

from paper_2503_06433_amd import build as bld

EPI_STORE, EPI_RESIDUAL, EPI_SWIGLU, EPI_STORE_F32, EPI_HEAD, EPI_UPLOAD = 0, 1, 2, 3, 100, 101


@pytest.fixture(scope="module", params=[(), ("-DSS_HALF_F16",)], ids=["bf16", "half"])
def kernels(request, tmp_path_factory):
    """(element, row tiles, column tiles, waves, chunks on their way, epilogue) of every kernel"""
    if not shutil.which("hipcc"):
        pytest.skip("hipcc not on PATH")
    out = str(tmp_path_factory.mktemp("few_rows") / "k.s")
    r = subprocess.run(["hipcc", *bld.FLAGS, *request.param, "--cuda-device-only", "-S", bld.CSRC + "/k_gemm_direct.hip", "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found, name = {}, None
    with open(out) as f:
        for line in f:
            m = re.match(r"^_ZN\w*gemm_direct_kernelI([tf])((?:Li\d+E){5})\w*:", line)
            if m:
                name = (m.group(1), *(int(v) for v in re.findall(r"\d+", m.group(2))))
                found[name] = None
            m = re.match(r"^; ScratchSize: (\d+)", line)
            if m and name:
                found[name], name = int(m.group(1)), None
    return bool(request.param), found


def test_only_shapes_that_a_rule_can_choose(kernels):
    half, found = kernels
    assert {k[0] for k in found} == ({"t"} if half else {"t", "f"})
    for t, mt, nt, waves, chunks, epi in found:
        assert not (half and epi == EPI_HEAD)
        assert waves == 8 or (t, mt, waves, chunks) == ("t", 1, 16, 2) and (nt == 1 or (nt, epi) == (2, EPI_SWIGLU))
    for shape in {k[:5] for k in found if (k[2], k[3]) != (2, 16)}:
        assert {k[5] for k in found if k[:5] == shape} == {EPI_STORE, EPI_UPLOAD, EPI_RESIDUAL, EPI_SWIGLU, EPI_STORE_F32} | (set() if half else {EPI_HEAD})


def test_no_kernel_spills(kernels):
    assert {k: v for k, v in kernels[1].items() if v != 0} == {}
