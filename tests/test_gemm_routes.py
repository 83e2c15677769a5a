"""The GEMM cases run on a GPU (test_gpu_gemm.py, and the layers in test_gpu_model.py and
test_gpu_graph.py that are about one kernel family) take the family that they name: the
choice is made on the host by sizes, so it is checked here without a GPU."""
import pytest

pytest.importorskip("torch")

import test_gpu_gemm as gemm  # noqa: E402

LISTS = ("LINK", "BIG", "TALL", "WHOLE_NARROW", "SMALL", "MANY", "CUT", "REUSE", "STREAM", "WIDE", "SPLIT")


@pytest.mark.parametrize("name", LISTS)
def test_cases_take_the_kernel_they_name(name):
    for m, n, k, epi, kernel in getattr(gemm, name):
        assert gemm.kernel_of(m, n, k, epi) == kernel, (m, n, k, epi)


def test_precision_cases_take_the_kernel_they_name():
    for m, n, k, kernel, _, _ in gemm.WIDE_CHAINS:
        assert gemm.kernel_of(m, n, k, "store") == kernel
    for m, n, k, _, _ in gemm.CHAINS:
        assert gemm.kernel_of(m, n, k, "store") == "stream"


def test_whole_gate_up_cases():
    for m, n, k in gemm.GLU:
        assert gemm.kernel_of(m, n, k, "swiglu") == "glu"


def test_layer_cases_with_cut_tiles():
    import test_gpu_graph as graph
    import test_gpu_model as model
    for hq, hkv, d in model.CUT_ROPE:
        assert gemm.kernel_of(64, (hq + 2 * hkv) * d, 14336, "rope", True) == "cut"
    wl = graph.CUT_MODEL
    assert gemm.kernel_of(wl.suffix_len, 2 * wl.ffn, wl.hidden, "swiglu", True) == "cut"


# (m, n, k, epilogue), how much longer the route before took than cut tiles: where they make
# whole rounds, so that nothing is cut, and where few rows meet heavy weights
FASTER_CUT = [
    (257, 16384, 2048, "swiglu", 1.13), (320, 16384, 2048, "store", 1.09), (448, 16384, 4096, "swiglu", 1.13),
    (769, 8192, 4096, "residual", 1.13),
    (256, 32768, 4096, "store", 1.21), (64, 16384, 14336, "store", 1.26),
]


@pytest.mark.parametrize("m,n,k,epi,_", FASTER_CUT)
def test_cut_tiles_where_they_were_measured_faster(m, n, k, epi, _):
    assert gemm.kernel_of(m, n, k, epi) == "cut"


def test_refused_sizes_have_no_kernel():
    assert gemm.kernel_of(4, 100, 64, "store") == ""
    assert gemm.kernel_of(4, 128, 48, "store") == ""
    assert gemm.kernel_of(0, 128, 64, "store") == ""
