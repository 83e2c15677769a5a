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


def test_whole_gate_up_cases():
    for m, n, k in gemm.GLU:
        assert gemm.kernel_of(m, n, k, "swiglu") == "glu"


def test_layer_cases_with_cut_tiles():
    import test_gpu_graph as graph
    import test_gpu_model as model
    for wl in model.CUT_ROPE + [graph.CUT_MODEL]:
        n = (wl.num_q_heads + 2 * wl.num_kv_heads) * wl.head_dim
        assert gemm.kernel_of(wl.suffix_len, n, wl.hidden, "rope") == "cut"


def test_refused_sizes_have_no_kernel():
    assert gemm.kernel_of(4, 100, 64, "store") == ""
    assert gemm.kernel_of(4, 128, 48, "store") == ""
    assert gemm.kernel_of(0, 128, 64, "store") == ""
