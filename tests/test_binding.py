"""The Python binding's own behaviour (no GPU needed: every call here ends in the library's argument
checks, or in a stand-in for its entry point)."""
import pytest
import torch

from paper_2609_24433_amd import fq

M, K, N = 4, 1024, 16


@pytest.fixture(autouse=True)
def no_stream(monkeypatch):
    monkeypatch.setattr(fq, "_stream_handle", lambda: 0)


def tensors():
    return dict(x=torch.zeros((M, K), dtype=torch.bfloat16), codes=torch.zeros((M, K // 2), dtype=torch.uint8),
                delta=torch.zeros((M,)), w=torch.zeros((N * K // 2,), dtype=torch.uint8), sw=torch.zeros((N,)),
                blocks=torch.zeros((K // 64, 64, 64)))


@pytest.mark.parametrize("call,names", [
    (lambda t: fq.gemm(t["codes"], t["delta"], t["w"], t["sw"], N, K, 4), ("delta", "w", "sw")),
    (lambda t: fq.linear(t["x"], t["w"], t["sw"], N, 64, 4), ("w", "sw")),
    (lambda t: fq.linear_static(t["x"], t["w"], t["sw"], N, 64, 4), ("w", "sw")),
    (lambda t: fq.gemm_w4a16(t["x"], t["w"], t["sw"], N), ("w", "sw")),
    (lambda t: fq.rotate_quant(t["x"], None, t["blocks"], 64, 4), ("blocks",)),
], ids=["gemm", "linear", "linear_static", "gemm_w4a16", "rotate_quant"])
def test_a_missing_tensor_is_the_librarys_null_error(call, names):
    for name in names:
        t = tensors()
        t[name] = None
        with pytest.raises(fq.FQError) as e:
            call(t)
        assert e.value.status == 1


def test_output_of_a_tensor_subclass_is_a_plain_tensor(monkeypatch):
    class Sub(torch.Tensor):
        pass

    class Lib:  # accepts the call
        fq_linear_workspace_bytes = staticmethod(lambda *a: 0)
        fq_linear = staticmethod(lambda *a: fq.FQ_OK)
    monkeypatch.setattr(fq, "LIB", Lib)
    t = tensors()
    y = fq.linear(t["x"].as_subclass(Sub), t["w"], t["sw"], N, 64, 4)
    assert type(y) is torch.Tensor and y.shape == (M, N) and y.dtype == torch.bfloat16
