"""The binding's native path: it takes every ordinary call, builds the same jobs as the
ctypes path, and leaves anything else to the checks that name the fault."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2206_01299_amd import binding as B


@pytest.fixture
def call():
    if not torch.cuda.is_available():
        pytest.fail("these tests need the MI355X; run them with -m gpu on the GPU box")
    d = torch.device("cuda:0")
    desc = B.make_desc(batch=2, n_per=128, n_samples=5, bits=4, group=64, dtype="bf16", rng_seed=2**63 + 5)
    return desc, dict(act=torch.ones((2, 128), dtype=torch.bfloat16, device=d),
                      ids=torch.tensor([3, 1], device=d), m=torch.zeros((5, 128), dtype=torch.bfloat16, device=d),
                      codes=torch.zeros(B.codes_bytes(desc) + 16, dtype=torch.uint8, device=d),
                      scales=torch.zeros(B.scales_count(desc), device=d),
                      out=torch.zeros((2, 128), dtype=torch.bfloat16, device=d))


def test_ordinary_calls_are_taken_and_odd_ones_handed_back(call):
    desc, t = call
    B.version()
    enc = lambda **k: B._native.encode(desc, *[{**t, **k}[n] for n in ("act", "ids", "m", "codes", "scales")],  # noqa: E731
                                       k.get("stream"))
    assert B._native.encode is not None and enc() == 0
    assert enc(stream=torch.cuda.Stream()) == 0
    for bad in (dict(act=t["act"].float()), dict(act=t["act"][:1]), dict(ids=t["ids"].int()), dict(m=t["m"][:4]),
                dict(codes=t["codes"][:8]), dict(scales=t["scales"].double()), dict(act=t["act"].cpu()),
                dict(act=torch.ones((128, 2), dtype=torch.bfloat16, device="cuda").t()), dict(stream=3), dict(ids=None)):
        assert enc(**bad) is None
    with pytest.raises(ValueError, match="sample_ids"):
        B.encode(desc, t["act"], t["ids"].int(), t["m"], t["codes"], t["scales"])
    bad = B.make_desc(batch=2, n_per=128, n_samples=5, bits=5, group=64, dtype="bf16")
    with pytest.raises(B.AqsgdError) as e:                   # the library's own status comes through
        B.encode(bad, t["act"], t["ids"], t["m"], t["codes"], t["scales"])
    assert e.value.status == -2


def test_native_jobs_equal_the_ctypes_ones(call, monkeypatch):
    desc, t = call
    makers = [lambda: B.encode_job(desc, t["act"], t["ids"], t["m"], t["codes"], t["scales"]),
              lambda: B.decode_job(desc, t["codes"], t["scales"], t["ids"], t["m"], t["out"]),
              lambda: B.grad_quant_job(desc, t["act"], t["codes"], t["scales"]),
              lambda: B.grad_dequant_job(desc, t["codes"], t["scales"], t["out"])]
    native = [ctypes.string_at(ctypes.addressof(j), ctypes.sizeof(j)) for j in (f() for f in makers)]

    class HandBack:
        def __getattr__(self, name):
            return lambda *a: None
    monkeypatch.setattr(B, "_native", HandBack())
    plain = [ctypes.string_at(ctypes.addressof(j), ctypes.sizeof(j)) for j in (f() for f in makers)]
    assert native == plain and len(set(native)) == 4
