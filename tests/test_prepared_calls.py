"""A prepared call keeps the tensors whose pointers it holds alive: a program
may drop its own references (a workspace passed as a temporary, a list of
payloads that it fills anew) and go on calling.  Runs on the CPU with a stand-in for the library."""
import gc
import weakref

import pytest

torch = pytest.importorskip("torch")
from paper_2108_00951_amd import binding as efs  # noqa: E402


class _Library:
    """Accepts every call."""

    @staticmethod
    def sparse_apply(*args):
        return efs.EFS_OK

    sparse_accumulate = sparse_apply


@pytest.mark.parametrize("as_list", [False, True])
@pytest.mark.parametrize("kind", ["accumulate", "sgd", "momentum"])
def test_prepared_call_keeps_its_tensors(kind, as_list, monkeypatch):
    monkeypatch.setattr(efs, "load_library", lambda *a: _Library)
    monkeypatch.setattr(efs, "_require", lambda *a: torch)
    monkeypatch.setattr(efs, "_stream_handle", lambda s: 0)
    d = 64
    tensors = {"idx": torch.zeros(4, dtype=torch.int32), "val": torch.zeros(4),
               "counter": torch.zeros(4, dtype=torch.int32), "x": torch.zeros(d),
               "ws": torch.zeros(256, dtype=torch.uint8)}
    if kind == "momentum":
        tensors["m"] = torch.zeros(d)
    t = tensors
    payload = (t["idx"], t["val"], t["counter"])
    payloads = [list(payload) if as_list else payload]
    if kind == "accumulate":
        call = efs.prepare_sparse_accumulate(payloads, d, t["x"], t["ws"])
    else:
        mode = efs.APPLY_SGD if kind == "sgd" else efs.APPLY_MOMENTUM
        call = efs.prepare_sparse_apply(payloads, d, mode, t["x"], t["ws"], m=t.get("m"))
    alive = [weakref.ref(v) for v in tensors.values()]
    if as_list:   # the caller's own list, put to another use
        payloads[0].clear()
        payloads.clear()
    del tensors, t, payload, payloads
    gc.collect()
    call()
    assert all(r() is not None for r in alive)
    del call
    gc.collect()
    assert all(r() is None for r in alive)
