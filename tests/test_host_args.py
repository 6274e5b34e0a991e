"""The binding's argument checks where a tensor has the right shape and type but not the right
layout or place, and where an argument is no tensor of the expected rank; the stream a call goes
to (no GPU needed)."""

import pytest
import torch

import paper_2602_07721_amd as pk
import workloads

f16 = torch.float16


def _call(**change):
    cfg = pk.Config(2, 4, 64, workloads.rotation_signs(3))
    a = dict(q=torch.zeros((1, 8, 128), dtype=f16), K=torch.zeros((1, 2, 64, 128), dtype=f16),
             V=torch.zeros((1, 2, 64, 128), dtype=f16), out=torch.zeros((1, 8, 128)),
             out_idx=torch.zeros((1, 8, 8), dtype=torch.int32), workspace=torch.zeros(1024, dtype=torch.uint8))
    index = pk.Index(torch.zeros((1, 2, 64, 16), dtype=torch.uint8), torch.zeros((1, 2, 64, 128), dtype=torch.uint8),
                     torch.zeros((1, 2, 16, 256), dtype=torch.int32))
    if "ids" in change:
        index.ids = change.pop("ids")
    a.update(change)
    q, K, V = a.pop("q"), a.pop("K"), a.pop("V")
    return pk.retrieve_attend(cfg, index, q, 64, pk.Budget(16, 32, 8), K, V, 0.1, **a)


@pytest.mark.parametrize("name,value", [
    ("q", torch.zeros((1, 8, 256), dtype=f16)[:, :, ::2]), ("K", torch.zeros((1, 2, 128, 64), dtype=f16).mT),
    ("V", torch.zeros((1, 2, 128, 128), dtype=f16)[:, :, ::2]), ("out", torch.zeros((128, 8, 1)).permute(2, 1, 0)),
    ("out_idx", torch.zeros((1, 8, 16), dtype=torch.int32)[:, :, ::2]),
    ("workspace", torch.zeros(2048, dtype=torch.uint8)[::2]),
    ("ids", torch.zeros((1, 2, 64, 32), dtype=torch.uint8)[..., ::2]),
])
def test_strided_tensors_are_refused(name, value):
    with pytest.raises(ValueError, match="must be contiguous"):
        _call(**{name: value})


@pytest.mark.parametrize("name,value,error,message", [
    ("K", [1, 2], TypeError, "K must be a torch tensor"), ("V", None, ValueError, "V is required"),
    ("K", torch.zeros((2, 64, 128), dtype=f16), ValueError, "K must have shape"),
    ("V", torch.zeros((1, 2, 63, 128), dtype=f16), ValueError, "V must have shape"),
    ("K", torch.zeros((1, 2, 64, 128)), TypeError, "K must be torch.float16"),
    ("workspace", torch.zeros((2, 512), dtype=torch.uint8), ValueError, "workspace must have shape"),
    ("workspace", torch.zeros(1024, dtype=torch.int8), TypeError, "workspace must be torch.uint8"),
    ("out", 3, TypeError, "out must be a torch tensor"), ("q", torch.zeros((8, 128), dtype=f16), ValueError, "q must be"),
])
def test_wrong_arguments_are_named(name, value, error, message):
    with pytest.raises(error, match=message):
        _call(**{name: value})


def test_every_shape_is_checked_before_the_place():
    with pytest.raises(ValueError, match="must be a GPU tensor"):
        _call()
    with pytest.raises(ValueError, match="index.ids must have shape"):
        _call(ids=torch.zeros((1, 2, 63, 16), dtype=torch.uint8))


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_the_stream_needs_no_private_name_of_torch(monkeypatch, missing):
    class Stream:
        cuda_stream = 4711

    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 815, raising=False)
    assert pk._stream(None) == 815 and pk._stream(Stream()) == 4711
    monkeypatch.delattr(torch._C, missing)
    assert pk._stream(None) == 4711
