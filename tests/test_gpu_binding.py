"""The binding's stream and its checks of shapes and devices."""

import threading

import pytest
import torch

import paper_2609_33410_amd as F
from paper_2609_33410_amd import fold

pytestmark = pytest.mark.gpu


def test_stream_is_the_callers_current_one():
    """In a stream context, in another thread beside it, and under capture."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    other = []
    with torch.cuda.stream(side):
        assert fold._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
        th = threading.Thread(target=lambda: other.append(fold._stream(None)))
        th.start()
        th.join()
        g = torch.cuda.CUDAGraph()
        x = torch.zeros(4, device="cuda")
        with torch.cuda.graph(g):
            assert fold._stream(None) == torch.cuda.current_stream().cuda_stream
            x.add_(1)
    assert other == [torch.cuda.default_stream().cuda_stream]
    assert fold._stream(None) == torch.cuda.current_stream().cuda_stream
    assert fold._stream(side) == side.cuda_stream


@pytest.mark.parametrize("name", ["_RAW_STREAM", "_RAW_DEVICE"])
def test_stream_without_torchs_raw_handle(name, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setattr(fold, name, None)
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert fold._stream(None) == side.cuda_stream


@pytest.mark.parametrize("what", ["part_A", "part_A rank", "part_L", "part_Lcut", "z", "device",
                                  "view device"])
def test_slots_of_another_shape_or_place_are_refused(what):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    b, h, hkv, d, n, s = 2, 4, 2, 64, 32, 3
    k = torch.zeros(b, hkv, n, d, dtype=torch.bfloat16, device="cuda")
    lens = torch.full((b,), n, dtype=torch.int32, device="cuda")
    q = torch.zeros(b, h, d, dtype=torch.bfloat16, device="cuda")
    shapes = {"part_A": (s, b, h, d), "part_L": (s, b, h), "part_Lcut": (s, b, h), "z": (b, h)}
    if what == "part_A rank":
        shapes["part_A"] = (s, b, h * d)
    elif what in shapes:
        shapes[what] = shapes[what][:-1] + (shapes[what][-1] - 1,)
    t = {nm: torch.zeros(sh, device="cuda") for nm, sh in shapes.items()}
    if what == "device":
        t["part_L"] = t["part_L"].cpu()
    if what == "view device":
        lens = lens.cpu()
    kv = F.kv_view(k, k, lens, num_kv_heads=hkv, max_seq_len=n)
    with pytest.raises(ValueError, match="view tensor 2" if what == "view device" else
                       "part_L must be a device" if what == "device" else what.split()[0]):
        F.fold_decode_split(kv, F.q_view(q), 1.0, t["z"], 16.0, s, 0, t["part_A"], t["part_L"],
                            part_Lcut=t["part_Lcut"])
