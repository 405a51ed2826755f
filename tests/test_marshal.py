"""The binding's native operand checks: what they hand over, and what they leave
to the binding's own checks (by returning None).  And the schedule's codes as
the library reads them, whatever sequence they come in."""
import array

import numpy as np
import pytest
import torch

from paper_2609_18145_amd import hcmix

bf, f32 = torch.bfloat16, torch.float32


def call(ts, count, shape, dtype=f32, dev="cpu"):
    return hcmix._native().pointers(ts, count, shape, dtype, torch.device(dev))


def test_cpu_tensors_and_other_operands_are_left_to_the_binding():
    t = torch.zeros(2, 3)
    assert call([t], 1, (2, 3)) is None                       # not in GPU memory
    assert call([t.tolist()], 1, (2, 3), dev="cuda:0") is None
    assert call([t], 2, (2, 3), dev="cuda:0") is None         # fewer than count
    assert call(iter([t]), 1, (2, 3), dev="cuda:0") is None   # no list or tuple
    assert call([torch.zeros(2, 3, device="meta")], 1, (2, 3), dev="meta") is None
    assert call([], 0, (2, 3)) == b""


@pytest.mark.parametrize("kind", [list, tuple, bytes, bytearray, np.array,
                                  lambda v: array.array("q", v), lambda v: [np.int64(e) for e in v],
                                  lambda v: np.array(v, dtype=np.uint8),
                                  lambda v: [float(e) for e in v], lambda v: memoryview(bytes(v))])
@pytest.mark.parametrize("codes", [[0, 1, 2, 3], [2, 0, 1], [5]])
def test_layer_codes_of_any_sequence(kind, codes):
    """One code per item, as int32: lengths that are and are not a multiple of
    four, which is what bytes taken for machine words would go by."""
    assert np.frombuffer(hcmix._layers(kind(codes)), dtype=np.int32).tolist() == codes
    want = hcmix.decode_cache_bytes(4, 256, 64, codes, f32)
    assert want > 0 and hcmix.decode_cache_bytes(4, 256, 64, kind(codes), f32) == want


def test_layer_codes_of_a_range_and_of_the_local_layer():
    assert np.frombuffer(hcmix._layers(range(7)), dtype=np.int32).tolist() == list(range(7))
    codes = [hcmix.LAYER_NEAR, 3, 2 ** 40 + 1]      # the last one wraps, as in a C int
    assert np.frombuffer(hcmix._layers(codes), dtype=np.int32).tolist() == [-1, 3, 1]


@pytest.mark.gpu
def test_the_stream_is_the_current_one():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.zeros(1, device="cuda:0")
    side = torch.cuda.Stream()
    assert hcmix._stream(x) == torch.cuda.current_stream(x.device).cuda_stream
    with torch.cuda.stream(side):
        assert hcmix._stream(x) == side.cuda_stream != 0


@pytest.mark.gpu
def test_addresses_of_matching_tensors_only():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a = torch.zeros(4, 6, device="cuda:0")
    p = torch.nn.Parameter(torch.zeros(4, 6, device="cuda:0"))
    got = call((a, p), 2, (4, 6), dev="cuda:0")
    assert memoryview(got).cast("P").tolist() == [a.data_ptr(), p.data_ptr()]
    assert call([a, p], 1, (4, 6), dev="cuda:0") == got[:8]
    for bad in (a.t(), a[:, :3], a.to(bf), a.cpu(), torch.zeros(4, 7, device="cuda:0"),
                torch.zeros(4, 6, 1, device="cuda:0"), None, 3):
        assert call([a, bad], 2, (4, 6), dev="cuda:0") is None
    assert call([a.t()], 1, (6, 4), dev="cuda:0") is None     # not contiguous
