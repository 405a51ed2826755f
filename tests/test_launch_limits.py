"""A launch takes fewer than 2^32 threads along each axis of its grid.  The largest
calls whose operands the card's 288 GB hold, through the C ABI with the
runtime's launch calls recorded (launch_recorder.c): every grid has to fit, and
the launches together have to cover the call."""
import json
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

# runs in a process of its own, which must not have loaded the real runtime's
# symbols first: the recorder's take precedence in the order of loading
CHILD = """
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
class Launch(ctypes.Structure):
    _fields_ = [("grid", ctypes.c_uint32 * 3), ("block", ctypes.c_uint32 * 3),
                ("arg", ctypes.c_uint64 * 2)]
out = []
for name, args in json.loads(sys.argv[3]):
    conv, keep = [], []
    for kind, v in args:      # operands: addresses, lists of them, a schedule
        if kind in ("ptrs", "codes"):
            v = ((ctypes.c_void_p if kind == "ptrs" else ctypes.c_int32) * len(v))(*v)
            keep.append(v)
            conv.append(v)
        else:
            conv.append(getattr(ctypes, "c_" + kind)(v))
    ctypes.c_int.in_dll(rec, "launch_count").value = 0
    status = getattr(lib, name)(*conv)
    n = ctypes.c_int.in_dll(rec, "launch_count").value
    ls = (Launch * 64).in_dll(rec, "launches")
    out.append([status, [[list(l.grid), list(l.block), l.arg[0]] for l in ls[:n]]])
print(json.dumps(out))
"""


def i64(*v):
    return [["int64", e] for e in v]


def i32(*v):
    return [["int32", e] for e in v]


def mem(k):
    """An operand's address: 1 TiB apart, nothing is behind it."""
    return ["void_p", (1 << 44) + (k << 40)]


NONE = ["void_p", None]


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    from paper_2609_18145_amd import hcmix
    rec = str(tmp_path_factory.mktemp("rec") / "recorder.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-std=c11",
                           os.path.join(HERE, "launch_recorder.c"), "-o", rec])

    def run(name, args):
        res = subprocess.run([sys.executable, "-c", CHILD, rec, hcmix.LIB_PATH,
                              json.dumps([[name, args]])], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        status, ls = json.loads(res.stdout.splitlines()[-1])[0]
        assert status == 0 and 0 < len(ls) <= 64, (status, len(ls))
        for grid, block, _ in ls:
            assert all(g * b < 1 << 32 for g, b in zip(grid, block)), (grid, block)
        return ls
    return run


@pytest.mark.parametrize("rows", [(1 << 29) - 512, 1 << 29, (1 << 30) - 512, 1 << 30])
@pytest.mark.parametrize("layer", [3, -1])
def test_fp32_layer(launches, rows, layer):
    ls = launches("hcmix_forward", i64(rows // 512, 512, 1) + i32(layer, 1, 0)
                  + [mem(0), mem(1), mem(2), mem(3), NONE])
    assert len(ls) == 1
    (x, y, z), _, _ = ls[0]
    assert y == 1 and x * z * 64 >= rows > (x - 1) * z * 64


@pytest.mark.parametrize("rows,n_in,n_out", [((1 << 21) - 2, 64, 1 << 16), (1 << 21, 64, 1 << 16),
                                             (27692708, 192, 5120), (1 << 30, 64, 64)])
def test_linear_map(launches, rows, n_in, n_out):
    """Outputs of just under 2^37 elements (256 GiB), of those and of more."""
    ls = launches("hcmix_linear_forward",
                  i64(rows, n_in, n_out) + [mem(0), mem(1), mem(2), NONE])
    assert len(ls) == 1
    (x, _, _), (threads, _, _), _ = ls[0]
    tile = {512: (128, 128), 256: (256, 64)}[threads]     # rows and columns of a block
    assert x == -(-rows // tile[0]) * (n_out // tile[1])
    # the input's gradient is the same product with the widths exchanged
    ls = launches("hcmix_linear_backward",
                  i64(rows, n_out, n_in) + [mem(0), mem(1), mem(2), mem(3), NONE] + i32(0)
                  + [NONE, ["size_t", 0], NONE])
    assert len(ls) == 1 and ls[0][0][0] == x


@pytest.mark.parametrize("batch,width,dtype", [((1 << 23) - 1, 64, 1), (1 << 23, 64, 1),
                                               (1 << 23, 32, 0), (933054, 576, 1),
                                               (1 << 22, 128, 1)])
def test_channel_shared_forward(launches, batch, width, dtype):
    """Windows of 128 positions, 128 GiB per tensor: launches that start where the
    one before ended and cover every window and slice of channels."""
    n, es, slices = 128, 2 if dtype else 4, width // (64 if dtype else 32)
    ls = launches("hcmix_shared_stack_forward",
                  i64(batch, n, width) + i32(1) + [["codes", [0]]] + i32(1, dtype)
                  + [mem(0), ["ptrs", [mem(1)[1]]], ["ptrs", [mem(2)[1]]], NONE])
    assert (len(ls) == 1) == (batch * slices * 512 < 1 << 32)
    done = 0
    for (x, _, _), _, x0 in ls:
        assert x % slices == 0 and x0 == mem(0)[1] + done * n * width * es
        done += x // slices
    assert done == batch


@pytest.mark.parametrize("rows,n_in,n_out,tile", [
    (2, 64, 64, 128), (512, 512, 512, 128), (8192, 256, 512, 128), (8192, 512, 512, 128),
    (2048, 512, 1536, 128), (8192, 512, 1536, 256), (32768, 512, 512, 256),
    (16384, 8192, 8192, 256), (1 << 20, 64, 64, 128)])
def test_weight_gradient_plan(launches, rows, n_in, n_out, tile):
    """The tile that was measured to be the faster, ranges that fit the workspace
    that the query answers, one round of blocks unless the tiles alone are more."""
    from paper_2609_18145_amd import hcmix
    nbytes = hcmix.load().hcmix_linear_backward_workspace_bytes(rows, n_in, n_out)
    ls = launches("hcmix_linear_backward",
                  i64(rows, n_in, n_out) + [mem(0), mem(1), mem(2), NONE, mem(3)] + i32(0)
                  + [mem(4), ["size_t", nbytes], NONE])
    (blocks, _, _), (threads, _, _), _ = ls[0]
    assert len(ls) == 2 and threads == 2 * tile           # the gradient, the sum of the ranges
    tiles = -(-n_out // tile) * -(-n_in // 128)
    assert blocks % tiles == 0
    splits = blocks // tiles
    assert blocks <= max(256, tiles) and splits <= -(-rows // 64)
    assert splits * n_in * n_out * 4 <= nbytes
