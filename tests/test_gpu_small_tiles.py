"""Every block shape of the mixing, local and linear products (few rows to
many), at its tiles' edges: row counts that leave a tile ragged, widths of an
odd number of 64-column tiles, weights read as given and transposed.  Against
the CPU oracle (the linear maps against their definition)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_18145_amd import hcmix, inputs
from tests.util import TOL, fro_rel_err, row_rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    hcmix.load()


# (batch, n, width): small, mid and big blocks of both kinds of width
SHAPES = [(3, 2, 64), (35, 2, 448), (3, 256, 512), (33, 64, 512), (63, 64, 512), (129, 64, 512),
          (33, 128, 192), (65, 256, 192), (1, 1024, 1024), (5, 512, 1024), (9, 1024, 1024),
          (33, 64, 200), (130, 64, 328), (128, 64, 200), (512, 64, 136)]


def tile(rows, width, transposed):
    """The block shape of a hypercube layer's product (rows / 2 pairs; the local
    layer's counts are the same), and whether the width is ragged in it."""
    pairs, wide = rows // 2, -(-width // 64) % 2 == 0
    big = 256 if not transposed and width % 256 == 0 and width >= 1024 else 128 if wide else 64

    def blocks(p, c):
        return -(-pairs // p) * -(-width // c)

    if blocks(32, 64 if transposed else 32) <= (256 if transposed else 512):
        kind = "small"
    else:
        mid, large = (-(-b // 256) for b in (blocks(64, 64), blocks(128, big)))
        kind = "mid" if mid * 4 <= large * {256: 14, 128: 7, 64: 5}[big] else f"big{big}"
    return kind, width % 64 != 0


def test_the_shapes_reach_every_block():
    got = {(*tile(b * n, w, t), t) for b, n, w in SHAPES for t in (False, True)}
    for ragged in (False, True):
        for kind in ("small", "mid", "big64", "big128"):
            assert (kind, ragged, False) in got and (kind, ragged, True) in got, (kind, ragged)
    assert ("big256", False, False) in got


@pytest.mark.parametrize("batch,n,width", SHAPES)
@pytest.mark.parametrize("layer", [0, 5, -1])
def test_layer_and_stack_dx(batch, n, width, layer):
    print(f"case: {batch}x{n}x{width} layer={layer}", flush=True)
    code, ref = (hcmix.LAYER_NEAR, oracle.NEAR) if layer < 0 else (layer, layer)
    x, ws, wo, dy = inputs.make_layer(batch, n, width, "bf16", seed=width + n)
    tx, tws, two, tdy = (to_dev(a, "bf16") for a in (x, ws, wo, dy))
    y = hcmix.forward(tx, tws, two, code, True)
    dx, dws, dwo = hcmix.backward(tx, tws, two, tdy, code, True)
    # a two-layer data chain: the same products on transposed copies
    dx2, grads = hcmix.stack_backward_data([tws] * 2, [two] * 2, [code] * 2, tdy, True)
    torch.cuda.synchronize()
    ry = oracle.forward(x, ws, wo, ref, True)
    rdx, rws, rwo = oracle.backward(x, ws, wo, dy, ref, True)
    assert row_rel_err(to_host(y), ry) <= TOL["bf16"]
    assert row_rel_err(to_host(dx), rdx) <= TOL["bf16"]
    assert row_rel_err(to_host(grads[0]), rdx) <= TOL["bf16"]
    assert fro_rel_err(to_host(dws), rws) <= 1e-4 and fro_rel_err(to_host(dwo), rwo) <= 1e-4


@pytest.mark.parametrize("rows,n_in,n_out", [(2, 64, 64), (70, 128, 448), (770, 512, 1536),
                                             (2050, 512, 512), (4098, 192, 512),
                                             (8200, 512, 192)])
def test_linear(rows, n_in, n_out):
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn(rows, n_in, generator=g, device="cuda").bfloat16()
    w = (torch.randn(n_out, n_in, generator=g, device="cuda") * n_in ** -0.5).bfloat16()
    dy = torch.randn(rows, n_out, generator=g, device="cuda").bfloat16()
    y = hcmix.linear_forward(x, w)
    dx, dw = hcmix.linear_backward(x, w, dy)
    torch.cuda.synchronize()
    xd, wd, gd = (t.double().cpu().numpy() for t in (x, w, dy))
    assert row_rel_err(to_host(y), xd @ wd.T) <= TOL["bf16"]
    assert row_rel_err(to_host(dx), gd @ wd) <= TOL["bf16"]
    assert fro_rel_err(to_host(dw), gd.T @ xd) <= 1e-4


@pytest.mark.parametrize("rows,n_in,n_out", [(64, 64, 128), (130, 192, 320), (8192, 128, 96 * 2),
                                             (4098, 512, 1536)])
def test_linear_weight_gradient_on_whole_and_least_workspace(rows, n_in, n_out):
    """Row ranges of the whole plan and of the least workspace (as many partials
    as 128 x 128 tiles need to make 256 blocks), ragged last ranges among them."""
    print(f"case: linear dW {rows}x{n_in}x{n_out}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn(rows, n_in, generator=g, device="cuda").bfloat16()
    w = torch.zeros(n_out, n_in, device="cuda").bfloat16()
    dy = torch.randn(rows, n_out, generator=g, device="cuda").bfloat16()
    tiles = -(-n_out // 128) * -(-n_in // 128)
    steps = -(-rows // 64)
    s = max(1, min(-(-256 // tiles), steps))
    least = -(-steps // -(-steps // s)) * n_in * n_out * 4
    ref = dy.double().cpu().numpy().T @ x.double().cpu().numpy()
    whole = hcmix.load().hcmix_linear_backward_workspace_bytes(rows, n_in, n_out)
    assert whole >= least
    for nbytes in (whole, least):
        wsp = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        dw = torch.full((n_out, n_in), 0.25, device="cuda")
        hcmix.linear_backward(x, w, dy, dw=dw, with_dx=False, accumulate=True, workspace=wsp)
        torch.cuda.synchronize()
        assert fro_rel_err(to_host(dw) - 0.25, ref) <= 1e-4
