"""fp32 stacks and bf16 widths that are no multiple of 64: the matrix-core tiles'
edges (a width just below, at and above a tile, odd fp32 widths on the scalar
loads), row counts that split the weight-gradient sums, and the backward on the
whole and on the least workspace, against the CPU oracle.

Tolerances: those of the other parity tests for the activations; weight
gradients of a single layer see no rounding below fp32, so 1e-5 (fp32) and 1e-4
(bf16 operands, whose products are exact in fp32) bound the order of the sums."""
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


@pytest.mark.parametrize("batch,n,width,dtype,layer", [
    (3, 16, 1, "f32", 1), (1, 2, 33, "f32", 0), (3, 32, 63, "f32", 2), (2, 32, 68, "f32", -1),
    (5, 64, 129, "f32", 5), (1, 512, 100, "f32", -1), (2, 64, 256, "f32", 3),
    (3, 32, 56, "bf16", 0), (2, 64, 120, "bf16", 5), (1, 512, 136, "bf16", 8),
    (3, 64, 200, "bf16", -1), (5, 64, 264, "bf16", 2), (1, 2, 72, "bf16", 0)])
@pytest.mark.parametrize("causal", [False, True])
def test_layer(batch, n, width, dtype, layer, causal):
    if layer < 0 and not causal:
        pytest.skip("the local layer is causal")
    print(f"case: layer {batch}x{n}x{width} {dtype} layer={layer} causal={causal}", flush=True)
    code, ref = (hcmix.LAYER_NEAR, oracle.NEAR) if layer < 0 else (layer, layer)
    x, ws, wo, dy = inputs.make_layer(batch, n, width, dtype, seed=width + n)
    tx, tws, two, tdy = (to_dev(a, dtype) for a in (x, ws, wo, dy))
    y = hcmix.forward(tx, tws, two, code, causal)
    dx, dws, dwo = hcmix.backward(tx, tws, two, tdy, code, causal)
    torch.cuda.synchronize()
    ry = oracle.forward(x, ws, wo, ref, causal)
    rdx, rws, rwo = oracle.backward(x, ws, wo, dy, ref, causal)
    assert row_rel_err(to_host(y), ry) <= TOL[dtype]
    assert row_rel_err(to_host(dx), rdx) <= TOL[dtype]
    tol = 1e-5 if dtype == "f32" else 1e-4
    assert fro_rel_err(to_host(dws), rws) <= tol and fro_rel_err(to_host(dwo), rwo) <= tol


def test_misaligned_fp32_tensors():
    """fp32 operands need only 4-byte alignment: the scalar loads."""
    batch, n, width = 2, 32, 64
    x, ws, wo, dy = inputs.make_layer(batch, n, width, "f32", seed=4)

    def off(a):
        t = to_dev(a, "f32")
        buf = torch.zeros(t.numel() + 1, device="cuda")
        v = buf[1:].view(t.shape)
        v.copy_(t)
        return v

    tx, tws, two, tdy = (off(a) for a in (x, ws, wo, dy))
    y = hcmix.forward(tx, tws, two, 2, True)
    dx, dws, dwo = hcmix.backward(tx, tws, two, tdy, 2, True)
    torch.cuda.synchronize()
    ry = oracle.forward(x, ws, wo, 2, True)
    rdx, rws, rwo = oracle.backward(x, ws, wo, dy, 2, True)
    assert row_rel_err(to_host(y), ry) <= 1e-5 and row_rel_err(to_host(dx), rdx) <= 1e-5
    assert fro_rel_err(to_host(dws), rws) <= 1e-5 and fro_rel_err(to_host(dwo), rwo) <= 1e-5


@pytest.mark.parametrize("batch,n,width,dtype,schedule", [
    (17, 64, 33, "f32", [0, 1, 2, 5]),          # two row ranges, the second ragged
    (8, 256, 64, "f32", [7, -1, 0]),            # four, a local layer among them
    (17, 64, 72, "bf16", [0, 3, 5, -1]),
    (8, 256, 136, "bf16", [7, 1])])
def test_stack_backward_with_whole_and_least_workspace(batch, n, width, dtype, schedule):
    print(f"case: stack {batch}x{n}x{width} {dtype} {schedule}", flush=True)
    L = len(schedule)
    codes = [hcmix.LAYER_NEAR if v < 0 else v for v in schedule]
    refs = [oracle.NEAR if v < 0 else v for v in schedule]
    s = inputs.make_stack(batch, n, width, L, True, dtype, seed=width, layers=refs)
    ws, wo = ([to_dev(w, dtype) for w in m] for m in (s.w_self, s.w_off))
    x, dy = to_dev(s.x, dtype), to_dev(s.dy, dtype)
    xs = hcmix.stack_forward(x, ws, wo, codes, True)
    whole = hcmix.stack_workspace_bytes(batch, n, width, L, x.dtype)
    act = (x.numel() * x.element_size() + 255) // 256 * 256
    assert whole > 2 * act                       # partial sums: the rows are split
    base = [torch.full((width, width), 0.5, device="cuda") for _ in range(2 * L)]
    got = []
    for nbytes in (whole, 2 * act):
        wsp = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        acc = [t.clone() for t in base]
        dx, _, _ = hcmix.stack_backward(xs, ws, wo, codes, dy, True, dws=acc[:L], dwo=acc[L:],
                                        accumulate=True, workspace=wsp)
        got.append((dx, acc))
    again = hcmix.stack_backward(xs, ws, wo, codes, dy, True)
    _, grads = hcmix.stack_backward_data(ws, wo, codes, dy, True)
    apart = hcmix.stack_weight_gradients(xs[:L], [*grads, dy], codes, True)
    torch.cuda.synchronize()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][0], again[0])
    for a, b in zip(again[1] + again[2], apart[0] + apart[1]):
        assert torch.equal(a, b)
    ref = oracle.stack_forward(s.x, s.w_self, s.w_off, refs, True)
    rdx, rws, rwo = oracle.stack_backward(ref, s.w_self, s.w_off, refs, s.dy, True)
    assert row_rel_err(to_host(xs[-1]), ref[-1]) <= TOL[dtype]
    assert row_rel_err(to_host(got[0][0]), rdx) <= TOL[dtype]
    for _, acc in got:
        for g, r in zip(acc, rws + rwo):
            assert fro_rel_err(to_host(g) - 0.5, r) <= TOL[dtype]


def _near(codes):
    return [hcmix.LAYER_NEAR if v == oracle.NEAR else v for v in codes]


@pytest.mark.parametrize("batch,n,width,layers,causal", [
    (5, 16, 129, 24, True),       # 80 rows (a ragged slice), scalar loads, ragged second tile
    (5, 16, 132, 24, False),      # the same by 16 bytes
    (17, 64, 129, 13, True),      # two row ranges, the second shorter
    (17, 64, 256, 12, False),     # whole tiles
    (5, 16, 65, 96, True)])       # 64 x 64 tiles again, in launches of 64 and 32 layers
@pytest.mark.parametrize("accumulate", [False, True])
def test_fp32_weight_gradients_on_128_tiles(batch, n, width, layers, causal, accumulate):
    """Stacks that have 192 blocks of 128 x 128 outputs (layers x row ranges x two
    matrices x tiles): those tiles, as against 64 x 64 below."""
    rows, te, batched = batch * n, -(-width // 128), min(layers, 64)
    splits = max(1, min(-(-512 // (batched * 2 * te * te)), rows // 512))
    assert width > 64 and (batched * splits * 2 * te * te >= 192) == (layers < 96)
    print(f"case: fp32 dW {rows}x{width} L={layers} causal={causal} splits={splits}", flush=True)
    codes = [v % (n.bit_length() - 1) for v in range(layers)]
    if causal:
        codes[3] = codes[layers - 2] = oracle.NEAR
    rng = np.random.default_rng(width)
    xs, dys = (rng.standard_normal((layers, batch, n, width)).astype(np.float32) for _ in "xg")
    zero = np.zeros((width, width), dtype=np.float32)
    start = 0.5 if accumulate else 7.0
    dws, dwo = ([torch.full((width, width), start, device="cuda") for _ in codes] for _ in "so")
    hcmix.stack_weight_gradients([to_dev(x, "f32") for x in xs], [to_dev(g, "f32") for g in dys],
                                 _near(codes), causal, dws=dws, dwo=dwo, accumulate=accumulate)
    torch.cuda.synchronize()
    for l, code in enumerate(codes):
        _, rws, rwo = oracle.backward(xs[l], zero, zero, dys[l], code, causal)
        for got, ref in ((dws[l], rws), (dwo[l], rwo)):
            assert fro_rel_err(to_host(got) - (start if accumulate else 0.0), ref) <= 1e-5


@pytest.mark.parametrize("batch,n,width,dtype,layers", [
    (3, 32, 20, "f32", 66), (3, 32, 33, "f32", 130), (17, 64, 72, "bf16", 66)])
def test_stack_backward_of_more_layers_than_a_launch_takes(batch, n, width, dtype, layers):
    """Chunks of 64 layers' weight gradients, the ring of gradient buffers reused
    from chunk to chunk: the same sums as the data chain with every gradient
    kept, and the oracle's."""
    print(f"case: ring {batch}x{n}x{width} {dtype} L={layers}", flush=True)
    codes = [v % (n.bit_length() - 1) for v in range(layers)]
    codes[2] = codes[65] = oracle.NEAR
    s = inputs.make_stack(batch, n, width, layers, True, dtype, seed=layers, layers=codes)
    ws, wo = ([to_dev(w, dtype) for w in m] for m in (s.w_self, s.w_off))
    x, dy = to_dev(s.x, dtype), to_dev(s.dy, dtype)
    xs = hcmix.stack_forward(x, ws, wo, _near(codes), True)
    dx, dws, dwo = hcmix.stack_backward(xs, ws, wo, _near(codes), dy, True)
    dx2, grads = hcmix.stack_backward_data(ws, wo, _near(codes), dy, True)
    aws, awo = hcmix.stack_weight_gradients(xs[:layers], [*grads, dy], _near(codes), True)
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2)
    for a, b in zip(dws + dwo, aws + awo):
        assert torch.equal(a, b)
    # each layer's products alone, from the operands that the launch was given
    tol = 1e-5 if dtype == "f32" else 1e-4
    for l in (0, 1, 2, 63, 64, 65, layers - 1):
        g = to_host(dy if l == layers - 1 else grads[l])
        _, rws, rwo = oracle.backward(to_host(xs[l]), s.w_self[l], s.w_off[l], g, codes[l], True)
        assert fro_rel_err(to_host(dws[l]), rws) <= tol
        assert fro_rel_err(to_host(dwo[l]), rwo) <= tol


@pytest.mark.parametrize("batch,width,dtype,off", [
    (17, 1, "f32", 0), (5, 33, "f32", 0), (16, 64, "f32", 0), (3, 64, "f32", 1), (18, 272, "f32", 0),
    (17, 40, "bf16", 0), (3, 264, "bf16", 0)])
def test_decode(batch, width, dtype, off):
    """Widths off the kernel's steps and columns, and 4-byte aligned fp32 (off)."""
    n, codes, refs = 8, [0, 2, hcmix.LAYER_NEAR, 1], [0, 2, oracle.NEAR, 1]
    s = inputs.make_stack(batch, n, width, 4, True, dtype, seed=width, layers=refs, with_dy=False)
    want = oracle.stack_forward(s.x, s.w_self, s.w_off, refs, True)[-1]

    def dev(a):
        t = to_dev(np.ascontiguousarray(a), dtype)
        buf = torch.zeros(t.numel() + off, dtype=t.dtype, device="cuda")
        v = buf[off:].view(t.shape)
        v.copy_(t)
        return v

    ws, wo = ([dev(w) for w in m] for m in (s.w_self, s.w_off))
    cache = hcmix.alloc_decode_cache(batch, n, width, codes, ws[0].dtype, ws[0].device)
    cache.fill_(0xFF)
    got = np.stack([to_host(hcmix.decode_step(dev(s.x[:, pos]), ws, wo, codes, n, pos, cache))
                    for pos in range(n)], 1)
    # (four bf16 roundings of rows of 40 values: two thirds of the tolerance)
    assert row_rel_err(got, want) <= TOL[dtype]
