"""The weight gradients of a layer and the input gradient of its QKV projection in one launch, or side by side on two streams: whole and
masked tiles, both tile widths of the input gradient, gradients added onto given ones, against float64 products of the tensors that the pass itself
left, and one and two streams bit for bit."""
import pytest
import torch

import helpers
import paper_2204_06514_amd as fax
from helpers import DEV, dims_of, view_bytes
from workloads import BlockShape

pytestmark = pytest.mark.gpu

# streams, and which tile the input gradient takes on the CUs left over
SHAPES = [
    (BlockShape(B=2, S=1024, D=1024, H=16, dh=64, F=4096, dtype="bf16", sigma_w=0.02), 1),   # 192 weight-gradient tiles, 64 CUs for 32 tiles
    (BlockShape(B=4, S=1024, D=2048, H=8, dh=64, F=2048, dtype="bf16", sigma_w=0.02), 2),    # a tensor-parallel share, 64 CUs for 128 tiles
    (BlockShape(B=3, S=2048, D=1024, H=16, dh=64, F=4096, dtype="bf16", sigma_w=0.02), 2),
    (BlockShape(B=5, S=1111, D=1000, H=10, dh=96, F=4000, dtype="bf16", sigma_w=0.02), 2),   # nothing a multiple of the tile
    (BlockShape(B=7, S=146, D=1000, H=10, dh=64, F=4000, dtype="bf16", sigma_w=0.02), 1),    # 172 tiles: no multiple of the XCDs
    (BlockShape(B=11, S=512, D=1024, H=1, dh=128, F=4096, dtype="bf16", sigma_w=0.02), 2),   # 140
    (BlockShape(B=28, S=384, D=896, H=7, dh=128, F=10752, dtype="bf16", sigma_w=0.02), 2),   # 396 tiles: two rounds on 200 CUs
    (BlockShape(B=12, S=512, D=2176, H=11, dh=128, F=8704, dtype="bf16", sigma_w=0.02), 2),  # 819 tiles: four on 208
]
SEVERAL_ROUNDS = (6, 7)


class _Pass:
    def __init__(self, sh, seed):
        self.sh = sh
        g = torch.Generator(device=DEV).manual_seed(seed)
        rnd = lambda shape, s: (s * torch.randn(shape, generator=g, device=DEV)).bfloat16()  # noqa: E731
        D, Hd, F = sh.D, sh.Hd, sh.F
        self.shapes = dict(ln1_g=(D,), ln1_b=(D,), wqkv=(D, 3 * Hd), bqkv=(3 * Hd,), wo=(Hd, D), bo=(D,), ln2_g=(D,), ln2_b=(D,), w1=(D, F),
                           b1=(F,), w2=(F, D), b2=(D,))
        self.p = {k: rnd(v, 1.0 if k.endswith("_g") else 0.02) for k, v in self.shapes.items()}
        self.x, self.dy = rnd((sh.T, D), 1.0), rnd((sh.T, D), 1.0)
        self.lay = fax.fax_block_saved_layout(dims_of(sh))
        self.saved = torch.empty(self.lay.total, dtype=torch.uint8, device=DEV)
        self.wsb = fax.fax_block_workspace_bytes(dims_of(sh))
        self.ws, y = torch.empty(self.wsb, dtype=torch.uint8, device=DEV), torch.empty_like(self.x)
        fax.fax_block_fwd(dims_of(sh), self.p, self.x, y, self.saved, None, None, self.ws, self.wsb)

    def backward(self, flags=0, accumulate=0, over=False, dh1=None):
        dy = self.dy.clone()
        out = {k: torch.full(v, 0.5, dtype=torch.float32, device=DEV) for k, v in self.shapes.items()}
        out["dx"] = dy if over else torch.empty_like(dy)
        self.ws.fill_(255)
        fax.fax_block_bwd(dims_of(self.sh, flags), self.p, self.x, dy, self.saved, out["dx"], out, accumulate, dy if dh1 == "dy" else None, None, self.ws, self.wsb)
        torch.cuda.synchronize()
        return out

    def left(self, buf, offset, cols):
        return view_bytes(buf, offset, (self.sh.T, cols), torch.bfloat16).double()


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_products(i, accumulate):
    sh, streams = SHAPES[i]
    assert fax.fax_block_bwd_streams(dims_of(sh)) == streams
    _check_products(sh, i, 0, accumulate)


@pytest.mark.parametrize("i", SEVERAL_ROUNDS)
def test_products_of_several_rounds_on_one_stream(i):
    _check_products(SHAPES[i][0], i, fax.FAX_FLAG_SINGLE_STREAM, 1)


def _check_products(sh, seed, flags, accumulate):
    s = _Pass(sh, seed)
    got = s.backward(flags, accumulate=accumulate)
    bl, D, Hd, F = fax.fax_block_bwd_layout(dims_of(sh)), sh.D, sh.Hd, sh.F
    dqkv, dx1, du = s.left(s.ws, bl.dqkv, 3 * Hd), s.left(s.ws, bl.dx1, D), s.left(s.ws, bl.du, F)
    dh1 = s.left(s.ws, bl.dh1, D)
    ref = dqkv @ s.p["wqkv"].double().t()
    assert (dh1 - ref).norm() <= 4e-3 * ref.norm()  # one rounding to bf16
    assert ((dh1 - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4 * ref.abs().max()).all()
    for k, act, grad in (("w2", s.left(s.saved, s.lay.a, F), s.dy.double()), ("w1", s.left(s.saved, s.lay.h2, D), du),
                         ("wo", s.left(s.saved, s.lay.ctx, Hd), dx1), ("wqkv", s.left(s.saved, s.lay.h1, D), dqkv)):
        for name, ref in ((k, act.t() @ grad), ("b" + k[1:], grad.sum(0))):
            ref = ref + 0.5 * accumulate
            if name == "bqkv":  # the key third is a sum of what cancels
                scale = ref.abs().max()
                assert ((got[name].double() - ref).abs() <= 1e-5 * scale).all(), name
            else:
                assert (got[name].double() - ref).abs().max() <= 1e-5 * ref.abs().max(), name


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_same_bits_on_one_and_two_streams_and_over_dy(i):
    sh, _ = SHAPES[i]
    s = _Pass(sh, 10 + i)
    want = s.backward(fax.FAX_FLAG_SINGLE_STREAM)
    for flags, over, dh1 in ((0, False, None), (0, True, None), (fax.FAX_FLAG_SINGLE_STREAM, True, None), (fax.FAX_FLAG_SINGLE_STREAM, False, "dy")):
        got = s.backward(flags, over=over, dh1=dh1)
        # dh1 over dy, which a weight gradient reads: not in one launch then, and on tiles that may add up in another order
        for k in ("w1", "b1", "w2", "b2", "wo", "bo", "wqkv", "bqkv") if dh1 else want:
            assert torch.equal(got[k], want[k]), (k, flags, over, dh1)


# dh1 may take dy's place on two streams too; attention's two weight gradients together or apart besides the shapes above
@pytest.mark.parametrize("sh", [s for s, streams in SHAPES if streams == 2] + [
    BlockShape(B=4, S=777, D=512, H=8, dh=64, F=2048, dtype="bf16", sigma_w=0.02), BlockShape(B=8, S=512, D=1024, H=16, dh=64, F=4096, dtype="bf16", sigma_w=0.02)])
def test_dh1_over_dy_on_two_streams(sh):
    assert fax.fax_block_bwd_streams(dims_of(sh)) == 2
    s = _Pass(sh, 30)
    want, got = s.backward(fax.FAX_FLAG_SINGLE_STREAM, dh1="dy"), s.backward(0, dh1="dy")
    for k in want:
        assert torch.equal(got[k], want[k]), k


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_launches(i):
    """One launch of all weight gradients; on one stream it does the input gradient's work too, on two that has a launch on the CUs left over."""
    sh, streams = SHAPES[i]
    s = _Pass(sh, 20 + i)
    fax.fax_timing_enable(1)
    try:
        s.backward()
        rows = {r["name"]: (r["launches"], r["work"]) for r in fax.fax_timing_report(64)}
    finally:
        fax.fax_timing_enable(0)
    assert not any("f32out" in r for r in rows), rows
    n, work = rows.get("gemm_mfma_group_input", (0, 0))
    assert (n, work) == (streams - 1, (streams - 1) * 6.0 * sh.T * sh.D * sh.Hd)
    n, work = rows["gemm_mfma_group"]
    want = 2.0 * sh.T * sh.D * (4 * sh.Hd + 2 * sh.F + (3 * sh.Hd if streams == 1 else 0))
    assert n == 1 and abs(work - want) <= 1e-6 * want
