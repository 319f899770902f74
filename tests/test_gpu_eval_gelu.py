"""The validation step leaves GELU's derivative out where its product's kernel can: the same loss as the training step's, to the bit, in every
tile class that has a flavour for it."""
import pytest
import torch

import paper_2204_06514_amd as fax
from helpers import DEV, dims_of
from test_gpu_train import run_train_step, _dev_params
from workloads import BlockShape, ModelShape, make_model_inputs

pytestmark = pytest.mark.gpu
WHOLE, EDGE = fax.FAX_GEMM_MFMA, fax.FAX_GEMM_EDGE


ROUTES = [(32, 256, 256, 4096, (WHOLE, 256, 256)), (32, 128, 512, 2048, (WHOLE, 256, 128)), (32, 128, 256, 1024, (WHOLE, 128, 128)),
          (30, 100, 1200, 4800, (EDGE, 256, 256)), (28, 111, 512, 2048, (EDGE, 256, 128)), (30, 100, 1200, 1200, (EDGE, 128, 128)),
          (16, 128, 256, 1024, (fax.FAX_GEMM_SMALL, 128, 64))]


@pytest.mark.parametrize("B,S,D,F,route", ROUTES)
@pytest.mark.parametrize("gelu", ["tanh", "erf"])
def test_eval_loss_is_the_training_loss(B, S, D, F, route, gelu):
    ms = ModelShape(BlockShape(B=B, S=S, D=D, H=D // 8, dh=8, F=F, dtype="bf16", sigma_w=0.05, L=2, gelu=gelu), V=264, S_max=S)
    sh = ms.blk
    r = fax.fax_gemm_route(fax.FAX_BF16, 0, 0, sh.T, F, D)
    assert (r.form, r.tile_m, r.tile_n) == route
    p, tok, lab = make_model_inputs(ms, seed=2, generic=True)
    loss = run_train_step(ms, p, tok, lab, update=False)[0]
    md = fax.FaxModelDims(dims_of(sh), sh.L, ms.V, S, 0)
    wsb = fax.fax_eval_workspace_bytes(md)
    ws = torch.full((wsb,), 255, dtype=torch.uint8, device=DEV)   # NaN wherever a kernel reads what none has written
    out = torch.zeros(4, device=DEV)
    fax.fax_eval_step(md, _dev_params(p, "bf16"), torch.from_numpy(tok).to(DEV), torch.from_numpy(lab).to(DEV), out, ws, wsb)
    assert out[0].item() == loss
