"""GPU parity at the edges of the kernels that take any shape: sizes that are no multiple of a tile, the
smallest and the largest of a range, and the borders between two kernels of a dispatch."""
import numpy as np
import pytest
import torch

import als_inputs as I
import paper_2401_09135_amd as A
from oracle import lm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def _model(**kw):
    w = I.workload("tiny")
    w.update(dict(L=1, d=64, h=2, ff=64, V=64, S=8, B=2, dtype="f32"), **kw)
    return w


def _loss_grad(w, tok, flags=0):
    theta0 = I.theta0(lm.param_layout(w), w["seed"])
    ctx = A.Context(A.Config.from_workload(w, flags=flags), theta0, n_streams=1)
    loss, g = ctx.worker_loss_grad(0, torch.from_numpy(tok).to(DEV))
    ctx.close()
    return theta0, loss, g


@pytest.mark.parametrize("V,B,S", [(2, 1, 3),           # one bit
                                   (256, 3, 40), (257, 3, 40),        # one digit of 8 bits, two
                                   (4095, 2, 70), (4096, 2, 70),      # V + 1 entries in one and in two blocks of 4096
                                   (65537, 1, 65),                    # three digits
                                   (300, 17, 1000)])                  # more than one tile of 16384 positions
def test_token_order_of_the_embedding_gradient(V, B, S):
    """dE sums dx over the sorted position list of every token: a position out of place or missing
    puts a whole row of dx into the wrong sum.  fp32 mode, so the bound is that of the sums."""
    w = _model(V=V, B=B, S=S)
    tok = I.TokenStream(1, 0, B, S, V).take(1)[0]
    theta0, loss, g = _loss_grad(w, tok)
    rloss, rg = lm.loss_and_grad(theta0, tok, w)
    assert abs(loss - rloss) < 1e-5 * abs(rloss)
    assert _rel(lm.views(g, w)["E"], lm.views(rg, w)["E"]) < 1e-5
