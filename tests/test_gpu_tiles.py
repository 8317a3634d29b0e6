"""The tile walk's 32-row tiles run on across slice boundaries: whatever the
slice length, a call gives the same bits (no dropout, whose masks are the only
thing that depends on it), outputs, state and gradients, over one segment and
several; with dropout the masks keep following the slices (against the oracle
at slice lengths on both sides of a tile)."""

import pytest
import torch

import oracle as O
from synth import Workload, make_inputs
from tests.gpu_common import TOL, dev, host64, need_gpu, report

pytestmark = pytest.mark.gpu

# L, d, M, dtype, kind, segments forced (0: the library's plan)
CASES = [
    (131, 64, 256, "bf16", "favor+", 0),
    (200, 64, 256, "bf16", "favor+", 3),
    (97, 32, 64, "bf16", "relu", 2),
    (161, 64, 64, "f32", "favor+", 2),
]


def _run(x, C, kind, dropout=0.0):
    from paper_2012_11346_amd import slim

    Q, K, V, dY, W = (dev(x[k]) for k in ("Q", "K", "V", "dY", "W"))
    logD = torch.empty(Q.shape[:3], device="cuda")
    Y, st, ks = slim.fwd(Q, K, V, W, C, kind, dropout=dropout, seed=3, logD=logD)
    g = slim.bwd(Q, K, V, W, dY, C, ks, kind, dropout=dropout, seed=3, Y=Y, logD=logD)
    torch.cuda.synchronize()
    return [Y, st, *[t for t in g if t is not None]]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_slices_do_not_change_the_bits(case, monkeypatch):
    need_gpu()
    L, d, M, dtype, kind, P = case
    print(f"[tiles] {case}", flush=True)
    if P:
        monkeypatch.setenv("SLIM_SEGMENTS", str(P))
    x = make_inputs(Workload("tiles", 77, 1, 2, L, d, M, (L,), dtype, kind))
    ref = _run(x, L, kind)
    for C in (1, 31, 33, 64, 100):
        for i, (a, b) in enumerate(zip(ref, _run(x, C, kind))):
            assert torch.equal(a, b), (C, i)


@pytest.mark.parametrize("C", [7, 31, 33, 100])
def test_masks_follow_the_slices(C):
    need_gpu()
    print(f"[tiles] dropout C={C}", flush=True)
    L, p = 131, 0.3
    x = make_inputs(Workload("tilesd", 78, 1, 2, L, 64, 256, (L,), "bf16", "favor+"))
    Y = _run(x, C, "favor+", p)[0]
    mask = O.value_mask(1, 2, L, 64, C, p, 3)
    ref, _ = O.slim_forward(host64(x["Q"]), host64(x["K"]), host64(x["V"]) * mask, x["W"], L, "favor+", within="quadratic")
    report("Y", host64(Y), ref / (1.0 - p), TOL["bf16"])
