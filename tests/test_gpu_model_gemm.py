"""The model step's products (float32 values as sums of three bf16 ones on the
matrix cores) at the edges of their tiles, against the fp64 oracle.

Row counts around the 64- and 128-row tiles, an alphabet just past a 128-column
tile with 16-byte loads (132) and without (131), reductions with a last k tile
of 1 to 31 (row counts, in the weight gradients), the 128-row plan (at least 512
tiles) with two rows in its last tile, and the normalisation's two row widths.

Bar: a product of K terms rounds its sum every 16 terms, 2^-24 of the partial
sum each time, and leaves out parts of terms below 2^-24 of them: 2e-6 of the
gradients' norm lies an order above both through a layer's chain of products,
and a wrong or missing part of the split (2^-8 or 2^-16 of every term) far
above it.  The same bar with three slices: the state before the first is exactly
nothing, and the rounding of one recovered by subtraction lies at 2^-24 of it.
"""

import pytest

import oracle
from synth import ModelConfig
from tests.gpu_common import need_gpu
from tests.test_gpu_model import _gpu, _oracle

pytestmark = pytest.mark.gpu

CASES = [
    ModelConfig("gemm63", L=63, D=64, s=1, vocab=131, B=1),
    ModelConfig("gemm65", L=65, D=128, s=1, vocab=132, B=1),
    ModelConfig("gemm129", L=129, D=192, s=1, vocab=128, B=1),
    ModelConfig("gemm127x2", L=127, D=64, s=1, vocab=4, B=2),
    ModelConfig("gemm4098", L=2049, D=512, s=1, vocab=129, B=2),
    # layer normalisation with 4 values per thread, full, and with 16
    ModelConfig("ln1024", L=20, D=1024, s=1, vocab=64, B=2),
    ModelConfig("ln1088", L=33, D=1088, s=1, vocab=64, B=1),
    # rows enough for the normalisation to sum a split product's parts
    ModelConfig("parts1088", L=300, D=1088, s=1, vocab=64, B=1),
    ModelConfig("parts256", L=259, D=256, s=1, vocab=64, B=1),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_products_at_tile_edges(cfg):
    need_gpu()
    print(f"[model] cfg={cfg}", flush=True)
    ref_loss, ref = _oracle(cfg)
    for C in (cfg.L, cfg.L // 3 + 1):
        loss, g = _gpu(cfg, C)
        disc = oracle.grad_discrepancy(g, ref)
        print(f"  C {C} loss {loss:.7f} ref {ref_loss:.7f}; discrepancy {disc:.2e}", flush=True)
        assert abs(loss - ref_loss) <= 2e-6 * abs(ref_loss)
        assert disc <= 2e-6
