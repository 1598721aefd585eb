"""GPU parity of the products of verifications and short prompts for every tile
count their work-groups take.

One-layer models of d 128 (attention skipped: nothing is rounded to bfloat16 on
the way) whose gate/up product and head have 24 to 2000 tiles of 16 rows: three
tiles per work-group, four, or (two packings of the activations and more)
seven, with work-groups that are full, end in fewer tiles, or hold one ragged
tile.  5, 10 and 16 rows fill one, two and three packings.

Tolerance: the products of the activations' three bfloat16 terms are exact, so
only float32 sums round: at most 14000 terms in 3 x 437 matrix instructions and
8 + 4 partial sums of 2^-24 of the running sum each, in a chain of three
products; 3 x 1323 x 2^-24 = 2.4e-4 of the row's logit deviation bounds the
difference, and the sums' rounding is far from its worst case: 1e-4.
"""

import numpy as np
import pytest

import oracle
import sd_synth as S
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


REL = 1e-4
# (ffn_dim, vocabulary): gate/up has ffn_dim / 8 tiles, the head vocabulary / 16
SHAPES = [(256, 371), (8320, 16500), (13952, 27970), (8192, 32000)]
_models = {}


def _pair(F, V):
    if (F, V) not in _models:
        cfg = S.ModelConfig(f"tiles_{F}", 1, 128, 2, 1, 64, F, V, "bf16")
        w = S.make_weights(cfg, 7)
        _models[(F, V)] = (cfg, oracle.Model(cfg, w), U.device_model(cfg, w))
    return _models[(F, V)]


@pytest.mark.parametrize("rows", [3, 5, 6, 10, 11, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("F,V", SHAPES)
def test_tile_counts(F, V, rows):
    cfg, om, dm = _pair(F, V)
    toks = S.prompt(cfg, rows, seed=rows)
    skip = np.array([1, 0], np.uint8)
    ref = om.score(toks, skip)["logits"]
    out = torch.full((rows, V), float("nan"), dtype=torch.float32, device="cuda")
    dm.forward(toks, dm.cache(rows), skip=skip, logits=out)
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref).max(axis=1)
    worst = float((err / (REL * ref.std(axis=1))).max())
    print(f"F {F} V {V} {rows} rows: max |d| / tol {worst:.3f}")
    assert worst <= 1
