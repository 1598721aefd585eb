"""GPU parity of the large-M GEMMs at the edges of their tiles and of the
range of their operands.

- MLP and head products of one-layer models (attention skipped, so nothing is
  rounded to bfloat16 on the way): 17 to 64 rows on the thin GEMM and more on
  the tile GEMM (128 x 64 at these sizes), at every boundary of 16-row blocks
  and 64-row tiles; a shape whose reductions are no multiple of 64 or 32 takes
  the tile GEMM at every row count.
- Weight rows far from the others' magnitude, and an MLP activation 2^12 times
  the others that its down weights undo, beside one 2^-35 times the others.
- Powers of two on MLP channels that the down weights undo: the logits are, bit
  for bit, those of the model without them.
- MLP activations of every row near the ends of float32's range, the down
  weights undoing the factor.
- The rotary embedding and KV append in the thin QKV product, after a prefix
  and after a decode step over the keys it wrote.

Tolerance of the products: every output is a chain of three products of at most
2048 terms, accumulated in float32 in at most 3 (terms) x 64 (steps of 32)
matrix instructions and 8 partial sums, each rounding to 2^-24 of the running
sum.  The sum of their worst cases, 3 x 200 x 2^-24 = 3.6e-5 of the norm of the
row, bounds the difference to 5e-5 of the row's logit deviation times the factor
the oracle's own logit rows are scaled by.
"""

import numpy as np
import pytest

import oracle
import sd_synth as S
from tests import gpu_util as U
from tests import test_gpu_attention as A

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


MLP_REL = 5e-5
THIN = S.ModelConfig("terms_thin", 1, 256, 4, 2, 64, 1344, 777, "bf16")
RAGGED = S.ModelConfig("terms_ragged", 1, 136, 3, 1, 32, 200, 777, "bf16")
LONG_K = S.ModelConfig("terms_long_k", 1, 512, 4, 2, 64, 2048, 400, "bf16")
# head rows scaled far below and above the rest
HEAD_ROWS = {5: -30, 6: -30, 200: 9, 399: -60}
_models = {}


def _pair(cfg, scaled):
    if (cfg.name, scaled) not in _models:
        w = S.make_weights(cfg, 11)
        if scaled:
            F = cfg.ffn_dim
            for r, e in HEAD_ROWS.items():
                w["lm_head"][r] = S.scale_tensor(w["lm_head"][r], 2.0 ** e, "bf16")
            gu = w["layers.0.w_gate_up"]
            gu[F + 3] = S.scale_tensor(gu[F + 3], 2.0 ** 12, "bf16")
            gu[F + 40] = S.scale_tensor(gu[F + 40], 2.0 ** -35, "bf16")
            w["layers.0.w_down"][:, 3] = S.scale_tensor(np.ascontiguousarray(w["layers.0.w_down"][:, 3]), 2.0 ** -12,
                                                        "bf16")
        _models[(cfg.name, scaled)] = (w, oracle.Model(cfg, w), U.device_model(cfg, w))
    return _models[(cfg.name, scaled)]


def _check(cfg, rows, scaled):
    _, om, dm = _pair(cfg, scaled)
    toks = S.prompt(cfg, rows, seed=rows)
    skip = np.array([1, 0], np.uint8)
    ref = om.score(toks, skip)["logits"]
    out = torch.full((rows, cfg.vocab), float("nan"), dtype=torch.float32, device="cuda")
    dm.forward(toks, dm.cache(rows), skip=skip, logits=out)
    scale = np.ones(cfg.vocab)
    if scaled is True:
        for r, e in HEAD_ROWS.items():
            scale[r] = 2.0 ** e
    plain = scale == 1
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref) / scale
    worst = float((err / (MLP_REL * ref[:, plain].std(axis=1, keepdims=True))).max())
    print(f"{cfg.name} {rows} rows scaled {scaled}: max |d| / tol {worst:.3f}")
    assert worst <= 1


@pytest.mark.parametrize("rows", [17, 32, 33, 48, 49, 64, 65, 96, 129, 257, 513])
@pytest.mark.parametrize("cfg", [THIN, RAGGED], ids=lambda c: c.name)
def test_products_at_tile_edges(cfg, rows):
    _check(cfg, rows, False)


@pytest.mark.parametrize("rows", [33, 64, 100, 300])
@pytest.mark.parametrize("cfg", [THIN, LONG_K], ids=lambda c: c.name)
def test_rows_of_other_magnitudes(cfg, rows):
    _check(cfg, rows, True)


@pytest.mark.parametrize("rows", [33, 100])
@pytest.mark.parametrize("exp", [-112, 112])
def test_activations_near_the_ends_of_the_range(exp, rows):
    """Up weights times 2^exp, down weights times 2^-exp: both exact in bfloat16, and so is every product's factor."""
    key = (THIN.name, exp)
    if key not in _models:
        w = S.make_weights(THIN, 11)
        F = THIN.ffn_dim
        gu, down = w["layers.0.w_gate_up"], w["layers.0.w_down"]
        gu[F:] = S.scale_tensor(np.ascontiguousarray(gu[F:]), 2.0 ** exp, "bf16")
        down[:] = S.scale_tensor(down, 2.0 ** -exp, "bf16")
        _models[key] = (w, oracle.Model(THIN, w), U.device_model(THIN, w))
    _check(THIN, rows, exp)


@pytest.mark.parametrize("name", list(A.CONFIGS))
@pytest.mark.parametrize("rows", [17, 40, 64])
def test_thin_rotary_and_kv_append(name, rows):
    """rows after a prefix of 50 and one decode row over all of them."""
    cfg, _, om, dm = A._pair(name)
    toks = S.prompt(cfg, 50 + rows + 1, seed=rows + 1)
    oc, gc = om.cache(len(toks)), dm.cache(len(toks))
    for lo, hi in ((0, 50), (50, 50 + rows), (50 + rows, 51 + rows)):
        ref = om.forward(oc, toks[lo:hi])["logits"]
        out = torch.empty((hi - lo, cfg.vocab), dtype=torch.float32, device="cuda")
        dm.forward(toks[lo:hi], gc, logits=out)
        A._tight(ref, out.cpu().numpy(), f"{name} rows {lo}..{hi}")


# MLP channel -> exponent of a power of two on its up row, undone on its down column
CHANNELS = {
    # every down row has a largest magnitude near 2^-10 and elements down to 2^-35, the activations the reverse
    "spread": {k: 6 + k % 20 for k in range(THIN.ffn_dim)},
    # one MLP activation 2^24 and one 2^30 times the others
    "outliers": {3: 24, 40: 30},
}


@pytest.mark.parametrize("rows", [17, 33, 64, 100, 300])
@pytest.mark.parametrize("what", list(CHANNELS))
def test_powers_of_two_change_no_bit(what, rows):
    """The three terms hold an activation exactly and weights are multiplied as they are, so a power of two on a
    weight goes through every product and sum unchanged: the logits are those of the plain model, bit for bit."""
    _, _, plain = _pair(THIN, False)
    if (THIN.name, what) not in _models:
        w = S.make_weights(THIN, 11)
        F, gu, down = THIN.ffn_dim, w["layers.0.w_gate_up"], w["layers.0.w_down"]
        for k, e in CHANNELS[what].items():
            gu[F + k] = S.scale_tensor(gu[F + k], 2.0 ** e, "bf16")
            down[:, k] = S.scale_tensor(np.ascontiguousarray(down[:, k]), 2.0 ** -e, "bf16")
        _models[(THIN.name, what)] = U.device_model(THIN, w)
    toks, skip = S.prompt(THIN, rows, seed=rows), np.array([1, 0], np.uint8)
    got = []
    for dm in (plain, _models[(THIN.name, what)]):
        out = torch.full((rows, THIN.vocab), float("nan"), dtype=torch.float32, device="cuda")
        dm.forward(toks, dm.cache(rows), skip=skip, logits=out)
        got.append(out.cpu().numpy().astype(np.float64))
    worst = np.abs(got[0] - got[1]).max() / got[0].std()
    assert np.array_equal(got[0], got[1]), f"{what}, {rows} rows: {worst} of the deviation"


# vocabulary row -> exponent of a power of two on it
HEAD_POWERS = {0: -60, 5: -30, 200: 9, 399: 112, 776: 118}


@pytest.mark.parametrize("rows", [17, 33, 64, 100, 300])
def test_logits_near_the_ends_of_the_range(rows):
    """Head rows times powers of two up to 2^118: the logits are those of the plain model times the power, bit for
    bit, so no intermediate value leaves float32's range where the logit does not."""
    _, _, plain = _pair(THIN, False)
    if (THIN.name, "head") not in _models:
        w = S.make_weights(THIN, 11)
        for r, e in HEAD_POWERS.items():
            w["lm_head"][r] = S.scale_tensor(w["lm_head"][r], 2.0 ** e, "bf16")
        _models[(THIN.name, "head")] = U.device_model(THIN, w)
    toks, skip = S.prompt(THIN, rows, seed=rows), np.array([1, 0], np.uint8)
    got = []
    for dm in (plain, _models[(THIN.name, "head")]):
        out = torch.full((rows, THIN.vocab), float("nan"), dtype=torch.float32, device="cuda")
        dm.forward(toks, dm.cache(rows), skip=skip, logits=out)
        got.append(out.cpu().numpy().astype(np.float64))
    for r, e in HEAD_POWERS.items():
        got[1][:, r] *= 2.0 ** -e
    assert np.array_equal(got[0], got[1])
