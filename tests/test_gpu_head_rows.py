"""Greedy decisions over every row count of a verification: with nothing
skipped and no exit threshold every stage drafts K_max tokens and accepts them
all, so the verification has K_max + 1 rows, whose maxima come from K_max + 1
rows of tile statistics.  Tokens equal the oracle's autoregressive ones up to
its first near-tie, and every stage before it is full and fully accepted.
Vocabularies of 97 (a ragged last tile), 1000 and 1024."""

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


_models = {}


def _pair(cfg):
    if cfg.name not in _models:
        w = S.make_weights(cfg, 2)
        om = oracle.Model(cfg, w)
        prompt = S.prompt(cfg, 20, seed=4)
        toks, margin = om.generate_ar(prompt, 64)
        std = om.score(np.concatenate([prompt, toks[:-1]]))["logits"][len(prompt) - 1:].std(axis=1)
        _models[cfg.name] = (U.device_model(cfg, w), prompt, toks, margin, std)
    return _models[cfg.name]


@pytest.mark.parametrize("k_max", [1, 2, 3, 4, 5, 7, 8, 10, 13, 15])
@pytest.mark.parametrize("cfg", [S.MODELS["tiny"], U.MICRO_GQA, U.MINI_BF16], ids=lambda c: c.name)
def test_full_stages(cfg, k_max):
    dm, prompt, toks, margin, std = _pair(cfg)
    out, st = dm.generate_sd(prompt, 64, S.skip_mask(cfg, "none"), k_max, 0.0)
    n = U.check_free_running(cfg, out, toks, margin, std, f"{cfg.name} K_max {k_max}")
    full = n // (k_max + 1)
    assert (st["stages"][:full] == k_max).all(), st["stages"][:full]
    print(f"{cfg.name} K_max {k_max}: {n} of 64 tokens, {full} full stages")
