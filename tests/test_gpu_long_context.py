"""GPU parity of attention over contexts long enough that a work-group walks
several blocks of keys (decode: more than 1280 work-groups otherwise) and that
the large forward's attention splits the keys of a row block into many chunks.

One-layer attention models over a cache filled with N(0, 1) keys and values,
loaded into the oracle and the GPU alike; causal prefixes of one oracle forward
of 200 rows check GPU forwards of 1 to 200 rows.  The attention output is about
a quarter of the residual stream here, and leaving out one block of 64 keys of
10500 would move it by several percent: the tolerance of the attention tests
(1e-3 of the row's logit deviation) is far below that.
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


# ragged last blocks; 16 and 8 kv heads x 165 blocks of 64 (VALU), 2 kv heads x
# 8 query tiles x 165 blocks of 128 and 16 x 83 (matrix cores, 16 rows)
@pytest.mark.parametrize("name,ctx", [("mha_dh128", 10501), ("gqa2_dh128", 10501), ("gqa8_dh128", 21050),
                                      ("mha_dh32", 12345), ("gqa4_dh64", 3001)])
def test_long_contexts(name, ctx):
    cfg, _, om, dm = A._pair(name)
    rows = 200
    cap = ctx + rows + 1
    fill = S.kv_fill(cfg, 2 * cfg.n_kv_heads * ctx * cfg.head_dim, 3)
    toks = S.prompt(cfg, rows, seed=ctx)
    oc = om.cache(cap)
    oc.load(fill, ctx, "bf16")
    ref = om.forward(oc, toks)["logits"]
    buf = torch.zeros(dm.kv_cache_bytes(cap) // 2, dtype=torch.int16, device="cuda")
    buf.view(-1, cap, cfg.head_dim)[:, :ctx].copy_(
        torch.from_numpy(fill.view(np.int16)).view(-1, ctx, cfg.head_dim).to("cuda"))
    cache = dm.cache(cap, device_buf=buf)
    for n in (1, 2, 5, 16, 40, 129, 200):
        cache.set_length(ctx)
        out = torch.empty((n, cfg.vocab), dtype=torch.float32, device="cuda")
        dm.forward(toks[:n], cache, logits=out)
        A._tight(ref[:n], out.cpu().numpy(), f"{name} {n} rows over {ctx} keys")


F32 = {"tiny": S.MODELS["tiny"], "f32_dh128": S.ModelConfig("f32_dh128", 1, 256, 4, 2, 128, 256, 512, "f32"),
       "f32_dh16": S.ModelConfig("f32_dh16", 1, 128, 8, 4, 16, 256, 512, "f32")}
_f32 = {}


@pytest.mark.parametrize("ctx", [1, 120, 255, 500, 511, 700])
@pytest.mark.parametrize("name", list(F32))
def test_short_and_split_contexts_f32(name, ctx):
    """Both sides of the line between one work-group per query vector and the
    split over the keys (512 keys for float32 caches): forwards of 1 to 16 rows
    that end below, at and past it."""
    cfg = F32[name]
    if name not in _f32:
        w = S.make_weights(cfg, 9)
        _f32[name] = (oracle.Model(cfg, w), U.device_model(cfg, w))
    om, dm = _f32[name]
    cap = ctx + 16
    fill = S.kv_fill(cfg, cfg.n_layers * 2 * cfg.n_kv_heads * ctx * cfg.head_dim, 4)
    toks = S.prompt(cfg, 16, seed=ctx)
    oc = om.cache(cap)
    oc.load(fill, ctx, "f32")
    ref = om.forward(oc, toks)["logits"]
    buf = torch.zeros(dm.kv_cache_bytes(cap) // 4, dtype=torch.float32, device="cuda")
    buf.view(-1, cap, cfg.head_dim)[:, :ctx].copy_(torch.from_numpy(fill).view(-1, ctx, cfg.head_dim).to("cuda"))
    cache = dm.cache(cap, device_buf=buf)
    for n in (1, 2, 5, 12, 16):
        cache.set_length(ctx)
        out = torch.empty((n, cfg.vocab), dtype=torch.float32, device="cuda")
        dm.forward(toks[:n], cache, logits=out)
        U.check_logits(cfg, out.cpu().numpy(), ref[:n], f"{name} {n} rows over {ctx} keys")


@pytest.mark.parametrize("name", list(A.CONFIGS))
@pytest.mark.parametrize("ctx", [240, 250, 256])
def test_short_and_split_contexts_bf16(name, ctx):
    """The same line for bfloat16 caches (256 keys)."""
    cfg, _, om, dm = A._pair(name)
    cap = ctx + 16
    fill = S.kv_fill(cfg, 2 * cfg.n_kv_heads * ctx * cfg.head_dim, 5)
    toks = S.prompt(cfg, 16, seed=ctx)
    oc = om.cache(cap)
    oc.load(fill, ctx, "bf16")
    ref = om.forward(oc, toks)["logits"]
    buf = torch.zeros(dm.kv_cache_bytes(cap) // 2, dtype=torch.int16, device="cuda")
    buf.view(-1, cap, cfg.head_dim)[:, :ctx].copy_(
        torch.from_numpy(fill.view(np.int16)).view(-1, ctx, cfg.head_dim).to("cuda"))
    cache = dm.cache(cap, device_buf=buf)
    for n in (1, 2, 6, 7, 16):
        cache.set_length(ctx)
        out = torch.empty((n, cfg.vocab), dtype=torch.float32, device="cuda")
        dm.forward(toks[:n], cache, logits=out)
        A._tight(ref[:n], out.cpu().numpy(), f"{name} {n} rows over {ctx} keys")
