"""Every tile of the large-M GEMM with every kind of product, against float64.

Each tile runs shapes whose rows and columns are a multiple of it, one more and
one less, and reductions of one 8-element chunk to more stages than are in
flight, most of them no multiple of the 32-wide stage; split reductions also
with more splits than stages.  Activations span 2^-40 to 2^40, weights as many
octaves.  Whatever lies past the outputs keeps its contents.

Tolerance of a sum: the products are exact and a matrix instruction adds 32 of
them to a float32 sum; with three terms (K / 32 rounded up) x 3 instructions,
one addition per split and one for the sums of the small terms, each rounding
to 2^-23 of sum |x w|.
"""

import ctypes

import numpy as np
import pytest

from paper_2309_08168_amd import binding

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


STORE, RESID, SWIGLU, QKV = 0, 1, 2, 3
TILES = [(256, 256), (224, 256), (256, 128), (128, 128), (128, 64)]
SENTINEL = -77.0


def _operands(M, N, K, seed):
    """(W bf16 [N][K], x float32 [M][K], its three terms [3][M][K])"""
    g = torch.Generator(device="cuda").manual_seed(seed)

    def spread(*shape, octaves):
        e = torch.randint(-octaves, octaves + 1, shape, device="cuda", generator=g).float()
        return torch.randn(shape, device="cuda", generator=g) * torch.exp2(e)

    W = spread(N, K, octaves=12).bfloat16()
    x = spread(M, K, octaves=20) * torch.exp2(torch.randint(-20, 21, (M, 1), device="cuda", generator=g).float())
    terms, rest = [], x
    for _ in range(3):
        terms.append(rest.bfloat16())
        rest = rest - terms[-1].float()
    assert not rest.any()
    return W, x, torch.stack(terms)


def _run(tile, epi, splits, W, A, C, ldc, out=None, rope=None):
    """The product on the given tile; out [3][rows][F], rope (table, k, v, start, heads, kv heads, head_dim)."""
    (N, K), M = W.shape, A.shape[1]
    zero = torch.zeros(8, dtype=torch.bfloat16, device="cuda")
    table, k, v, start, H, KVH, dh = rope or (zero, zero, zero, 0, 1, 1, 32)
    p, i, l = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    rc = binding.load().sdk_prefill_gemm(
        i(tile), i(epi), i(splits), i(M), i(N), i(K), p(W.data_ptr()), p(A.data_ptr()), l(A.stride(0)),
        p(zero.data_ptr()), p(C.data_ptr() if C is not None else 0), l(ldc), p(out.data_ptr() if out is not None else 0),
        l(out.stride(0) if out is not None else 0), p(table.data_ptr()), p(k.data_ptr()), p(v.data_ptr()),
        l(k.stride(0) if rope else 0), i(start), i(H), i(KVH), i(dh), p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, rc
    torch.cuda.synchronize()


def _exact(W, x, splits=1):
    """(x W^T, what the sums may be off by)"""
    K = W.shape[1]
    xd, wd = x.double(), W.double()
    rounds = 3 * -(-K // 32) + splits + 1
    return xd @ wd.T.contiguous(), rounds * 2.0 ** -23 * (xd.abs() @ wd.abs().T.contiguous())


def _check(got, ref, tol, what):
    worst = float(((got - ref).abs() / tol.clamp_min(1e-300)).max())
    print(f"{what}: max |d| / tol {worst:.3f}", flush=True)
    assert worst <= 1, what


def _shapes(tile):
    bn, bm = TILES[tile]
    return [(bm, bn, 8), (bm + 1, bn + 1, 40), (bm - 1, 2 * bn - 1, 136), (2 * bm + 3, bn + 5, 200), (17, 36, 1000),
            (min(4 * bm + 1, 1000), 16, 96)]


@pytest.mark.parametrize("shape", range(6))
@pytest.mark.parametrize("tile", range(5), ids=lambda t: "%dx%d" % TILES[t])
def test_store(tile, shape):
    M, N, K = _shapes(tile)[shape]
    W, x, A = _operands(M, N, K, 100 * tile + shape)
    for ldc in (N, (N + 7) // 4 * 4):  # whatever N is, and rows on 16 bytes
        C = torch.full((M + 1, ldc), SENTINEL, device="cuda")
        _run(tile, STORE, 1, W, A, C, ldc)
        ref, tol = _exact(W, x)
        _check(C[:M, :N].double(), ref, tol, f"store {M} x {N} x {K}, pitch {ldc}")
        assert (C[M:] == SENTINEL).all() and (C[:, N:] == SENTINEL).all()


@pytest.mark.parametrize("splits", [1, 2, 3, 5, 8])
@pytest.mark.parametrize("tile", range(5), ids=lambda t: "%dx%d" % TILES[t])
def test_partial_sums(tile, splits):
    bn, bm = TILES[tile]
    M, N, K = min(bm + 1, 4096 // splits - 1), bn + 4, 136 + 8 * splits
    W, x, A = _operands(M, N, K, 10 * tile + splits)
    C = torch.full((splits * M + 1, N), SENTINEL, device="cuda")
    _run(tile, RESID, splits, W, A, C, N)
    ref, tol = _exact(W, x, splits)
    _check(C[:splits * M].double().view(splits, M, N).sum(0), ref, tol, f"{splits} partial sums {M} x {N} x {K}")
    assert (C[splits * M:] == SENTINEL).all()
    assert torch.isfinite(C).all()


@pytest.mark.parametrize("F,K,dm", [(8, 8, 0), (104, 40, 1), (120, 136, -1), (264, 200, 3)])
@pytest.mark.parametrize("tile", range(5), ids=lambda t: "%dx%d" % TILES[t])
def test_swiglu(tile, F, K, dm):
    M = TILES[tile][1] + dm
    g = torch.Generator(device="cuda").manual_seed(tile + F)
    W = (0.3 * torch.randn(2 * F, K, device="cuda", generator=g)).bfloat16()
    W[F:] = (W[F:].float() * torch.exp2(torch.arange(F, device="cuda").float() % 40 - 20)[:, None]).bfloat16()
    x = torch.randn(M, K, device="cuda", generator=g)
    a = x.bfloat16()
    b = (x - a.float()).bfloat16()
    A = torch.stack([a, b, (x - a.float() - b.float()).bfloat16()])
    out = torch.full((3, M + 1, F), SENTINEL, dtype=torch.bfloat16, device="cuda")
    _run(tile, SWIGLU, 1, W, A, None, 0, out=out)
    (gate, up), (tg, tu) = (t.split(F, 1) for t in _exact(W, x))
    silu = gate / (1 + torch.exp(-gate))
    # |silu'| <= 1.1; exponential, division and two products: 8 roundings; the terms are exact
    tol = 1.1 * tg * (up.abs() + tu) + silu.abs() * tu + 8 * 2.0 ** -23 * (silu * up).abs()
    _check(out[:, :M].double().sum(0), silu * up, tol, f"swiglu {M} x {F} x {K}")
    assert (out[:, M:] == SENTINEL).all()


@pytest.mark.parametrize("H,KVH,dh,K,dm", [(1, 1, 32, 8, 0), (3, 1, 64, 40, 1), (6, 2, 128, 136, -1), (5, 5, 32, 200, 3)])
@pytest.mark.parametrize("tile", range(5), ids=lambda t: "%dx%d" % TILES[t])
def test_rotary_and_kv_append(tile, H, KVH, dh, K, dm):
    M, N, half, start = TILES[tile][1] + dm, (H + 2 * KVH) * dh, dh // 2, 5
    W, x, A = _operands(M, N, K, 7 * tile + H)
    cap = start + M + 1
    ang = torch.rand(cap, half, device="cuda", generator=torch.Generator(device="cuda").manual_seed(tile)) * 6.28
    table = torch.stack([torch.cos(ang), torch.sin(ang)], -1).contiguous()
    k, v = (torch.full((KVH, cap, dh), SENTINEL, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q = torch.full((M + 1, H * dh), SENTINEL, device="cuda")
    _run(tile, QKV, 1, W, A, q, H * dh, rope=(table, k, v, start, H, KVH, dh))
    ref, tol = (t.view(M, H + 2 * KVH, dh) for t in _exact(W, x))
    cos, sin = (table[start:start + M, None, :, i].double() for i in (0, 1))

    hk = H + KVH
    a, b = ref[:, :hk].split(half, 2)
    rot = torch.cat([a * cos - b * sin, b * cos + a * sin], -1)
    # what the sums may be off by, and three roundings of the rotation
    a, b = (tol[:, :hk] + 3 * 2.0 ** -23 * ref[:, :hk].abs()).split(half, 2)
    rtol = torch.cat([a * cos.abs() + b * sin.abs(), b * cos.abs() + a * sin.abs()], -1)
    _check(q[:M].double().view(M, H, dh), rot[:, :H], rtol[:, :H], f"q {M} x {N} x {K}")
    for got, want, t, name in ((k, rot[:, H:], rtol[:, H:], "k"), (v, ref[:, hk:], tol[:, hk:], "v")):
        _check(got[:, start:start + M].double(), want.transpose(0, 1), (t + 2.0 ** -8 * (want.abs() + t)).transpose(0, 1),
               f"{name} {M} x {N} x {K}")
        assert (got[:, :start] == SENTINEL).all() and (got[:, start + M:] == SENTINEL).all()
    assert (q[M:] == SENTINEL).all()
