"""The large-M attention kernels alone, against float64: head_dim 128 (128 query
rows share 64-key stages, split over chunks of the keys) with up to 64 heads
and with more (a wave per 16 rows), head_dim 32 and 64; rows at the edges of
the 16-, 32- and 128-row shares, contexts at the edges of blocks and chunks,
grouped heads.  Rows past the last and the other terms' rows keep their
contents.

Tolerance: with p the weights of a row's n keys, the output is off by at most
(2 ds + r) sum p |v| / sum p.  ds, of a score: three roundings of q and k's
products with it in at most 24 matrix instructions, 27 x 2^-23 sum |q k| /
sqrt(head_dim), 2^-22 of the maximum's difference and 2^-22 for the
exponential.  r, of the two sums: per 32 keys six matrix instructions, a
rescaling and an addition, 8 (n / 32 + 1) + 16 for the lanes, the chunks and the
division, times 2^-23.
"""

import ctypes
import math

import pytest

from paper_2309_08168_amd import binding

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


SENTINEL = -77.0


def _attention(q, k, v, start, H):
    """The output [M][H][dh] of q [M][H dh] over caches [KVH][cap][dh]."""
    M, KVH, dh = q.shape[0], k.shape[0], k.shape[2]
    part = torch.empty(4096 * H * dh, device="cuda")
    ml = torch.empty(4096 * H * 2, device="cuda")
    out = torch.full((3, M + 1, H * dh), SENTINEL, dtype=torch.bfloat16, device="cuda")
    p, i, l = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    rc = binding.load().sdk_prefill_attention(
        i(M), i(start), i(H), i(KVH), i(dh), p(q.data_ptr()), p(k.data_ptr()), p(v.data_ptr()), l(k.stride(0)),
        p(part.data_ptr()), p(ml.data_ptr()), p(out.data_ptr()), l(out.stride(0)),
        p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, rc
    torch.cuda.synchronize()
    assert (out[:, M:] == SENTINEL).all()
    return out[:, :M].double().sum(0).view(M, H, dh)


@pytest.mark.parametrize("M,start", [(17, 0), (33, 300), (127, 1), (128, 0), (129, 63), (300, 212), (64, 5000), (1024, 31)])
@pytest.mark.parametrize("H,KVH,dh", [(4, 4, 128), (8, 2, 128), (66, 3, 128), (4, 2, 64), (3, 1, 32)])
def test_against_float64(H, KVH, dh, M, start):
    g = torch.Generator(device="cuda").manual_seed(1000 * M + H + dh)
    q = 1.4 * torch.randn(M, H * dh, device="cuda", generator=g)
    # (a cache with room past the context: its contents must not matter)
    k, v = (torch.randn(KVH, start + M + 9, dh, device="cuda", generator=g).bfloat16() for _ in range(2))
    k[:, start + M:], v[:, start + M:] = float("nan"), float("nan")
    got = _attention(q, k, v, start, H)
    n = start + M
    see = torch.arange(n, device="cuda")[None] <= torch.arange(start, n, device="cuda")[:, None]
    worst = 0.0
    for h in range(H):
        qh, kh, vh = q.view(M, H, dh)[:, h].double(), k[h // (H // KVH), :n].double(), v[h // (H // KVH), :n].double()
        s = (qh @ kh.T.contiguous() / math.sqrt(dh)).masked_fill(~see, -math.inf)
        size = (qh.abs() @ kh.abs().T.contiguous() / math.sqrt(dh)).masked_fill(~see, 0.0).amax(1)
        drop = (s.amax(1) - s.masked_fill(~see, math.inf).amin(1))
        ds = 27 * 2.0 ** -23 * size + 2.0 ** -22 * drop + 2.0 ** -22
        w = torch.softmax(s, -1)
        tol = (2 * ds + (8 * (n / 32 + 1) + 16) * 2.0 ** -23)[:, None] * (w @ vh.abs())
        worst = max(worst, float(((got[:, h] - w @ vh).abs() / tol).max()))
    print(f"{H}/{KVH} heads of {dh}, {M} rows at {start}: max |d| / tol {worst:.3f}")
    assert worst <= 1


def test_sum_of_equal_weights():
    """One key above many with equal scores: the sum of the weights of a chunk's 15256 keys takes one rounding per 32
    keys, at most 2^-24 of the sum so far, which is half the whole on average, and 24 beside.  With one per key they
    would err the same way each time: 2.9e-5 here."""
    M, start, H = 1024, 60000, 4
    g = torch.Generator(device="cuda").manual_seed(9)
    n = torch.arange(start + 1, start + M + 1, device="cuda", dtype=torch.float64)[:, None]
    q = torch.zeros(M, H, 128, device="cuda")
    q[:, :, 0] = math.sqrt(128) * (0.3 + 3 * torch.rand(M, H, device="cuda", generator=g))
    k, v = (torch.zeros(1, start + M, 128, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    k[0, 0, 0] = 1
    v[0, 0] = 1
    got = _attention(q.view(M, H * 128), k, v, start, H)
    top = torch.exp(q[:, :, 0].double() / math.sqrt(128))
    ref = (top / (top + n - 1))[:, :, None]
    worst = float(((got - ref).abs() / ref).max())
    tol = (15256 / 32 / 2 + 24) * 2.0 ** -24
    print(f"relative error {worst:.2e}, tolerance {tol:.2e}")
    assert worst <= tol
