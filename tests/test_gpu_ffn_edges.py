"""The expert MLP's grouped GEMMs at the edges of their tiles (GPU).

Row counts around the 32-row matrix-core blocks, the waves' 64- and 128-row
shares and the 256-row tiles, widths that end inside a 64-deep stage and inside
a tile's columns, experts without rows. The first cases' weight gradients take
the 128 x 128 tiling and their d-wide row products the 256 x 192 one; WEIGHT_CASES
and ROW_CASES name the tiling they are there for and check it against the
library's rule. Every product is compared on its own
with a float64 product of the same bf16 operands (the backward's and the
down-projection's operands are the GPU's own earlier outputs), and rows past an
expert's count hold NaN on input and must stay as they were on output.

Bound per element: an f32 sum of K exact products lies within
gamma_K sum |a b| of the exact one (gamma_K ~ K 2^-24; K + 8 here for the bias
and partial sums), a bf16 result is rounded once more (2^-9, and 2^-8 is
allowed). gelu and gelu' of a value off by b are off by at most 1.13 b and
0.8 b (the largest |gelu'| and |gelu''|) and by their own error, 1e-6. f32
layers (32 x 32 and 64 x 64 tiles, four waves splitting k) are held to the same
bounds without the bf16 rounding.
"""
import numpy as np
import pytest
import torch

from paper_2608_16188_amd import vmoe as V

from .gpu_common import row_tile, say, weight_grad_tile

pytestmark = pytest.mark.gpu

# (d, f, rows per expert)
CASES = [
    (72, 200, [1, 31, 32, 33, 0, 63, 64, 65]),
    (128, 264, [127, 128, 129, 0, 96, 97]),
    (192, 768, [255, 256, 257, 288, 289, 16]),
    (320, 136, [511, 513, 40, 320, 321]),
    (64, 64, [2, 191, 193]),
    (520, 1032, [300, 5, 0, 449]),
    (1024, 256, [33, 17, 290, 640]),
    # a few rows in buffers of two, three and four m-tiles: column parts
    (512, 128, [500, 20, 32]),
    (512, 128, [600, 20, 1]),
    (448, 128, [900, 9, 32]),
    (192, 64, [700, 30]),
    # buffers of at most 64 and 32 rows: the small-batch forward
    (72, 200, [64, 1, 33, 0, 63, 32]),
    (520, 136, [32, 31, 0, 2]),
    (768, 264, [52, 40, 64]),
    # two m-tiles an expert, rows split evenly
    (136, 328, [257, 320, 321, 448, 512]),
]
# 16 and more experts: dxe beside the weight gradients
MANY = (200, 520, [0, 1, 7, 32, 33, 34, 63, 64, 65, 100, 127, 128, 129, 200, 255, 256, 257])
# weight gradients on the 256-row tiles, rows being k here: none, one, a stage of
# 64 and its neighbours, an odd number of stages; (tiling, d, f, rows, quota
# scheduling). 544, 1056 and 160 make rows of whole 128-byte lines, 520, 1032 and
# 136 of split ones
_K = [0, 1, 31, 33, 63, 64, 65, 128, 129, 257, 192, 2]
WEIGHT_CASES = [
    ("big", 520, 1032, [0, 1, 33, 64, 65, 129, 257, 31], False),
    ("big", 520, 1032, [63, 128, 0, 2, 192, 64, 1, 130], True),
    ("big", 544, 1056, [0, 1, 33, 64, 65, 129, 257, 31], False),
    ("big", 520, 1056, [63, 128, 0, 2, 192, 64, 1, 130], False),
    ("narrow", 136, 520, [_K[e % 12] for e in range(64)], False),
    ("narrow", 136, 520, [_K[e * 5 % 12] for e in range(64)], True),
    ("narrow", 160, 544, [_K[e * 7 % 12] for e in range(64)], False),
]
# d-wide row products on 256 x 256 tiles, buffers of one, two and four m-tiles
# (light experts in one, two and four column parts): (tiling, d, f, rows, quota)
ROW_CASES = [
    ("big", 1000, 64, [(17 * e + 1) % 257 for e in range(64)], False),
    ("big", 1000, 64, [500, 257] + [(11 * e) % 40 for e in range(30)], False),
    ("big", 1000, 72, [800, 0, 1, 31, 32, 33, 64, 257, 512, 513, 769, 16, 65, 255, 256, 20], False),
    ("big", 1000, 72, [800, 0, 1, 31, 32, 33, 64, 257, 512, 513, 769, 16, 65, 255, 256, 20], True),
]
# f32 layers: k shares of no, one and an odd number of 8-deep runs, tiles of 32
# and (enough of them in a launch) of 64
F32_CASES = [
    (8, 40, [1, 31, 32, 33, 0, 64, 65]),
    (72, 200, [7, 8, 9, 0, 63, 100]),
    (192, 768, [197, 200, 3, 0, 160, 161, 129, 96]),
    (512, 1032, [40, 64, 65, 0, 7, 33, 1, 30]),
    (72, 3080, [512, 500, 449, 0, 64, 65, 480, 1]),
    (3080, 40, [512, 500, 449, 0, 64, 65, 480, 1]),
]
# f32, twelve and more 64 x 64 tiles a CU in the up-projection: 64 x 64 tiles of a short k
F32_MANY_TILES = [
    (40, 328, [2049, 0, 1, 63, 64, 65, 2000, 300] * 2),
    (224, 520, [1473, 0, 33, 64, 1408, 127, 128, 129] * 2),
    (232, 520, [1473, 0, 33, 64, 1408, 127, 128, 129] * 2),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


def _gamma(k):
    return (k + 8) * 2.0 ** -24


def _check(name, got, ref, bound):
    got = got.double().cpu()
    bad = ~((got - ref).abs() <= bound)  # NaN counts as bad
    assert not bad.any(), (name, int(bad.sum()), float((got - ref).abs().max()))


def _rounded(ref, bound):
    """Bound of a result that is rounded to bf16."""
    return bound + 2.0 ** -8 * (ref.abs() + bound)


@pytest.mark.parametrize("d,f,rows", CASES + [MANY], ids=lambda v: str(v) if isinstance(v, int) else "")
def test_products_at_tile_edges(d, f, rows):
    _products(d, f, rows, torch.bfloat16)


@pytest.mark.parametrize("d,f,rows", F32_CASES + F32_MANY_TILES, ids=lambda v: str(v) if isinstance(v, int) else "")
def test_f32_products_at_tile_edges(d, f, rows):
    _products(d, f, rows, torch.float32)


@pytest.mark.parametrize("tile,d,f,rows,quota", WEIGHT_CASES,
                         ids=lambda v: "" if isinstance(v, list) else str(v))
def test_weight_gradients_at_tile_edges(tile, d, f, rows, quota):
    assert weight_grad_tile(d, f, len(rows)) == tile
    _products(d, f, rows, torch.bfloat16, quota)


@pytest.mark.parametrize("tile,d,f,rows,quota", ROW_CASES,
                         ids=lambda v: "" if isinstance(v, list) else str(v))
def test_row_products_at_tile_edges(tile, d, f, rows, quota):
    assert row_tile(max(rows), d, len(rows)) == tile
    _products(d, f, rows, torch.bfloat16, quota)


def _products(d, f, rows, dt, quota=False):
    say("ffn edges", d, f, rows, dt, quota)
    fwd = V.vmoe_expert_ffn_fwd_quota if quota else V.vmoe_expert_ffn_fwd
    bwd = V.vmoe_expert_ffn_bwd_quota if quota else V.vmoe_expert_ffn_bwd

    def _stored(ref, bound):  # a stored result: rounded once more in bf16
        return _rounded(ref, bound) if dt == torch.bfloat16 else bound

    E, R = len(rows), max(rows)
    s = V.make_shape(R * E, 1, d, f, E, 1, 1.0,
                     V.VMOE_BF16 if dt == torch.bfloat16 else V.VMOE_F32, capacity_override=R)
    assert V.vmoe_capacity(s) == R
    gen = torch.Generator().manual_seed(d * 1000 + f)

    def randn(*shape, scale=1.0):
        return (torch.randn(*shape, generator=gen) * scale).to(dt)

    def padded(t):
        for e, n in enumerate(rows):
            t[e, n:] = float("nan")
        return t.cuda()

    xe, dye = padded(randn(E, R, d)), padded(randn(E, R, d, scale=0.3))
    w1, w2 = randn(E, f, d, scale=0.06).cuda(), randn(E, d, f, scale=0.06).cuda()
    b1, b2 = randn(E, f, scale=0.1).cuda(), randn(E, d, scale=0.1).cuda()
    counts = torch.tensor([rows], dtype=torch.int32).cuda()

    def out(*shape, dtype=dt):
        return torch.full(shape, 77.0, dtype=dtype, device="cuda")

    act, act_grad, ye = out(E, R, f), out(E, R, f), out(E, R, d)
    fwd(s, xe, counts, w1, b1, w2, b2, act, act_grad, ye)
    dh, dxe = out(E, R, f), out(E, R, d)
    g = {n: out(*sh, dtype=torch.float32) for n, sh in
         dict(dw1=(E, f, d), db1=(E, f), dw2=(E, d, f), db2=(E, d)).items()}
    bwd(s, xe, counts, w1, w2, act, act_grad, dye, dh, dxe, g["dw1"], g["db1"], g["dw2"], g["db2"])
    torch.cuda.synchronize()

    c = {n: t.double().cpu() for n, t in dict(xe=xe, dye=dye, w1=w1, w2=w2, b1=b1, b2=b2, act=act,
                                              act_grad=act_grad, dh=dh).items()}
    for e, n in enumerate(rows):
        for name, t in dict(act=act, act_grad=act_grad, ye=ye, dh=dh, dxe=dxe).items():
            assert (t[e, n:] == 77.0).all(), f"{name}[{e}]: rows past the expert's were written"
        x, dy, a, ag, h = (c[k][e, :n] for k in ("xe", "dye", "act", "act_grad", "dh"))
        W1, W2 = c["w1"][e], c["w2"][e]
        H, Hb = x @ W1.T + c["b1"][e], _gamma(d) * (x.abs() @ W1.abs().T + c["b1"][e].abs())
        cdf = 0.5 * (1 + torch.erf(H * np.sqrt(0.5)))
        pdf = torch.exp(-0.5 * H * H) / np.sqrt(2 * np.pi)
        _check("act", act[e, :n], H * cdf, _stored(H * cdf, 1.13 * Hb + 1e-6))
        _check("act_grad", act_grad[e, :n], cdf + H * pdf, _stored(cdf + H * pdf, 0.8 * Hb + 1e-6))
        Y = a @ W2.T + c["b2"][e]
        _check("ye", ye[e, :n], Y, _stored(Y, _gamma(f) * (a.abs() @ W2.abs().T + c["b2"][e].abs())))
        D = (dy @ W2) * ag
        _check("dh", dh[e, :n], D, _stored(D, _gamma(d) * (dy.abs() @ W2.abs()) * ag.abs()))
        X = h @ W1
        _check("dxe", dxe[e, :n], X, _stored(X, _gamma(f) * (h.abs() @ W1.abs())))
        for name, p, q in (("dw1", h, x), ("dw2", dy, a)):
            _check(name, g[name][e], p.T @ q, _gamma(n) * (p.abs().T @ q.abs()))
        for name, p in (("db1", h), ("db2", dy)):
            _check(name, g[name][e], p.sum(0), _gamma(n) * p.abs().sum(0))
