"""The scoring passes' launch forms against a 64-bit softmax: small-call
kernels, aligned and crossing persistent blocks, slabs shared by waves, every
row-block count and output layout, and row sums that leave the range of a
block's reference.  A host test checks that the forms named here launch the
kernels they name."""

from __future__ import annotations

import math

import pytest

pytestmark = pytest.mark.gpu


def _run(nl, H, G, d, W, Lp, dtype, per_head, spike, at=None):
    import torch
    from paper_2606_01790_amd import starkv as sk
    g = torch.Generator(device="cuda").manual_seed(nl * 1000 + Lp)
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    L = Lp + W
    k = torch.randn(nl, G, L + 3, d, generator=g, device="cuda").to(tt)
    q = torch.randn(nl, H, W, d, generator=g, device="cuda").to(tt)
    if spike:
        # keys that grow along the cache and one far above the rest (at a
        # third of it, or `at`), neither in a block's last slab
        k[:, :, Lp // 3 if at is None else at] *= spike
        k[:, :, :Lp // 2] *= torch.linspace(0.1, 4.0, Lp // 2, device="cuda").to(tt)[:, None]
    dims = sk.make_dims(nl, H, G, d, L, W, sk.F32 if dtype == "f32" else sk.BF16, per_head)
    p = sk.params_default()
    lay = sk.contiguous_layout(k, dims)
    S = torch.empty(nl, dims.Ns, Lp, device="cuda")
    sbar = torch.empty(nl, Lp, device="cuda")
    gstar = torch.empty(nl, Lp, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sk.workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    sk.score(dims, p, q, k, lay, S, sbar, gstar, ws)
    torch.cuda.synchronize()
    ref = torch.zeros(nl, dims.Ns, Lp, dtype=torch.float64, device="cuda")
    hps = H // dims.Ns
    ymax = 0.0
    for l in range(nl):
        for h in range(H):
            kk = k[l, h // (H // G), :Lp].double()
            y = (q[l, h].double() @ kk.t().contiguous()) / math.sqrt(d)
            ymax = max(ymax, float(y.abs().max()) * math.log2(math.e))
            ref[l, h // hps] += torch.softmax(y, 1).sum(0)
    ref = torch.nn.functional.avg_pool1d(ref, 5, stride=1, padding=2) / hps
    # per value: the rounding of y, of c and of their difference, each up to
    # 2^-24 of a magnitude of at most ymax + 32 (c adds log2 of the row sum),
    # the fp32 dot product's d steps, and the sums over rows; doubled
    tol = 2 * (3 * (ymax + 32) + d * ymax / 8 + 64) * 2.0 ** -24
    # values far below the row's mass may underflow to zero on the way
    err = ((S.double() - ref).abs() / (ref + 1e-25)).max()
    assert float(err) <= tol, (float(err), tol)


# (layers, H, G, d, W, Lp, dtype, per_head)
FORMS = [
    (1, 28, 4, 128, 32, 700, "bf16", False),      # small kernels, nrb 7
    (2, 28, 4, 128, 32, 2915, "bf16", False),     # small pass 1, pass 2 above a block per CU
    (2, 8, 8, 64, 8, 130, "bf16", False),         # small, one row block, ragged
    (1, 8, 2, 128, 32, 321, "f32", False),        # small, fp32
    (1, 8, 2, 128, 32, 321, "bf16", True),        # small, per head
    (1, 8, 2, 128, 16, 321, "bf16", True),        # small pass 1, 8-row heads in pass 2
    (40, 14, 2, 64, 32, 700, "bf16", False),      # small pass 1, aligned pass 2
    (28, 28, 4, 128, 32, 1025, "bf16", False),    # aligned
    (28, 28, 4, 128, 32, 1025, "bf16", True),
    (28, 12, 2, 128, 24, 1025, "bf16", True),     # 8-row heads that cross row blocks
    (3, 2, 2, 64, 512, 14001, "bf16", False),     # sixteen row blocks, few groups
    (1, 15, 1, 128, 32, 30001, "bf16", False),    # fifteen row blocks, small pass 1
    (11, 32, 8, 64, 16, 9001, "bf16", False),     # aligned pass 1, pass 2 crossing groups
    (9, 16, 4, 128, 8, 9001, "f32", False),       # fp32, one 32-token tile at a time
    (9, 16, 4, 64, 8, 9001, "f32", True),
]


@pytest.mark.parametrize("form", FORMS, ids=["-".join(map(str, f)) for f in FORMS])
def test_score_form(form):
    _run(*form, spike=0.0)


@pytest.mark.parametrize("form", [FORMS[0], FORMS[7], FORMS[8], FORMS[11], FORMS[12], FORMS[13]],
                         ids=["small", "aligned", "per-head", "persistent", "crossing", "f32"])
def test_sums_beyond_the_reference(form):
    """Logits that rise far above their block's reference: the row sums are
    taken again against a higher one, or, where they are not finite, against
    running maxima."""
    _run(*form, spike=24.0)


def _layers_error(nl, H, G, d, W, Lp, dtype, top, layers, fill=None):
    """S against 64 bits over some layers, unpooled: the 2-norm of the
    difference over that of the result.  Every group has one key (at a third
    of the cache) about `top` log2 units above the others, if any; fill =
    (rows, level): the last keys, at about `level`, and the others low."""
    import torch
    from paper_2606_01790_amd import starkv as sk
    g = torch.Generator(device="cuda").manual_seed(Lp)
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    L = Lp + W
    k = torch.empty(nl, G, L, d, dtype=tt, device="cuda").normal_(generator=g)
    u = torch.randint(0, 2, (nl, G, d), generator=g, device="cuda").float() * 2 - 1
    q = torch.randn(nl, H, W, d, generator=g, device="cuda")
    q = (q + (3 * u.repeat_interleave(H // G, 1)[:, :, None] if top or fill else 0)).to(tt)
    unit = 3 * math.sqrt(d) * math.log2(math.e)      # q.u of a key u, in log2 units
    if fill:
        k *= 0.1
    if top:
        k[:, :, Lp // 3] = (top / unit * u).to(tt)
    if fill:
        k[:, :, Lp - fill[0]:Lp] = (fill[1] / unit * u).to(tt)[:, :, None]
    dims = sk.make_dims(nl, H, G, d, L, W, sk.F32 if dtype == "f32" else sk.BF16, False)
    p = sk.params_default()
    p.pool_kernel = 1
    S = torch.empty(nl, G, Lp, device="cuda")
    sbar = torch.empty(nl, Lp, device="cuda")
    gstar = torch.empty(nl, Lp, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sk.workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    sk.score(dims, p, q, k, sk.contiguous_layout(k, dims), S, sbar, gstar, ws)
    num = den = 0.0
    for l in layers:
        for i in range(G):
            kk = k[l, i, :Lp].double().t().contiguous()
            y = q[l, i * (H // G):(i + 1) * (H // G)].double().reshape(-1, d) @ kk
            ref = torch.softmax(y / math.sqrt(d), 1).sum(0) / (H // G)
            num += float((S[l, i].double() - ref).pow(2).sum())
            den += float(ref.pow(2).sum())
    return math.sqrt(num / den)


@pytest.mark.parametrize("form,top", [((28, 28, 4, 128, 32, 2915, "bf16"), 0),
                                      ((28, 28, 4, 128, 32, 2915, "bf16"), 24),
                                      ((28, 14, 2, 64, 32, 9001, "bf16"), 0),
                                      ((16, 16, 4, 128, 8, 4114, "f32"), 0)])
def test_row_sums_logarithm_is_unbiased(form, top):
    """S over many rows: each row's own roundings (of y, c and y - c, half an
    ulp each) average out over a group's 32 to 224 rows.  What is left: the
    exponential's error, at most an ulp (2^-23), which may lean to one side,
    and the sums', as much again.  A logarithm of the whole row sum adds up to
    an ulp of about 10 (2^-20), or of 24, to one side (3.1e-7, 3.6e-7)."""
    assert _layers_error(*form, top, range(2)) <= 2.0 ** -22


@pytest.mark.parametrize("form", [(28, 28, 28, 128, 1, 2915, "bf16"), (64, 8, 8, 64, 1, 9001, "bf16"),
                                  (64, 8, 8, 64, 1, 2915, "f32")])
def test_sums_far_above_their_reference(form):
    """One window row per group, whose top key (12 log2 units, most of the
    mass) stands 48 above every block's last slab: the row's statistics are as
    exact as with a near reference.  Roundings of the row, half an ulp each
    times ln 2: c below 16, 3.3e-7; against a near reference the exponent of
    pass 1 below 16, as much, and that of pass 2, near 0; uniform, so a
    2-norm over the groups of 0.58 of their root sum of squares, 2.7e-7, and
    2^-22 for the exponential and the sums as above.  Against the last slab an
    exponent of 32 to 64 is off by up to 1.3e-6, 7.6e-7 in the 2-norm."""
    nl, H, G, d, W, Lp, dtype = form
    fill = (Lp - Lp // 3 - 1, -36)      # every key behind the top one
    err = _layers_error(*form, 12, range(4), fill)
    assert err <= 2.7e-7 + 2.0 ** -22, err


# 130 groups of 63 slabs on 256 CUs: both passes' blocks take equal ranges of
# 31 or 32 slabs that cross from one group into the next
CROSSING = [
    (13, 20, 10, 128, 48, 4001, "bf16", False),
    (13, 20, 10, 128, 32, 4001, "bf16", True),
    (13, 20, 10, 64, 32, 4001, "bf16", False),
    (13, 10, 10, 64, 24, 4001, "f32", False),
    (13, 20, 10, 128, 32, 4001, "f32", True),
]


@pytest.mark.parametrize("at", [None, -130])
@pytest.mark.parametrize("form", CROSSING, ids=["-".join(map(str, f)) for f in CROSSING])
def test_crossing_blocks(form, at):
    """Blocks of several groups: window rows, references, sums and records of
    one segment after another.  With a key far above the others 130 tokens
    before the cache's end, the sums are redone in segments that other
    segments of the same block follow."""
    _run(*form, spike=24.0 if at else 0.0, at=at and form[5] + at)


# every row-block count of the persistent kernels: 44 groups of 21 slabs, the
# last ragged; W = 32 nrb - 8 rows of one head per group (a padded last row
# block), or nrb heads of 32 rows with an output each
ROW_BLOCKS = [(11, 4, 4, 128, 32 * n - 8, 1313, "bf16", False) for n in range(1, 16)] + \
             [(11, 4 * n, 4, 128, 32, 1313, "bf16", True) for n in range(2, 16)]
# and of the larger small-call kernels (nine row blocks and more)
SMALL_ROW_BLOCKS = [(1, 2, 2, d, 32 * n - 8, 321, "bf16", False)
                    for d, n in ((128, 9), (128, 12), (128, 15), (64, 9), (64, 16))] + \
                   [(1, 2 * n, 2, d, 32, 321, "bf16", True)
                    for d, n in ((128, 9), (128, 12), (128, 15), (64, 9), (64, 16))]


# pass 2's waves share a slab, four and two of them
SHARED = [(2, 28, 4, 128, 64, 2915, "bf16", False), (2, 8, 4, 64, 32, 2915, "f32", False)]


@pytest.mark.parametrize("form", ROW_BLOCKS + SMALL_ROW_BLOCKS + SHARED,
                         ids=["-".join(map(str, f)) for f in ROW_BLOCKS + SMALL_ROW_BLOCKS + SHARED])
def test_row_blocks(form):
    _run(*form, spike=0.0)
