"""INT4 decode: queries and weights as fixed-point digits (saw_fixed.h) where rounding, the units and the digits' range could go wrong.

Caches are made of chosen logits: every token of a kv head has the same codes and zero-point, so that its logits are its key scale times
one number per query head; values are random codes.  Against attention in 64 bits over the same bytes, row by row in the 2-norm.
What a row may be off by: its logits (up to X in base 2) and their exponentials are fp32 numbers, (X + 4) 2^-22 of the weights; n weights
rounded to 2^-(TOP + 1) of the largest p s are n 2^-(TOP + 1) of it, times the values' range of 15 over the row's own size; fp32 sums over the n / 64
batches of the p and of the p s (z - 8), z = 5, round by 2^-25 of them in each; and 2^-20 for the rest."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

# query heads per kv head, kv heads, head_dim: single 64-channel heads, head_dim 128, pairs of 64-channel heads
SHAPES = [(8, 1, 64), (4, 3, 64), (1, 1, 64), (2, 3, 64), (4, 2, 128), (8, 1, 128), (1, 3, 128), (2, 1, 128), (4, 4, 64), (2, 2, 64), (1, 2, 64)]

TOP = 27                                   # log2 of the largest weight when the unit is set, at least


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


def _make(saw, G, Hkv, d, B, L, k_scale, v_scale, seed=3, sizes=None):
    """k_scale, v_scale: [L] or [Hkv, L] scales of the tokens.  Every sequence has pages of its own with the same bytes.
    sizes: [Hkv, G] logits of a key scale of 1."""
    g = torch.Generator().manual_seed(seed)
    pages = (L + 16) // 16
    c = saw.Cache(B * pages, Hkv, d, 1)
    pad = lambda x: torch.cat([x.expand(Hkv, L), torch.full((Hkv, 16 * pages - L), float("nan"))], 1).view(Hkv, pages, 16).transpose(0, 1)
    kc = torch.randint(0, 256, (1, Hkv, 1, d // 2), generator=g, dtype=torch.uint8).expand(pages, Hkv, 16, d // 2)
    vc = torch.randint(0, 256, (pages, Hkv, 16, d // 2), generator=g, dtype=torch.uint8)
    km = torch.stack([pad(k_scale), torch.full((pages, Hkv, 16), 7.0)], -1)
    vm = torch.stack([pad(v_scale), torch.full((pages, Hkv, 16), 5.0)], -1)
    for dst, src in ((c.k_codes, kc), (c.v_codes, vc), (c.k_meta, km), (c.v_meta, vm)):
        dst.copy_(src.repeat(B, 1, 1, 1))
    pt = torch.arange(B * pages, dtype=torch.int32).view(B, pages).cuda()
    q = torch.randn((Hkv * G, d), generator=g)
    x = lambda codes: torch.stack([codes & 15, codes >> 4], -1).flatten(-2).double()
    one = torch.einsum("hgd,hd->hg", q.double().view(Hkv, G, d), x(kc[0, :, 0]) - 7) / d ** 0.5     # logit of scale 1, natural units
    q = q / (one.abs().flatten()[:, None] / one.sign().flatten()[:, None]).float()                     # ... made 1 for every head
    q = q * (torch.linspace(1.0, 0.8, G).repeat(Hkv) if sizes is None else sizes.flatten())[:, None]
    one = torch.einsum("hgd,hd->hg", q.double().view(Hkv, G, d), x(kc[0, :, 0]) - 7) / d ** 0.5
    V = (x(vc) - 5).transpose(0, 1).reshape(Hkv, 16 * pages, d)[:, :L] * v_scale.double().expand(Hkv, L)[..., None]
    return c, pt, q, one, V


def _logit_error(made):
    """[Hkv, G] what a logit may be off by, relative, in 2^-24: the query times its scale and log2(e) (three roundings an element), q.c and sum q as two
    halves each (two and two), their difference, the pair's scale times the unit and the product (three)."""
    c, q, one = made[0], made[2].double(), made[3]
    kc = c.k_codes[0, :, 0].cpu()
    codes = torch.stack([kc & 15, kc >> 4], -1).flatten(-2).double()[:, None]
    q = q.view(one.shape + (-1,))
    parts = 3 * (q * (codes - 7)).abs().sum(-1) + 2 * (q * codes).sum(-1).abs() + 2 * 7 * q.sum(-1).abs()
    return parts / q.shape[-1] ** 0.5 / one.abs() + 3


def _exact(one, V, k_scale, v_scale, logit_error=4.0):
    """logit_error: of the logits, relative, in 2^-24."""
    Hkv, L = V.shape[:2]
    v_scale = v_scale.expand(Hkv, L)[:, None]
    logits = one[..., None] * k_scale.double().expand(Hkv, L)[:, None]        # [Hkv][G][L]
    p = torch.softmax(logits, -1)
    o = p @ V
    X = float(logits.abs().max()) / math.log(2)
    most = (p * v_scale.double()).amax(-1)
    n, d = V.shape[-2:]
    sums = n / 64 * 2 ** -25 * (o.norm(dim=-1) + 3 * d ** 0.5 * (p * v_scale.double()).sum(-1))
    w = (X * logit_error + 16) * 2 ** -24                              # of a weight, relative
    tol = w * torch.sqrt((p ** 2) @ (V ** 2).sum(-1, keepdim=True)).squeeze(-1) + w * o.norm(dim=-1) + n * 2.0 ** -(TOP + 1) * most * 15 * d ** 0.5 + sums + 2 ** -20 * o.norm(dim=-1)
    return o.flatten(0, 1), tol.flatten()


def _check(saw, made, k_scale, v_scale, B, L, splits=(1, 3, 0), tag="", lost=(), logit_error=4.0):
    """lost: kv heads whose values are not finite, nor are their outputs."""
    c, pt, q, one, V = made
    want, tol = _exact(one, V, k_scale, v_scale, logit_error)
    rows = torch.ones(one.shape, dtype=torch.bool)
    rows[list(lost)] = False
    rows = rows.flatten()
    for s in splits:
        out = torch.full((B,) + q.shape, float("nan"), device="cuda")
        saw.paged_decode_attn(c, q.expand(B, *q.shape).contiguous().cuda(), pt, torch.full((B,), L, dtype=torch.int32).cuda(),
                              num_splits=s, out=out)
        err = (out.cpu().double() - want)[:, rows].norm(dim=-1)
        print(f"[fixed {tag} splits={s}] worst error over bound {float((err / tol[rows]).max()):.3f}", flush=True)
        assert (err <= tol[rows]).all()
        assert not out.cpu()[:, ~rows].isfinite().any()


def _logits(kind, L):
    t = torch.arange(L, dtype=torch.float32)
    if kind == "rising":                       # the reference moves in nearly every batch
        return 1 + t * (60.0 / L)
    if kind == "falling":
        return 61 - t * (60.0 / L)
    # a sink in front of a long even tail, 14 or 20 powers of two below it, whose weights round all alike
    s = torch.full((L,), 0.5)
    s[L // 3] = 0.5 + (14 if kind == "sink14" else 20) * math.log(2)
    return s


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("kind", ["rising", "falling", "sink14", "sink20"])
@pytest.mark.parametrize("B,L", [(2, 1), (2, 65), (2, 4001), (300, 333)])
def test_chosen_logits(saw, G, Hkv, d, kind, B, L):
    k = _logits(kind, L)
    v = 0.5 + 0.4 * torch.cos(torch.arange(L, dtype=torch.float32))
    _check(saw, _make(saw, G, Hkv, d, B, L, k, v), k, v, B, L, tag=f"{kind} G={G} Hkv={Hkv} d={d} B={B} L={L}")


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("lo,hi", [(-60, 60), (-95, -80), (-126, -122), (60, 90), (90, 120)])
def test_value_scales_far_apart(saw, G, Hkv, d, lo, hi):
    """Scales of the values over many powers of two, some zero: units follow the weights p s, not the p."""
    L = 1000
    t = torch.arange(L)
    v = torch.exp2((lo + (hi - lo) * ((37 * t) % 101) / 101).float())
    v[t % 9 == 4] = 0.0
    k = 2 + 3 * torch.sin(t.float())
    _check(saw, _make(saw, G, Hkv, d, 2, L, k, v), k, v, 2, L, tag=f"scales {lo} {hi} G={G} Hkv={Hkv} d={d}")


def _late(kind, Hkv, G, L):
    """Key and value scales [Hkv, L] (logits in base 2 before the head's size), sizes [Hkv, G], and the kv heads whose outputs are not
    finite.  The first half of the tokens sets the references of every wavefront and opens the first partitions."""
    t = torch.arange(L)
    late = t >= L // 2
    k = 2 + torch.sin(t.float())
    v = (0.5 + 0.4 * torch.cos(t.float())).repeat(Hkv, 1)
    sizes = torch.linspace(1.0, 0.8, G).repeat(Hkv, 1)
    lost = ()
    outlier = late & (t % 97 == 5)
    if kind == "unattended":                   # far below the others even times its scale
        k[outlier] = -180.0
        v[:, outlier] = 2.0 ** 102
    elif kind == "outweighs":                  # 2^-50 of the attention, 2^14 of the output
        k[outlier] = -50.0
        v[:, outlier] = 2.0 ** 64
    elif kind == "one head's":                 # what one query head attends to and the next one of the same kv head does not
        k[outlier] = 100.0
        v[:, outlier] = 2.0 ** 70
        sizes[:, 1::2] *= -1
    elif kind == "neighbour's":                # in every second kv head
        v[1::2, late] = 2.0 ** 100
    elif kind == "neighbour's infinity":
        v[1::2, outlier] = float("inf")
        lost = range(1, Hkv, 2)
    elif kind == "zero, then large":           # equal logits: denominators of both halves count alike
        k[:] = 2.0
        v[:, ~late], v[:, late] = 0.0, 2.0 ** 28
    elif kind == "tiny, then large":
        k[:] = 2.0
        v[:, ~late], v[:, late] = 2.0 ** -95, 2.0 ** 60
    elif kind == "large, then tiny":
        k[:] = 2.0
        v[:, ~late], v[:, late] = 2.0 ** 60, 2.0 ** -95
    elif kind == "zero rising":                # weights of 0 whose denominators grow by 2^27, then ordinary tokens
        k[:] = torch.where(t < L // 4, 1.0, 28.0)
        v[:, t < L - L // 4] = 0.0
        sizes[:] = 1.0
    elif kind == "zero rising far":            # ... by 2^127.5: every p is finite, the sum of a few is not
        k[:] = torch.where(t < L // 4, 1.0, 128.5)
        v[:, t < L - L // 4] = 0.0
        sizes[:] = 1.0
    return (k * math.log(2)).repeat(Hkv, 1), v, sizes, lost


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("kind", ["unattended", "outweighs", "one head's", "neighbour's", "neighbour's infinity", "zero, then large",
                                  "tiny, then large", "large, then tiny", "zero rising", "zero rising far"])
@pytest.mark.parametrize("B,L", [(1, 2100), (300, 520)])
def test_value_scales_that_change_within_a_range(saw, G, Hkv, d, kind, B, L):
    """A head's outputs follow its own values only, whatever its neighbours' are and whatever comes late in a range."""
    k, v, sizes, lost = _late(kind, Hkv, G, L)
    made = _make(saw, G, Hkv, d, B, L, k, v, sizes=sizes)
    _check(saw, made, k, v, B, L, lost=lost, logit_error=_logit_error(made), tag=f"{kind} G={G} Hkv={Hkv} d={d} B={B}")


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("B", [1, 4, 300])
def test_new_token_whose_logit_is_minus_infinity(saw, G, Hkv, d, B):
    """It counts for nothing: the step's output is that of the cached tokens (key scales of 2^-120 make ordinary logits of such queries)."""
    L = 200
    k = (2 + torch.sin(torch.arange(L).float())) * 2.0 ** -120
    made = _make(saw, G, Hkv, d, B, L, k, torch.ones(L), sizes=torch.linspace(1.0, 0.8, G).repeat(Hkv, 1) * 2.0 ** 120)
    c, pt, q, one, V = made
    want, tol = _exact(one, V, k, torch.ones(L), _logit_error(made))
    x = (q.view(Hkv, G, d)[:, 0].sign() * -1024).to(torch.bfloat16).expand(B, Hkv, d).contiguous().cuda()
    rows = torch.arange(Hkv) * G                   # (the heads whose signs the new keys have)
    out = saw.append_decode_attn(c, x, torch.ones_like(x), q.expand(B, *q.shape).contiguous().cuda(), pt,
                                 torch.full((B,), L, dtype=torch.int32).cuda(), out=torch.empty((B,) + q.shape, device="cuda"))
    err = (out.cpu().double() - want)[:, rows].norm(dim=-1)
    print(f"[-inf G={G} Hkv={Hkv} d={d} B={B}] worst error over bound {float((err / tol[rows]).max()):.3f}", flush=True)
    assert (err <= tol[rows]).all()


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
def test_smallest_queries(saw, G, Hkv, d):
    """A query row below 2^-119 (its unit is the smallest fp32 number then) with key scales that make ordinary logits of it."""
    L = 300
    k = (2 + torch.sin(torch.arange(L).float())) * 2.0 ** 118
    made = _make(saw, G, Hkv, d, 2, L, k, torch.ones(L), sizes=torch.linspace(1.0, 0.8, G).repeat(Hkv, 1) * 2.0 ** -118)
    _check(saw, made, k, torch.ones(L), 2, L, logit_error=_logit_error(made), tag=f"smallest G={G} Hkv={Hkv} d={d}")


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
def test_all_value_scales_zero(saw, G, Hkv, d):
    L, k = 200, torch.linspace(1, 3, 200)
    c, pt, q, _, _ = _make(saw, G, Hkv, d, 1, L, k, torch.zeros(L))
    for s in (1, 2):
        out = saw.paged_decode_attn(c, q[None].cuda(), pt, torch.tensor([L], dtype=torch.int32).cuda(), num_splits=s)
        assert (out == 0).all()


@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_a_query_row_that_is_not_finite_is_nan_alone(saw, G, Hkv, d, bad):
    L, k = 150, torch.linspace(1, 3, 150)
    c, pt, q, _, _ = _make(saw, G, Hkv, d, 1, L, k, torch.ones(L))
    lens = torch.tensor([L], dtype=torch.int32).cuda()
    for s in (1, 2):
        want = saw.paged_decode_attn(c, q[None].cuda(), pt, lens, num_splits=s)
        q2 = q.clone()
        q2[-1, 11] = bad
        got = saw.paged_decode_attn(c, q2[None].cuda(), pt, lens, num_splits=s)
        assert got[0, -1].isnan().all()
        # (a row that is NaN has the others' units set anew in every batch: another rounding of fp32 sums)
        assert G * Hkv == 1 or float((got - want)[0, :-1].abs().max() / want.abs().max()) < 2 ** -20


@pytest.mark.parametrize("G,Hkv,d", [(8, 1, 64), (1, 1, 64), (4, 1, 128), (4, 2, 64)])
def test_long_even_range(saw, G, Hkv, d):
    """One partition of 281617 tokens, all weights alike."""
    L = 4 * 64 * 1100 + 17
    k, v = torch.full((L,), 0.25), torch.full((L,), 0.75)
    _check(saw, _make(saw, G, Hkv, d, 1, L, k, v), k, v, 1, L, splits=(1,), tag=f"long G={G} d={d}")


@pytest.mark.parametrize("G,Hkv,d", [(8, 1, 64), (1, 1, 64), (4, 1, 128), (8, 1, 128), (4, 2, 64), (1, 2, 64)])
def test_more_batches_than_the_digits_hold(saw, G, Hkv, d):
    """One partition whose wavefronts would each add up more than 31 bits of the largest digits: codes as far from the middle as they go, and
    weights just under the most that four digits hold behind a first batch 15.6 times below them.  Logits are 0 and every weight is a whole
    number, so what rounds is the running fp32 sums: a batch of one wavefront each, 2^-25 of the sum and of the smaller one of p s (z - 8)."""
    pages = 8 * 4 * 2200
    c = saw.Cache(pages, Hkv, d, 1)
    waves = saw.decode_schedule(c, 1, Hkv * G, 16 * pages, num_splits=1)["waves"]
    batches = 2110                                           # of each wavefront
    L = 64 * waves * batches
    assert L <= 16 * pages
    least, most = 0.5, 7.8
    digit = round(2 ** 28 * most / 2 ** 24)                  # (the first batch's largest p s, 1/2, is 2^27)
    assert 2 ** 28 * most < 2.1e9 and 64 * batches * digit * 128 > 2 ** 31
    c.k_meta.zero_()
    c.v_meta[..., 0], c.v_meta[..., 1] = most, 5.0
    c.v_meta[:4 * waves, ..., 0] = least
    pt = torch.arange(pages, dtype=torch.int32).view(1, pages).cuda()
    q = torch.randn((1, Hkv * G, d), generator=torch.Generator().manual_seed(1)).cuda()
    out = saw.paged_decode_attn(c, q, pt, torch.tensor([L], dtype=torch.int32).cuda(), num_splits=1, out=torch.empty_like(q))
    want = -5 * (least + (batches - 1) * most) / batches
    err = float((out.double() / want - 1).abs().max())
    print(f"[digits G={G} Hkv={Hkv} d={d} waves={waves}] error {err:.1e}", flush=True)
    assert err <= 2 * batches * 2 ** -25 + 2 ** -20


def _attend64(c, pt, q, lens):
    """Attention in 64 bits over the cache's bytes, blocks of 64 channels rotated."""
    H = torch.ones((1, 1), dtype=torch.float64)
    while H.shape[0] < 64:
        H = torch.cat([torch.cat([H, H], 1), torch.cat([H, -H], 1)], 0)
    d, Hkv = q.shape[-1], c.n_kv_heads
    R = torch.block_diag(*[H / 8] * (d // 64)).cuda()
    out = []
    for b, n in enumerate(lens):
        def rows(codes, meta):
            w, m = codes[pt[b].long()], meta[pt[b].long()].double()
            x = torch.stack([w & 15, w >> 4], -1).flatten(-2).double()
            return ((x - m[..., 1:]) * m[..., :1]).transpose(0, 1).flatten(1, 2)[:, :n]
        K, V = rows(c.k_codes, c.k_meta), rows(c.v_codes, c.v_meta)
        p = torch.softmax((q[b].double() @ R).view(Hkv, -1, d) @ K.transpose(1, 2).contiguous() / d ** 0.5, -1)
        out.append(((p @ V) @ R).flatten(0, 1))
    return torch.stack(out)


@pytest.mark.parametrize("G,Hkv,d", SHAPES + [(8, 2, 128), (4, 8, 128), (4, 8, 64), (8, 8, 64)])
@pytest.mark.parametrize("size", [1.0, 2.0 ** -90, 2.0 ** 80])
@pytest.mark.parametrize("heads", ["all", "odd"])
@pytest.mark.parametrize("B", [4, 40, 66])
def test_new_token_opens_the_state(saw, G, Hkv, d, size, heads, B):
    """The fused step, and a decode of what it stored, against attention in 64 bits: the new token first in a wavefront's running state, or one of a
    batch's, its values as large as the cached ones, far below or far above, in all kv heads or in every second one.  Both are within
    2^-20 (n 2^-28 included), row by row."""
    g = torch.Generator().manual_seed(B)
    lens = [(0, 1, 64, 65, 700, 1300)[b % 6] for b in range(B)]
    pages = 1301 // 16 + 1
    c = saw.Cache(B * pages, Hkv, d, 64)
    pt = torch.arange(B * pages, dtype=torch.int32).view(B, pages).cuda()
    for codes, meta in ((c.k_codes, c.k_meta), (c.v_codes, c.v_meta)):
        codes.copy_(torch.randint(0, 256, codes.shape, generator=g, dtype=torch.uint8))
        meta.copy_(torch.stack([torch.rand(meta.shape[:-1], generator=g) * 0.2 + 0.05, torch.full(meta.shape[:-1], 7.0)], -1))
    q = torch.randn((B, Hkv * G, d), generator=g).cuda()
    k, v = (torch.randn((B, Hkv, d), generator=g).to(torch.bfloat16).cuda() for _ in range(2))
    sizes = torch.ones(Hkv, 1)
    sizes[(1 if heads == "odd" else 0)::(2 if heads == "odd" else 1)] = size
    n = torch.tensor(lens, dtype=torch.int32).cuda()
    got = [saw.append_decode_attn(c, k, (v.float() * sizes.cuda()).to(torch.bfloat16), q, pt, n, out=torch.empty_like(q))]
    got += [saw.paged_decode_attn(c, q, pt, n + 1, num_splits=s, out=torch.empty_like(q)) for s in (0, 1)]
    want = _attend64(c, pt, q, [x + 1 for x in lens])
    for i, out in enumerate(got):
        err = (out.double() - want).norm(dim=-1) / want.norm(dim=-1)
        print(f"[open G={G} Hkv={Hkv} d={d} size={size:.1e} {heads} B={B} call={i}] worst {float(err.max()):.2e}", flush=True)
        assert (err <= 2 ** -20).all()
