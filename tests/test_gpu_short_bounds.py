"""Short bounds: several wavefronts over each whole sequence instead of partitions, pair blocks and the in-kernel ranking; the
short partitions of one sequence and of the 16-bit call.

Both sides of each line of the rules, in (sequence, kv head) items and in tokens, decode and fused step, with and without the
caller's order, 64-channel heads in pairs and one at a time, a learned rotation and the 16-bit cache; lengths from zero to the bound,
every (scale, zero) pair its own.  Against attention in 64 bits over the same bytes, row by row, in the 2-norm over a row's channels.
What a row may be off by, worked out from its own weights p, values v and scales s (`_attend`):
  * the query and the weights are rounded to u (two bf16 limbs: 2^-16; single 64-channel heads and the 16-bit call of 64 channels or eight
    query heads carry 24 bits, and a logit's and exp2's fp32 sums make 2^-21 of it): a weight by u, and by u sqrt(sum (q k)^2) / sqrt(d)
    through its logit, signs at random: 2 u (1 + X) sqrt(sum p^2 |v|^2);
  * the matrix cores cut a running sum of weights times codes off at 2^-23 of it in each of the two steps a 64-token batch of a partition, and it grows
    up to M sum p s (codes are held as 128 + c: M = 143; as integers up to 16 where 24 bits are carried; 16-bit values as they are);
  * 2^-20 of the row for the rest."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


def _lens(B, bound):
    v = [(37 * i * i + 11 * i) % (bound + 1) for i in range(B)]
    v[B // 2], v[-1], v[0] = 0, min(1, bound), bound      # (the last one wins in a batch of one)
    return v


def _hadamard(h, d):
    H = torch.ones(1, 1, dtype=torch.float64)
    while H.shape[0] < h:
        H = torch.cat([torch.cat([H, H], 1), torch.cat([H, -H], 1)])
    return torch.block_diag(*[H / h ** 0.5] * (d // h)).cuda()


def _cache(saw, B, n_kv, d, bound, dense):
    need = (bound + 16) // 16
    R = torch.linalg.qr(torch.randn(128, 128, generator=torch.Generator().manual_seed(7)))[0] if dense else None
    c = saw.Cache(B * need, n_kv, d, 64, 3, dense=R)
    g = torch.Generator(device="cuda").manual_seed(B + bound)
    for codes, meta in ((c.k_codes, c.k_meta), (c.v_codes, c.v_meta)):
        codes.random_(0, 256, generator=g)
        meta[..., 0].uniform_(0.03, 0.2, generator=g)
        meta[..., 1] = torch.randint(5, 11, meta.shape[:-1], device="cuda", generator=g).float()
    pt = torch.randperm(B * need, device="cuda", generator=g).to(torch.int32).view(B, need)
    rot = _hadamard(64, d) @ (R.double().cuda() if dense else torch.eye(d, dtype=torch.float64, device="cuda"))
    return c, pt, g, rot


def _chunk(saw, c, B, Hq, bound):
    """tokens of a fixed partition (a batch cut by its lengths: up to all)"""
    parts = saw.decode_schedule(c, B, Hq, bound)["partitions"] or 1
    return 64 * math.ceil(math.ceil(bound / 64) / parts)


def _attend(K, V, size, q, chunk, u, M):
    """K, V [L][Hkv][d] of one sequence, size [L][Hkv] (scale, or largest value), q [Hq][d], all fp64 -> rows [Hq][d], what they may be off"""
    n, n_kv, d = K.shape
    if n == 0:
        return torch.zeros_like(q), torch.zeros_like(q[:, 0])
    qh, Kt = q.view(n_kv, -1, d), K.permute(1, 2, 0).contiguous()
    p = torch.softmax(torch.matmul(qh, Kt) / d ** 0.5, -1)
    o = torch.matmul(p, V.transpose(0, 1).contiguous())
    X = (torch.matmul(qh ** 2, Kt ** 2).amax(-1) / d).sqrt()
    spread = torch.matmul(p ** 2, (V ** 2).sum(-1).T.unsqueeze(-1)).squeeze(-1).sqrt()
    sums = math.ceil(min(n, chunk) / 64) * 2 ** -23 * M * torch.matmul(p, size.T.unsqueeze(-1)).squeeze(-1) * d ** 0.5
    return o.reshape(-1, d), (2 * u * (1 + X) * spread + sums + 2 ** -20 * o.norm(dim=-1)).flatten()


def _exact(c, q, pt, lens, rot, chunk, fine):
    def values(codes, meta, pages, n):
        w = codes[pages].permute(0, 2, 1, 3).flatten(0, 1)[:n]                        # [L][Hkv][d / 2]
        m = meta[pages].permute(0, 2, 1, 3).flatten(0, 1)[:n].double()
        x = torch.stack([w & 15, w >> 4], -1).flatten(-2).double()
        return (x - m[..., 1:]) * m[..., :1], m[..., 0]
    qr, out = q.double() @ rot, []
    for b, n in enumerate(lens.tolist()):
        pages = pt[b, :(n + 15) // 16].long()
        V, size = values(c.v_codes, c.v_meta, pages, n)
        out.append(_attend(values(c.k_codes, c.k_meta, pages, n)[0], V, size, qr[b], chunk, *((2 ** -21, 16) if fine else (2 ** -16, 143))))
    return torch.stack([o for o, _ in out]) @ rot.T, torch.stack([e for _, e in out])


def _same(out, ref, lens, what):
    assert torch.isfinite(out).all() and not out[lens == 0].any(), what
    want, allowed = ref
    worst = ((out.double() - want).norm(dim=-1) / allowed.clamp(min=1e-30)).max().item()
    print(f"{what}: {worst:.2f} of the bound", flush=True)
    assert worst <= 1, (what, worst)


@pytest.mark.parametrize("B,n_kv,G,d,bound,dense", [
    (257, 1, 4, 128, 64, False), (65, 4, 8, 128, 1024, False), (65, 4, 1, 128, 1025, False), (511, 1, 2, 128, 1024, False),
    (64, 8, 4, 128, 700, False), (64, 8, 4, 128, 700, True), (63, 8, 4, 128, 1280, True), (40, 8, 2, 128, 1281, True),
    (33, 8, 8, 128, 768, True), (33, 8, 8, 128, 769, True), (171, 3, 1, 128, 1984, False), (171, 3, 2, 128, 1985, False),
    (171, 3, 4, 128, 960, False), (171, 3, 4, 128, 961, False), (115, 5, 8, 128, 1025, False), (144, 4, 4, 128, 512, False),
    (144, 4, 4, 128, 513, False), (128, 8, 4, 128, 256, False), (205, 5, 4, 128, 256, False), (205, 5, 4, 128, 257, False),
    (164, 7, 2, 128, 40, True), (144, 8, 4, 128, 256, False), (144, 8, 8, 128, 257, False), (1030, 1, 4, 128, 200, False),
    (260, 8, 4, 128, 130, False), (33, 16, 4, 64, 768, False), (33, 16, 2, 64, 769, False), (64, 16, 4, 64, 400, False),
    (144, 16, 4, 64, 250, False), (135, 8, 1, 64, 1500, False), (33, 8, 8, 64, 1024, False), (33, 8, 8, 64, 1025, False), (39, 7, 4, 64, 1536, False),
    (39, 7, 4, 64, 1537, False), (96, 8, 8, 64, 300, False), (110, 7, 8, 64, 257, False), (128, 8, 8, 64, 768, False),
    (257, 3, 1, 64, 400, False), (259, 3, 1, 64, 400, False), (1, 8, 4, 128, 2600, False), (1, 16, 8, 128, 7168, True),
    (1, 16, 8, 128, 7169, True), (1, 1, 1, 128, 8192, False), (1, 16, 4, 64, 5000, False)])
def test_short_bounds(saw, B, n_kv, G, d, bound, dense):
    lens = torch.tensor(_lens(B, bound), dtype=torch.int32, device="cuda")
    c, pt, g, rot = _cache(saw, B, n_kv, d, bound, dense)
    fine = d == 64 and (n_kv % 2 == 1 or G == 8)
    q = torch.randn((B, n_kv * G, d), device="cuda", generator=g).bfloat16()
    chunk = _chunk(saw, c, B, n_kv * G, bound)
    ref = _exact(c, q, pt, lens, rot, chunk, fine)
    new = [torch.randn((B, n_kv, d), device="cuda", generator=g).bfloat16() for _ in range(2)]
    after = None
    for order in (None, saw.decode_order(lens, bound) if B <= 1024 else None):
        out = saw.paged_decode_attn(c, q, pt, lens, max_seq_len=bound, order=order)
        _same(out, ref, lens, ("decode", order is not None))
        # the fused step writes the same token to the same place each time: the second run starts from the same lengths
        got = saw.append_decode_attn(c, new[0], new[1], q, pt, lens, max_seq_len=bound, order=order)
        if after is None:
            after = _exact(c, q, pt, lens + 1, rot, _chunk(saw, c, B, n_kv * G, bound + 1), fine)
        _same(got, after, lens + 1, ("fused", order is not None))
    if 256 < B * n_kv <= 800:                                        # one partition asked for
        _same(saw.paged_decode_attn(c, q, pt, lens, max_seq_len=bound, num_splits=1), ref, lens, "one partition")


@pytest.mark.parametrize("B,n_kv,G,d,bound", [
    (257, 1, 4, 128, 256), (257, 1, 4, 128, 257), (48, 8, 1, 128, 200), (512, 4, 4, 128, 100), (3, 8, 1, 128, 256), (3, 8, 1, 128, 257),
    (28, 8, 8, 128, 320), (28, 8, 8, 128, 321), (1, 2, 4, 128, 3000), (16, 7, 4, 128, 1100), (320, 1, 4, 128, 500), (321, 1, 4, 128, 500),
    (1, 1, 4, 128, 28672), (2, 1, 8, 128, 28673), (1, 1, 8, 64, 20000), (1, 1, 4, 64, 57345), (5, 4, 4, 64, 900), (20, 8, 8, 64, 1200)])
def test_short_bounds_kv16(saw, B, n_kv, G, d, bound):
    lens = torch.tensor(_lens(B, bound), dtype=torch.int32, device="cuda")
    if B == 1:
        lens[0] = bound - 5
    need = (bound + 16) // 16
    g = torch.Generator(device="cuda").manual_seed(bound)
    c = saw.Kv16Cache(B * need, n_kv, d, torch.bfloat16)
    for t in (c.k_pages, c.v_pages):
        t.normal_(generator=g).mul_(0.5)
    pt = torch.randperm(B * need, device="cuda", generator=g).to(torch.int32).view(B, need)
    q = torch.randn((B, n_kv * G, d), device="cuda", generator=g).bfloat16()
    u, M = (2 ** -21, 2) if d == 64 or G == 8 else (2 ** -16, 2)
    ref = []
    for b, n in enumerate(lens.tolist()):
        K, V = (t[pt[b, :(n + 15) // 16].long()].permute(0, 2, 1, 3).flatten(0, 1)[:n].double() for t in (c.k_pages, c.v_pages))
        ref.append(_attend(K, V, V.abs().amax(-1) if n else V[..., 0], q[b].double(), _chunk(saw, c, B, n_kv * G, bound), u, M))
    ref = tuple(torch.stack(r) for r in zip(*ref))
    _same(saw.kv16_paged_decode_attn(c, q, pt, lens, max_seq_len=bound), ref, lens, "kv16")
