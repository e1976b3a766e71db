"""Short bounds: several wavefronts over each whole sequence instead of partitions, pair blocks and the in-kernel ranking; the
16-bit call's shorter partitions.

Both sides of each line of the rules, in (sequence, kv head) items and in tokens, decode and fused step, with and without the
caller's order, 64-channel heads in pairs and one at a time, a learned rotation and the 16-bit cache; lengths from zero to the bound.  The call's own
plan against two fixed partitions per sequence and their merge pass: the same products, with weights that both sides round to bf16
against their own running maximum.  One weight p is off by at most 2^-9 p on either side; over n tokens of about equal weight these
roundings, of either sign, add up to 2^-8 |v| / sqrt(n) in the norm of an output row (twice that is allowed), |v| <= 0.8 sqrt(d) here."""
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


def _cache(saw, B, n_kv, d, bound, dense):
    need = (bound + 16) // 16
    c = saw.Cache(B * need, n_kv, d, 64, 3, dense=torch.linalg.qr(torch.randn(128, 128, generator=torch.Generator().manual_seed(7)))[0] if dense else None)
    g = torch.Generator(device="cuda").manual_seed(B + bound)
    for codes, meta in ((c.k_codes, c.k_meta), (c.v_codes, c.v_meta)):
        codes.random_(0, 256, generator=g)
        meta[..., 0] = 0.1
        meta[..., 1] = 7.0
    pt = torch.randperm(B * need, device="cuda", generator=g).to(torch.int32).view(B, need)
    return c, pt, g


def _same(out, ref, lens, what):
    assert torch.isfinite(out).all(), what
    d = out.shape[-1]
    off = (out - ref).norm(dim=-1)
    allowed = 2 ** -7 * 0.8 * d ** 0.5 / lens.clamp(min=1).float().sqrt()
    worst = (off / allowed[:, None]).max().item()
    assert worst <= 1, (what, worst)


@pytest.mark.parametrize("B,n_kv,G,d,bound,dense", [
    (257, 1, 4, 128, 64, False), (65, 4, 8, 128, 1535, False), (65, 4, 1, 128, 1536, False), (511, 1, 2, 128, 1537, False),
    (64, 8, 4, 128, 700, False), (64, 8, 4, 128, 700, True), (63, 8, 4, 128, 2047, True), (171, 3, 1, 128, 960, False),
    (171, 3, 4, 128, 961, False), (115, 5, 8, 128, 1025, False), (144, 4, 4, 128, 512, False), (144, 4, 4, 128, 513, False),
    (128, 8, 4, 128, 256, False), (205, 5, 4, 128, 256, False), (205, 5, 4, 128, 257, False), (164, 7, 2, 128, 40, True),
    (144, 8, 4, 128, 256, False), (144, 8, 8, 128, 257, False), (1030, 1, 4, 128, 200, False), (260, 8, 4, 128, 130, False),
    (33, 16, 4, 64, 1279, False), (33, 16, 2, 64, 1281, False), (64, 16, 4, 64, 400, False), (144, 16, 4, 64, 250, False),
    (33, 8, 8, 64, 1536, False), (33, 8, 8, 64, 1537, False), (96, 8, 8, 64, 300, False), (110, 7, 8, 64, 257, False),
    (128, 8, 8, 64, 768, False), (257, 3, 1, 64, 400, False), (259, 3, 1, 64, 400, False),
    (1, 8, 4, 128, 2600, False), (1, 16, 8, 128, 8191, True), (1, 1, 1, 128, 8192, False), (1, 16, 4, 64, 5000, False)])
def test_short_bounds(saw, B, n_kv, G, d, bound, dense):
    lens = torch.tensor(_lens(B, bound), dtype=torch.int32, device="cuda")
    c, pt, g = _cache(saw, B, n_kv, d, bound, dense)
    q = torch.randn((B, n_kv * G, d), device="cuda", generator=g).bfloat16()
    ref = saw.paged_decode_attn(c, q, pt, lens, max_seq_len=bound, num_splits=2 if bound > 64 else 1).float()
    new = [torch.randn((B, n_kv, d), device="cuda", generator=g).bfloat16() for _ in range(2)]
    after = None
    for order in (None, saw.decode_order(lens, bound) if B <= 1024 else None):
        out = saw.paged_decode_attn(c, q, pt, lens, max_seq_len=bound, order=order).float()
        _same(out, ref, lens, ("decode", order is not None))
        # the fused step writes the same token to the same place each time: the second run starts from the same lengths
        got = saw.append_decode_attn(c, new[0], new[1], q, pt, lens, max_seq_len=bound, order=order).float()
        if after is None:
            after = saw.paged_decode_attn(c, q, pt, lens + 1, max_seq_len=bound + 1, num_splits=2).float()
        _same(got, after, lens + 1, ("fused", order is not None))


@pytest.mark.parametrize("B,n_kv,G,bound", [(257, 1, 4, 256), (257, 1, 4, 257), (48, 8, 1, 200), (512, 4, 4, 100),
                                           (3, 8, 1, 256), (3, 8, 1, 257), (28, 8, 8, 320), (28, 8, 8, 321), (1, 2, 4, 3000),
                                           (16, 7, 4, 1100), (320, 1, 4, 500), (321, 1, 4, 500)])
def test_short_bounds_kv16(saw, B, n_kv, G, bound):
    lens = torch.tensor(_lens(B, bound), dtype=torch.int32, device="cuda")
    need = (bound + 16) // 16
    g = torch.Generator(device="cuda").manual_seed(bound)
    c = saw.Kv16Cache(B * need, n_kv, 128, torch.bfloat16)
    for t in (c.k_pages, c.v_pages):
        t.normal_(generator=g).mul_(0.5)
    pt = torch.randperm(B * need, device="cuda", generator=g).to(torch.int32).view(B, need)
    q = torch.randn((B, n_kv * G, 128), device="cuda", generator=g).bfloat16()
    ref = saw.kv16_paged_decode_attn(c, q, pt, lens, max_seq_len=bound, num_splits=2).float()
    out = saw.kv16_paged_decode_attn(c, q, pt, lens, max_seq_len=bound).float()
    _same(out, ref, lens, "kv16")
