"""Batches cut into partitions by their own lengths (saw_cut.h): the rule itself, mirrored on the CPU, and the decode
calls that use it against the one-partition call of the same shape."""
import numpy as np
import pytest
import torch

import parity
from paper_2604_19157_amd import synth


def _parts(n, c):
    """The kernel's ceil(n / c): an fp32 product with the reciprocal, off by one at most, put right."""
    x = np.asarray(n, np.int64) + c - 1
    q = (x.astype(np.float32) * (np.float32(1) / np.float32(c))).astype(np.int64)
    r = x - q * c
    return q + (r >= c) - (r < 0)


def _cut(nb, W, cmin=4):
    B, T = len(nb), int(sum(nb))
    lo = max(cmin, int(_parts(T, W)))
    if int(_parts(nb, lo).sum()) > W:
        hi = max(lo, int(_parts(T, W - B)))
        assert int(_parts(nb, hi).sum()) <= W
        while hi - lo > 1:
            mid = (lo + hi) // 2
            if int(_parts(nb, mid).sum()) > W:
                lo = mid
            else:
                hi = mid
        lo = hi
    return lo


def test_quotients_are_exact():
    rng = np.random.default_rng(1)
    for c in [1, 2, 3, 7, 64, 255, 256, 1023, 4095, 65537, (1 << 22) - 1]:
        n = np.concatenate([np.arange(0, 4 * c if c < 5000 else 20000), rng.integers(0, 1 << 23, 20000) - c % (1 << 22)])
        n = n[(n >= 0) & (n + c - 1 < 1 << 23)]
        assert np.array_equal(_parts(n, c), -(-n // c)), c


def test_slots_cover_every_batch_once():
    rng = np.random.default_rng(2)
    for _ in range(300):
        B = int(rng.integers(2, 257))
        W = int(rng.integers(2 * B, 1025))
        nb = rng.integers(0, int(rng.choice([2, 9, 70, 3000])), size=B)
        if rng.random() < 0.3:
            nb[rng.integers(0, B)] = 20000
        c = _cut(nb, W)
        P = _parts(nb, c)
        assert P.sum() <= W and np.array_equal(P == 0, nb == 0)
        if c > 4:                                                      # the smallest that fits
            assert _parts(nb, c - 1).sum() > W or c - 1 < -(-int(nb.sum()) // W)
        for n, p in zip(nb.tolist(), P.tolist()):
            at = 0
            for i in range(p):
                q, r = n // p, n % p
                first, end = i * q + min(i, r), i * q + min(i, r) + q + (i < r)
                assert first == at and 0 < end - first <= c
                at = end
            assert at == n


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,kw", [(2, 32, 8, {}), (15, 64, 8, {}), (63, 32, 8, {"dtype": torch.float16}), (64, 4, 4, {"sign_seed": 2}),
                                         (65, 8, 2, {"had_block": 16}), (129, 2, 1, {"rotate_mask": 1}), (250, 8, 1, {}),
                                         (40, 8, 8, {"dense_seed": 3}), (20, 16, 2, {"dense_seed": 3, "rotate_mask": 2}),
                                         (33, 32, 8, {"head_dim": 64, "had_block": 64}), (120, 4, 4, {"head_dim": 64, "had_block": 32})])
def test_cut_batches_agree_with_one_partition(saw, B, Hq, Hkv, kw):
    """Ragged lengths with empty sequences, partition and page edges and one sequence as long as all others together,
    under a tight and a loose bound; decode and fused append; fp32 outputs.  Both calls carry q and P in two bf16
    limbs (2^-16 of each): 1e-4 of the largest output, as the schedules' agreement elsewhere."""
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 900, size=B)
    lens[rng.integers(0, B, size=B // 6)] = 0
    lens[: min(B, 8)] = [0, 6000, 256, 257, 64, 1, 2600, 255][: min(B, 8)]
    w = synth.make_workload("highconc", batch=B, seq_lens=lens, n_q_heads=Hq, n_kv_heads=Hkv, table_width=1100, **kw)
    cache = saw.Cache(w.num_pages, Hkv, w.head_dim, w.had_block, w.rotate_mask, signs=w.signs, dense=w.dense)
    pt, sl = torch.from_numpy(w.page_table).cuda(), torch.from_numpy(w.seq_lens).cuda()
    for b in range(B):
        if lens[b]:
            K, V = synth.gen_kv(w, b, 0, int(lens[b]), device="cuda")
            saw.rotate_quant_store(cache, K, V, pt, torch.from_numpy(synth.slots_for(b, 0, int(lens[b]))).cuda())
    q = synth.gen_q(w, device="cuda")
    want = saw.paged_decode_attn(cache, q, pt, sl, num_splits=1).cpu().numpy()
    for bound in (int(lens.max()), 0):
        got = torch.full((B, Hq, w.head_dim), float("nan"), device="cuda")
        ws = torch.full((saw.decode_workspace_bytes(cache, B, Hq, bound or 17600),), 0xFF, dtype=torch.uint8, device="cuda")
        saw.paged_decode_attn(cache, q, pt, sl, max_seq_len=bound, out=got, workspace=ws)
        err = parity.attn_error(got.cpu().numpy(), want)
        print(f"[cut B={B} Hq={Hq}/{Hkv} {kw} bound={bound}] {err:.2e}", flush=True)
        assert err < 1e-4
    K = torch.randn((B, Hkv, w.head_dim), device="cuda").to(w.dtype)
    V = torch.randn((B, Hkv, w.head_dim), device="cuda").to(w.dtype)
    o = [saw.append_decode_attn(cache, K, V, q, pt, sl, max_seq_len=bound) for bound in (int(lens.max()), 0)]
    want = saw.paged_decode_attn(cache, q, pt, sl + 1, num_splits=1).cpu().numpy()
    for x in o:
        assert parity.attn_error(x.cpu().numpy(), want) < 1e-4
