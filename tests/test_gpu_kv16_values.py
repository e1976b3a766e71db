"""16-bit decode: values that limbs of 16 bits could lose - weights far below the largest one, infinities in the cache."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [(8, 1, 128), (8, 2, 64), (4, 2, 64), (2, 3, 64), (1, 2, 64)]       # the shapes that carry fp32 weights (G, kv heads, head_dim)


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


def _pages(x, lens, pt, n_pages):
    """Dense per-sequence [L][Hkv][d] values into pages [n_pages][Hkv][16][d] (unused slots NaN)."""
    Hkv, d = x[0].shape[1:]
    out = torch.full((n_pages, Hkv, 16, d), float("nan"), dtype=x[0].dtype)
    for b, L in enumerate(lens):
        for i in range((L + 15) // 16):
            t = x[b][16 * i:min(L, 16 * i + 16)]
            out[int(pt[b, i]), :, :t.shape[0]] = t.transpose(0, 1)
    return out


def _run(saw, K, V, q, lens, splits, dtype):
    Hkv, d = K[0].shape[1:]
    need = [(n + 15) // 16 for n in lens]
    pt = np.zeros((len(lens), max(max(need), 68)), np.int32)           # (pair blocks need a bound above 1024 tokens)
    o = 0
    for b, n in enumerate(need):
        pt[b, :n] = np.arange(o, o + n)
        o += n
    kc = saw.Kv16Cache(1, Hkv, d, dtype)
    kc.num_pages = o
    kc.k_pages, kc.v_pages = _pages(K, lens, pt, o).cuda(), _pages(V, lens, pt, o).cuda()
    out = torch.full(q.shape, float("nan"), device="cuda")
    saw.kv16_paged_decode_attn(kc, q.cuda(), torch.from_numpy(pt).cuda(), torch.tensor(lens, dtype=torch.int32).cuda(),
                               num_splits=splits, out=out)
    return out.cpu().double()


def _exact(K, V, q, G):
    """fp64 attention of one sequence: K, V [L][Hkv][d], q [Hq][d]."""
    k, v = K.double().transpose(0, 1), V.double().transpose(0, 1)
    Hkv, L, d = k.shape
    s = q.double().reshape(Hkv, G, 1, d) * k.reshape(Hkv, 1, L, d)
    p = torch.softmax(s.sum(-1) / np.sqrt(d), -1)                    # (a sum with one infinity is that infinity)
    return (p[..., None] * v[:, None]).sum(2).reshape(Hkv * G, d)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("L,B", [(8000, 2), (600, 260)])
def test_weights_far_below_the_largest_one(saw, dtype, G, Hkv, d, L, B):
    """One token `gap` powers of two above a long tail whose values have a mean: the tail is up to nearly all of the output
    and none of its weights may be lost.  B = 260: pair blocks.  A logit of `gap` base-2 units carries 2^-23 of itself in
    fp32, the tail's share of the output as much of itself times ln 2: 25 2^-23 ln 2 = 2e-6.  The running sums, of values and
    of weights, hold the dominant token while L / 32 batches are added to them, each of which rounds by 2^-25 of them.  With a
    small gap the sums grow evenly and round at random: sqrt(L / 32) 2^-25, a few units of 1e-7."""
    g = torch.Generator().manual_seed(L + G)
    for gap in (6, 14, 18, 22, 25):
        n = 3 if B > 2 else B
        K, V, Q, want = [], [], [], []
        for b in range(n):
            q = torch.randn((Hkv * G, d), generator=g)
            q = q.reshape(Hkv, G, d)[:, :1].expand(Hkv, G, d).reshape(Hkv * G, d) * torch.linspace(1.0, 0.9, Hkv * G)[:, None]
            k = 0.05 * torch.randn((L, Hkv, d), generator=g)
            q0 = q.reshape(Hkv, G, d)[:, 0]
            k[L // 3] = gap * np.log(2) * np.sqrt(d) * q0 / (q0 * q0).sum(-1, keepdim=True)
            v = 1 + 0.25 * torch.randn((L, Hkv, d), generator=g)
            v[L // 3] = 0.02
            k, v = k.to(dtype), v.to(dtype)
            K.append(k), V.append(v), Q.append(q), want.append(_exact(k, v, q, G))
        idx = [i % n for i in range(B)]
        want = torch.stack([want[i] for i in idx])
        for splits in (1, 0, 3):
            got = _run(saw, [K[i] for i in idx], [V[i] for i in idx], torch.stack([Q[i] for i in idx]), [L] * B, splits, dtype)
            err = float((got - want).abs().max() / want.abs().max())
            print(f"[kv16 sink {dtype} G={G} Hkv={Hkv} d={d} L={L} gap={gap} splits={splits}] {err:.2e}", flush=True)
            assert err < (1.5e-6 if gap == 6 else 2e-6 + L / 32 * 2.0 ** -24)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("G,Hkv,d", SHAPES)
@pytest.mark.parametrize("B", [2, 260])
def test_infinities_as_in_fp32(saw, dtype, G, Hkv, d, B):
    """A key with an infinite channel gives logits of -inf, which have no weight, or of +inf, which make the row NaN; an
    infinite value makes its channel infinite.  Every other row and channel is what it is without them."""
    g = torch.Generator().manual_seed(G + d)
    L, lens = 300, [300 - 41 * (b % 7) if b > 1 else 300 for b in range(B)]
    q = torch.randn((B, Hkv * G, d), generator=g).abs() + 0.1          # (every query has the key's -inf as a logit of -inf)
    K = [torch.randn((L, Hkv, d), generator=g).to(dtype) for _ in range(2)]
    V = [torch.randn((L, Hkv, d), generator=g).to(dtype) for _ in range(2)]
    K[0][7, 0, 3] = K[0][30, 0, d - 1] = K[0][L - 1, 0, 0] = float("-inf")
    V[0][20, 0, 5], V[0][41, Hkv - 1, d - 2] = float("inf"), float("-inf")
    V[1][9, 0, 1] = float("inf")
    idx = [b % 2 for b in range(B)]
    want = torch.stack([_exact(K[i][:lens[b]], V[i][:lens[b]], q[b], G) for b, i in enumerate(idx)])
    assert not want.isnan().any()
    for splits in (1, 0, 2):
        got = _run(saw, [K[i] for i in idx], [V[i] for i in idx], q, lens, splits, dtype)
        assert not got.isnan().any() and torch.equal(got.isinf(), want.isinf())
        assert torch.equal(got[got.isinf()], want[want.isinf()])
        err = float((got - want)[~want.isinf()].abs().max() / want[~want.isinf()].abs().max())
        print(f"[kv16 inf {dtype} G={G} Hkv={Hkv} d={d} B={B} splits={splits}] {err:.2e}", flush=True)
        assert err < 4e-6
    K[1][33, Hkv - 1, 2] = float("inf")
    got = _run(saw, [K[i] for i in idx], [V[i] for i in idx], q, lens, 0, dtype)
    assert got[1, (Hkv - 1) * G:].isnan().all() and not got[0].isnan().any()
