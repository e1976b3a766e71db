"""What a fused step stores for a token does not depend on the batch around it: with a learned rotation, whose products are sums
of 128 terms, every way of handing out work gives the same codes, scales and zero-points, bit for bit."""
import pytest
import torch

import gpu_cases as gc

pytestmark = pytest.mark.gpu
N_KV = 2
# sequences, columns of the page table (x 16: the bound), how the step is handed out
ROUTES = {"one wavefront": (1030, 1, dict(partitions=1, waves=1, pair_seqs=0)), "blocks of eight": (100, 1, dict(partitions=1, waves=8)),
          "blocks of four": (250, 1, dict(partitions=1, waves=4, pair_seqs=0)), "blocks of two": (500, 1, dict(partitions=1, waves=2, pair_seqs=0)),
          "pair blocks of four": (500, 128, gc.pairs(4)), "of four over three sequences": (700, 128, gc.pairs(4, 3)), "of two": (900, 128, gc.pairs(2)),
          "cut, four a slot": (20, 512, dict(partitions=0, waves=4)), "cut, two a slot": (120, 512, dict(partitions=0, waves=2)),
          "one sequence in partitions": (1, 512, dict(partitions=128, waves=1))}


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("mask,h,G", [(3, 128, 4), (3, 16, 8), (3, 1, 1), (1, 64, 2), (2, 64, 4)])
def test_stored_bytes_do_not_depend_on_the_schedule(saw, mask, h, G):
    g = torch.Generator(device="cuda").manual_seed(h + G)
    R = torch.linalg.qr(torch.randn(128, 128, generator=torch.Generator().manual_seed(7)))[0]
    n = max(B for B, _, _ in ROUTES.values())
    K, V = (torch.randn((n, N_KV, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    K[3], V[5] = 0.75, 0.0                                             # constant vectors
    q = torch.randn((n, N_KV * G, 128), device="cuda", generator=g).bfloat16()
    lens = (torch.arange(n, device="cuda") % 15 + 1).to(torch.int32)
    want = None
    for name, (B, width, expect) in ROUTES.items():
        c = saw.Cache(B, N_KV, 128, h, mask, dense=R)
        gc.check_schedule(saw, c, B, N_KV * G, 16 * width, expect)
        pt = torch.zeros((B, width), dtype=torch.int32, device="cuda")
        pt[:, 0] = torch.arange(B, device="cuda")
        out = saw.append_decode_attn(c, K[:B], V[:B], q[:B], pt, lens[:B])
        got = [t.view(torch.uint8).flatten(1).cpu() for t in (c.k_codes, c.v_codes, c.k_meta, c.v_meta)]
        assert torch.isfinite(out).all() and all(t.any(1).sum() >= B - 1 for t in got[2:]), name
        print(name, flush=True)
        want = want or got
        for i, (a, b) in enumerate(zip(got, want)):
            assert torch.equal(a, b[:B]), (name, i, int((a != b[:B]).any(1).sum()))
