"""Parity of the head_dim 64 INT4 decode with the fp64 oracle (Sec. 4.1, App. A.4: the block-diagonal
rotation only needs h | d, so 64-channel heads are served too).

With an even number of kv heads and at most 4 query heads per kv head the matrix-core kernel runs on
pairs of kv heads; other shapes take the kernel of one 64-channel head at a time.  Every way the kernel hands out work is
driven here at head_dim 64: one partition, split-KV with the merge pass, several wavefronts per
partition, pair mode, longest-first order, and the append entry point.
"""
import numpy as np
import pytest
import torch

import gpu_cases as gc
import test_gpu_append as TA
import test_gpu_decode as TD
from paper_2604_19157_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    binding.lib()
    return binding


def _w(name="highconc", **kw):
    kw.setdefault("head_dim", 64)
    kw.setdefault("had_block", 64)
    return synth.make_workload(name, **kw)


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (4, 2), (8, 2), (8, 8), (32, 8), (6, 6)])
def test_head_pairs_group_sizes(saw, Hq, Hkv):
    TD._decode_case(saw, _w(batch=3, ctx=(20, 150), n_q_heads=Hq, n_kv_heads=Hkv))


@pytest.mark.parametrize("Hq,Hkv", [(3, 3), (6, 3), (16, 2), (5, 5)])
def test_shapes_outside_the_pair_kernel(saw, Hq, Hkv):
    """Odd kv head counts and 8 query heads per kv head: the kernel of one 64-channel head at a time."""
    TD._decode_case(saw, _w(batch=3, ctx=(20, 150), n_q_heads=Hq, n_kv_heads=Hkv))


@pytest.mark.parametrize("h,mask", [(1, 3), (16, 3), (32, 3), (64, 3), (64, 1), (32, 2), (64, 0)])
@pytest.mark.parametrize("sign_seed", [None, 5])
def test_head_pairs_block_sizes_masks_signs(saw, h, mask, sign_seed):
    w = _w(batch=2, ctx=(40, 200), n_q_heads=16, n_kv_heads=4, had_block=h, rotate_mask=mask, sign_seed=sign_seed)
    TD._decode_case(saw, w)


@pytest.mark.parametrize("splits", [1, 2, 3, 0])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (8, 4), (16, 4)])
def test_head_pairs_split_kv(saw, splits, Hq, Hkv):
    w = _w("tiny", batch=3, ctx=(130, 700), n_q_heads=Hq, n_kv_heads=Hkv)
    TD._decode_case(saw, w, num_splits=splits, end_to_end=False)


def test_head_pairs_ragged_with_empty_and_single(saw):
    w = _w(batch=7, seq_lens=[0, 1, 15, 16, 17, 64, 333], n_q_heads=16, n_kv_heads=4)
    o, _ = TD._decode_case(saw, w, num_splits=2)
    assert not o[0].any()
    o, _ = TD._decode_case(saw, w, num_splits=1, end_to_end=False)
    assert not o[0].any()


@pytest.mark.parametrize("B,Hq,Hkv", [(140, 32, 8), (140, 16, 4), (150, 32, 8), (255, 8, 8), (300, 8, 8), (340, 16, 8),
                                      (340, 32, 8), (600, 8, 8)])
def test_head_pairs_many_sequences(saw, B, Hq, Hkv):
    """More (sequence, head pair) items than compute units, under a bound of 1024 tokens: four wavefronts a sequence (560 and
    280 items, the first two cases; the second by itself is cut by its lengths), pair mode (blocks of four from 576 to 1024 items: the third and fourth case; of four over three
    sequences from 1152 to 1536 items: the fifth and sixth, while the seventh, with eight query rows per head pair, takes blocks of two),
    longest first beyond 2304 items (the last case).
    Lengths include empty sequences and many ties."""
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 200, size=B)
    lens[rng.integers(0, B, size=B // 5)] = 64
    lens[:3] = [0, 199, 1]
    w = _w(batch=B, seq_lens=lens, n_q_heads=Hq, n_kv_heads=Hkv, table_width=64)
    items = B * Hkv // 2
    expect = gc.pairs(2) if 1152 <= items <= 2048 and Hq == 4 * Hkv else gc.by_items(items)
    TD._decode_case(saw, w, num_splits=1, end_to_end=False, max_seq_len=0, expect=expect)
    TD._decode_case(saw, w, num_splits=0, end_to_end=False, max_seq_len=0, expect=dict(partitions=0) if items < 512 else expect)


def test_head_pairs_long_context_several_wavefronts(saw):
    w = _w("longctx1", ctx=9000, n_q_heads=8, n_kv_heads=2)
    TD._decode_case(saw, w, num_splits=0, end_to_end=False)
    TD._decode_case(saw, w, num_splits=1, end_to_end=False)       # one partition, four wavefronts on it
    TD._decode_case(saw, w, num_splits=37, end_to_end=False)


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float16])
def test_head_pairs_output_and_query_dtypes(saw, out_dtype):
    w = _w("tiny", batch=2, ctx=75, n_q_heads=8, n_kv_heads=4)
    TD._decode_case(saw, w, out_dtype=out_dtype, q_dtype=torch.float32, sm_scale=0.11)


def test_head_pairs_fp16_cache_input(saw):
    TD._decode_case(saw, _w("tiny", batch=2, ctx=(30, 300), n_q_heads=8, n_kv_heads=2, dtype=torch.float16))


@pytest.mark.parametrize("B,Hq,Hkv,ctx", [(3, 8, 4, (20, 150)), (70, 32, 8, (1, 120)), (150, 16, 8, (0, 200)),
                                          (2, 8, 2, (700, 900))])
def test_append_then_attend(saw, B, Hq, Hkv, ctx):
    """saw_append_decode_attn at head_dim 64: what a store followed by a decode over one more token gives."""
    TA._case(saw, _w(batch=B, ctx=ctx, n_q_heads=Hq, n_kv_heads=Hkv))


@pytest.mark.parametrize("h,mask,sign_seed", [(64, 3, 5), (16, 3, None), (32, 1, 6), (64, 2, None), (1, 3, None)])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (16, 4)])
def test_append_block_sizes_masks_signs(saw, h, mask, sign_seed, Hq, Hkv):
    """The decode kernel's own append at head_dim 64: the new token's bytes per kv head of a pair."""
    TA._case(saw, _w(batch=4, ctx=(1, 200), n_q_heads=Hq, n_kv_heads=Hkv, had_block=h, rotate_mask=mask,
                     sign_seed=sign_seed))


def test_append_unmapped_page_and_odd_kv_heads(saw):
    # (the unmapped token must open a page of its own, or cached tokens would lose their page with it)
    TA._case(saw, _w(batch=3, seq_lens=[40, 64, 95], n_q_heads=8, n_kv_heads=4), unmapped=(1,))
    TA._case(saw, _w(batch=3, ctx=(20, 150), n_q_heads=6, n_kv_heads=3))


@pytest.mark.parametrize("Hq,Hkv,dtype,kw", [(8, 1, torch.bfloat16, {}), (3, 3, torch.float16, {"rotate_mask": 1}),
                                             (6, 3, torch.bfloat16, {"sign_seed": 3, "had_block": 16}),
                                             (4, 1, torch.float16, {"rotate_mask": 2, "sign_seed": 4}),
                                             (64, 8, torch.float16, {"had_block": 1})])
@pytest.mark.parametrize("B", [1, 16, 70, 300])
def test_one_head_at_a_time_batch_edges(saw, Hq, Hkv, dtype, kw, B):
    """Lengths around the 64-token batches and the pages, empty sequences, a long one: fixed partitions, a batch cut by
    its own lengths (automatic, up to 256 sequences; under a tight and a loose bound), one partition, and the fused
    append against store + decode.  The query and the weights carry 24 bits and the codes are exact, so what is left is
    the rounding of fp32 sums: Sum w c of up to 15 s, from which about half is taken away again with the zero-points
    (2^-24 a step of that, tens of steps: 2^-20 s), against outputs of a few s that shrink with sqrt(L) as the values
    average out: 4e-6 sqrt(max(L / 300, 1)) of the largest output."""
    from oracle import saw_oracle as O
    import parity
    rng = np.random.default_rng(B + Hq)
    limit = 4e-6 * (5000 / 300 if B == 1 else 1) ** 0.5
    edges = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 300, 1030, 255, 256, 257]
    lens = (edges * (B // 16 + 1))[:B] if B > 1 else [5000]
    w = _w(batch=B, seq_lens=lens, n_q_heads=Hq, n_kv_heads=Hkv, dtype=dtype, table_width=400, **kw)
    ref = gc.oracle_fill(w)
    cache = gc.upload_cache(ref, w, saw)
    pt, sl = torch.from_numpy(w.page_table).cuda(), torch.from_numpy(w.seq_lens).cuda()
    q = synth.gen_q(w).float() * 0.5
    want = O.paged_decode_attn(ref, q.numpy(), w.page_table, w.seq_lens, w.had_block, w.rotate_mask, signs=w.signs)
    for splits, bound in ((0, max(lens)), (0, 0), (1, 0), (3, 0)):
        out = torch.full((B, Hq, 64), float("nan"), device="cuda")
        saw.paged_decode_attn(cache, q.cuda(), pt, sl, max_seq_len=bound, out=out, num_splits=splits)
        err = parity.attn_error(out.cpu().numpy(), want)
        print(f"[one head at a time B={B} Hq={Hq}/{Hkv} splits={splits} bound={bound}] err={err:.2e}", flush=True)
        assert err < limit
        assert not out[[b for b in range(B) if lens[b] == 0]].any()
    # a scratch sized for the fixed partitions of the plan is enough
    s, _ = saw.decode_plan(cache, B, max(lens))
    ws = torch.empty(max(16, B * Hq * s * 66 * 4), dtype=torch.uint8, device="cuda")
    out = saw.paged_decode_attn(cache, q.cuda(), pt, sl, max_seq_len=max(lens), workspace=ws)
    assert parity.attn_error(out.cpu().numpy(), want) < limit
    # fused append: the attention of store + decode (a code on a rounding boundary may differ: one step of one value of
    # one token), and every stored token under the store criterion
    K = torch.from_numpy(rng.standard_normal((B, Hkv, 64))).to(dtype).cuda()
    V = torch.from_numpy(rng.standard_normal((B, Hkv, 64))).to(dtype).cuda()
    two = gc.upload_cache(ref, w, saw)
    slots = torch.from_numpy(np.stack([np.arange(B), w.seq_lens], 1).astype(np.int32)).cuda()
    saw.rotate_quant_store(two, K, V, pt, slots)
    o2 = saw.paged_decode_attn(two, q.cuda(), pt, sl + 1, num_splits=1)
    for bound in (max(lens), 0):
        o1 = saw.append_decode_attn(cache, K, V, q.cuda(), pt, sl, max_seq_len=bound)
        same = (cache.k_codes == two.k_codes).flatten(1).all(1) & (cache.v_codes == two.v_codes).flatten(1).all(1)
        assert (~same).sum() <= 2
        last = torch.tensor([w.page_table[b, n // 16] for b, n in enumerate(lens)]).cuda()
        rows = same[last].cpu().numpy()
        assert parity.attn_error(o1.cpu().numpy()[rows], o2.cpu().numpy()[rows]) < 2 * limit
    if B <= 70:
        TA._case(saw, w)


@pytest.mark.parametrize("Hq,Hkv", [(8, 1), (3, 3), (16, 2)])
@pytest.mark.parametrize("B", [2, 40, 300])
def test_append_of_a_length_below_zero_stores_nothing(saw, Hq, Hkv, B):
    """Such a sequence has no position for its token: its pages stay as they are, and the others' tokens are stored."""
    lens = [50 + (37 * b) % 900 for b in range(B)]
    w = _w(batch=B, seq_lens=lens, n_q_heads=Hq, n_kv_heads=Hkv, table_width=400)
    cache = gc.upload_cache(gc.oracle_fill(w), w, saw)
    pt = torch.from_numpy(w.page_table).cuda()
    sl = torch.tensor([-1 - b % 5 if b % 3 == 1 else n for b, n in enumerate(lens)], dtype=torch.int32).cuda()
    before = cache.k_codes.clone(), cache.v_codes.clone(), cache.k_meta.clone(), cache.v_meta.clone()
    K = torch.randn((B, Hkv, 64), device="cuda").to(w.dtype)
    saw.append_decode_attn(cache, K, K, synth.gen_q(w).cuda(), pt, sl)
    same = [(a == b).flatten(1).all(1).cpu() for a, b in zip(before, (cache.k_codes, cache.v_codes, cache.k_meta, cache.v_meta))]
    for b, n in enumerate(lens):
        mine = torch.from_numpy(w.page_table[b, : (n + 15) // 16]).long()
        if b % 3 == 1:
            assert all(s[mine].all() for s in same)
        else:
            assert not same[2][int(w.page_table[b, n // 16])]


def test_a_bound_beyond_what_can_be_cut_keeps_partitions(saw):
    """256 sequences under the bound of a page table of two million tokens: more 64-token batches than the device's cut
    counts, so the batch is split by that bound, and every partition that runs leaves a record in the workspace."""
    B, Hq, width = 256, 8, 131072
    w = _w(batch=B, seq_lens=[100 + b for b in range(B)], n_q_heads=Hq, n_kv_heads=1, table_width=32)
    cache = gc.upload_cache(gc.oracle_fill(w), w, saw)
    pt = torch.zeros((B, width), dtype=torch.int32, device="cuda")
    pt[:, :32] = torch.from_numpy(w.page_table).cuda()
    sl, q = torch.from_numpy(w.seq_lens).cuda(), synth.gen_q(w).cuda()
    ws = torch.full((saw.decode_workspace_bytes(cache, B, Hq, 16 * width),), 0xFF, dtype=torch.uint8, device="cuda")
    out = saw.paged_decode_attn(cache, q, pt, sl, workspace=ws)
    assert saw.decode_plan(cache, B, 16 * width)[0] > 1 and (ws != 0xFF).any()
    want = saw.paged_decode_attn(cache, q, pt[:, :32].contiguous(), sl, num_splits=1)
    import parity
    assert parity.attn_error(out.cpu().numpy(), want.cpu().numpy()) < 1e-5
