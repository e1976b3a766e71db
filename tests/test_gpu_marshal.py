"""The two marshalling modules of the binding, native and ctypes, make the same calls."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 40])
def test_native_and_ctypes_make_the_same_calls(monkeypatch, T):
    from paper_2604_19157_amd import binding as saw
    from paper_2604_19157_amd import marshal_ctypes
    saw.lib()
    g = torch.Generator(device="cuda").manual_seed(T)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    B, Hq, Hkv, d, signs = 3, 8, 2, 128, [1.0, -1.0] * 64
    pt = torch.randperm(B * 8, device="cuda").int().reshape(B, 8)
    slots = torch.tensor([(b, t) for b in range(B) for t in range(T)], dtype=torch.int32, device="cuda")
    K, V = ([rnd(B * T, Hkv, d) for _ in range(2)] for _ in range(2))
    q, new, lens = rnd(B, Hq, d), [rnd(B, Hkv, d) for _ in range(2)], torch.full((B,), T, dtype=torch.int32, device="cuda")
    kp = [rnd(B * 8, Hkv, 16, d) for _ in range(2)]
    got = []
    for native in (saw._marshal(), marshal_ctypes):
        monkeypatch.setattr(saw, "_native", native)
        caches = [saw.Cache(B * 8, Hkv, d, 64, signs=signs) for _ in range(2)]
        saw.rotate_quant_store(caches[0], K[0], V[0], pt, slots)
        saw.rotate_quant_store_layers(caches, K, V, pt, slots)
        order = saw.decode_order(lens)
        out = [saw.paged_decode_attn(caches[0], q, pt, lens), saw.paged_decode_attn(caches[1], q, pt, lens, max_seq_len=T, num_splits=1, sm_scale=0.1, order=order),
               saw.append_decode_attn(caches[1], new[0], new[1], q, pt, lens, order=order), *saw.flatten_dequant(caches[1], pt, 1, 0, T + 1)]
        k16 = saw.Kv16Cache(B * 8, Hkv, d, torch.bfloat16)
        k16.k_pages, k16.v_pages = kp
        out.append(saw.kv16_paged_decode_attn(k16, q, pt, lens, out_dtype=torch.bfloat16))
        got.append(out + [t for c in caches for t in (c.k_codes, c.v_codes, c.k_meta, c.v_meta)])
    for i, (a, b) in enumerate(zip(*got)):
        assert a.dtype == b.dtype and torch.equal(a, b), i
