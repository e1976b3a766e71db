"""How a decode call is handed to the chip, read from saw_decode_schedule on both sides of each line of the rules (no GPU): a line
that moves shows here, and the GPU tests of one schedule ask for it by name (gpu_cases.check_schedule)."""
import os

import pytest

from gpu_cases import pairs


@pytest.fixture(scope="module")
def saw():
    from paper_2604_19157_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2604_19157_amd import build
        build.build_library()
    return binding


def _got(saw, B, n_kv, G, bound, d=128, splits=0, order=False, cache16=False, learned=False):
    import torch
    c = saw.Kv16Cache(1, n_kv, d, torch.bfloat16, device="cpu") if cache16 else saw.Cache(1, n_kv, d, 64, device="cpu")
    if learned:
        c.dense_rot = torch.zeros(16, dtype=torch.uint8)               # (its presence is what the plan asks for)
    return saw.decode_schedule(c, B, n_kv * G, bound, splits, order)


def whole(waves):
    return dict(partitions=1, waves=waves, pair_seqs=0, longest_first=0)


FIRST = dict(partitions=1, waves=1, pair_seqs=0, longest_first=1)


@pytest.mark.parametrize("want,args,kw", [
    # 128-channel rows, one partition: by items and bound
    (whole(8), (32, 8, 4, 2304), {}), (whole(4), (33, 8, 4, 512), {}), (whole(4), (64, 8, 4, 4096), {}),
    (whole(2), (65, 8, 4, 960), {}), (whole(4), (65, 8, 4, 961), {}), (whole(2), (140, 4, 1, 1984), {}), (whole(4), (140, 4, 1, 1985), {}), (whole(2), (140, 4, 2, 1984), {}),
    (whole(2), (140, 8, 1, 1984), dict(d=64)), (whole(4), (140, 8, 2, 1984), dict(d=64)), (whole(2), (72, 8, 4, 512), {}), (pairs(4), (72, 8, 4, 513), {}), (whole(4), (71, 8, 4, 4096), {}),
    (pairs(4), (128, 8, 4, 4096), {}), (whole(2), (129, 8, 4, 4096), {}), (whole(2), (143, 8, 4, 4096), {}), (pairs(4, 3), (144, 8, 4, 4096), {}),
    (pairs(4, 3), (192, 8, 4, 4096), {}), (pairs(2), (193, 8, 4, 4096), {}), (pairs(2), (256, 8, 4, 4096), {}),
    (pairs(2, 3), (257, 8, 4, 4096), {}), (pairs(2, 3), (288, 8, 4, 4096), {}), (FIRST, (289, 8, 4, 4096), {}),
    (whole(1), (256, 8, 4, 256), {}), (pairs(2), (256, 8, 4, 257), {}), (whole(1), (400, 8, 4, 256), {}), (FIRST, (400, 8, 4, 257), {}),
    (whole(1), (1025, 8, 4, 4096), {}), (whole(2), (1024, 1, 4, 256), {}), (whole(1), (1025, 1, 4, 256), {}), (whole(1), (1150, 1, 8, 100), {}),
    # ... with the caller's order
    (whole(2), (128, 8, 4, 256), dict(order=True)), (pairs(4), (128, 8, 4, 257), dict(order=True)),
    (pairs(2), (130, 8, 4, 64), dict(order=True)), (whole(2), (130, 8, 4, 320), dict(order=True)), (pairs(2), (256, 8, 4, 64), dict(order=True)),
    (FIRST, (400, 8, 4, 64), dict(order=True)),
    # pairs of 64-channel heads: half the items; eight query rows never go over three sequences
    (pairs(4), (144, 8, 4, 1024), dict(d=64)), (pairs(4, 3), (288, 8, 2, 1024), dict(d=64)), (pairs(2), (288, 8, 4, 1024), dict(d=64)),
    (FIRST, (520, 8, 4, 1024), dict(d=64)),
    # one 64-channel head at a time: only the caller's order
    (whole(4), (64, 8, 8, 400), dict(d=64)), (dict(longest_first=1, waves=4), (64, 8, 8, 400), dict(d=64, order=True)),
    # ... one partition asked for: four wavefronts up to 768 heads, beyond that only where each keeps 512 tokens
    (whole(1), (32, 8, 8, 400), dict(d=64, splits=1)), (whole(4), (33, 8, 8, 400), dict(d=64, splits=1)), (whole(4), (96, 8, 8, 400), dict(d=64, splits=1)),
    (whole(1), (97, 8, 8, 400), dict(d=64, splits=1)), (whole(1), (250, 8, 8, 700), dict(d=64, splits=1)), (whole(4), (250, 8, 8, 1024), dict(d=64, splits=1)),
    (whole(1), (142, 7, 4, 200), dict(d=64, splits=1)), (whole(4), (100, 7, 4, 200), dict(d=64, splits=1)),
    # cut by the lengths: 512 slots of four wavefronts from eight a sequence on, 1024 of two otherwise
    (dict(partitions=0, slots=64, waves=4), (8, 8, 4, 8192), {}), (dict(partitions=0, slots=128, waves=2), (9, 8, 4, 8192), {}),
    (dict(partitions=0, slots=128, waves=2), (63, 8, 4, 4096), {}),
    # one sequence: partitions of 64 or 128 tokens, of half as many wavefronts with the learned rotation
    (dict(partitions=127), (1, 8, 4, 8128), {}), (dict(partitions=64), (1, 8, 4, 8128), dict(learned=True)),
    (dict(partitions=112), (1, 8, 4, 7168), dict(learned=True)), (dict(partitions=57), (1, 8, 4, 7169), dict(learned=True)),
    (dict(partitions=56), (1, 16, 4, 7168), dict(learned=True)), (dict(partitions=29), (1, 16, 4, 7169), dict(learned=True)),
    (dict(partitions=128), (1, 1, 1, 8192), {}), (dict(partitions=33), (1, 1, 1, 8193), {}), (dict(partitions=11), (1, 17, 4, 2600), {}),
    # ... but four wavefronts over whole sequences of short bounds
    (whole(4), (40, 8, 4, 1024), {}), (dict(partitions=0), (40, 8, 4, 1025), {}), (whole(4), (80, 8, 4, 768), dict(d=64)),
    (dict(partitions=0), (80, 8, 4, 769), dict(d=64)), (whole(4), (40, 8, 4, 1280), dict(learned=True)),
    (dict(partitions=0), (40, 8, 4, 1281), dict(learned=True)), (whole(4), (40, 8, 8, 768), dict(learned=True)),
    (dict(partitions=0), (40, 8, 8, 769), dict(learned=True)), (whole(4), (40, 8, 8, 1024), dict(d=64)),
    (dict(partitions=0), (40, 8, 8, 1025), dict(d=64)), (whole(4), (57, 7, 4, 1536), dict(d=64)), (dict(partitions=0), (57, 7, 4, 1537), dict(d=64)),
    (whole(4), (257, 1, 8, 1536), dict(d=64)),
    # the 16-bit call
    (pairs(2), (257, 1, 4, 257), dict(cache16=True, splits=1)), (whole(1), (257, 1, 4, 256), dict(cache16=True, splits=1)),
    (pairs(2), (257, 1, 8, 1025), dict(cache16=True, splits=1)), (whole(1), (257, 1, 8, 1024), dict(cache16=True, splits=1)),
    (whole(1), (256, 1, 4, 1025), dict(cache16=True, splits=1)), (whole(1), (1025, 1, 4, 1025), dict(cache16=True, splits=1)),
    # ... partitions of 64 or 128 tokens, at most 448 of them
    (dict(partitions=2), (4, 8, 4, 320), dict(cache16=True)), (dict(partitions=6), (4, 8, 4, 321), dict(cache16=True)),
    (dict(partitions=448), (1, 1, 4, 28672), dict(cache16=True)), (dict(partitions=225), (1, 1, 4, 28673), dict(cache16=True)),
    (dict(partitions=448), (1, 1, 4, 57344), dict(cache16=True)), (dict(partitions=225), (1, 1, 4, 57345), dict(cache16=True)),
    (dict(partitions=448), (1, 1, 8, 57344), dict(cache16=True, d=64)),
])
def test_lines_of_the_rules(saw, want, args, kw):
    got = _got(saw, *args, **kw)
    assert {k: got[k] for k in want} == want, got


def test_bad_arguments_are_refused(saw):
    for args in [(0, 8, 4, 100), (4, 8, 3, 100), (4, 8, 4, 0)]:
        with pytest.raises(saw.SawError):
            _got(saw, *args)
    with pytest.raises(saw.SawError):
        _got(saw, 4, 8, 4, 100, splits=2000)
