"""The decode products' tiles at their edges (bf16): token groups of 32, 64 and
128, more than one group, row tiles cut by the vocabulary or the intermediate
size, K of one stage and K taken in parts (rows a multiple of 8 KB apart), the
split down projection, and rows too long for the norm's registers; and the
32-row blocks that take products with few rows of W.  The bars are those of
test_gpu_decode."""

import numpy as np
import pytest

import oracle as O
from oracle import decode as D
import workloads as W
from routes import skinny_down, skinny_logits
from test_gpu_decode import check, make_case, run_decide, say

pytestmark = pytest.mark.gpu

CASES = [
    ("groups_1_stage", W.EXIT_NORM, 33, 64, 4200, 0),
    ("group_64", W.EXIT_NORM, 64, 128, 5001, 0),
    ("group_128", W.EXIT_NORM, 65, 192, 8449, 0),
    ("two_groups", W.EXIT_NORM, 129, 128, 3300, 0),
    ("many_blocks", W.EXIT_NORM, 260, 64, 128 * 130 + 1, 0),
    ("group_chunks", W.EXIT_NORM, 64 * 128 + 3, 64, 70, 0),
    ("parts_8_group_32", W.EXIT_NORM, 5, 4096, 16500, 0),
    ("parts_8_group_64", W.EXIT_NORM, 40, 4096, 6300, 0),
    ("parts_4_group_128", W.EXIT_NORM, 100, 4096, 4230, 0),
    ("embedding_parts", W.EXIT_EMBEDDING, 25, 4096, 8300, 0),
    ("mlp_ragged", W.EXIT_MLP, 2, 64, 70, 64),
    ("mlp_split_64_rows", W.EXIT_MLP, 20, 192, 300, 1600),
    ("mlp_split_group_64", W.EXIT_MLP, 50, 320, 200, 1344),
    ("mlp_split_group_128", W.EXIT_MLP, 128, 192, 200, 2240),
    ("mlp_split_two_groups", W.EXIT_MLP, 150, 128, 200, 2112),
    ("mlp_parts_gate_up", W.EXIT_MLP, 3, 4096, 200, 192),
    ("norm_in_registers_8192", W.EXIT_NORM, 2, 8192, 70, 0),
    ("norm_past_registers", W.EXIT_NORM, 2, 8256, 70, 0),
]


@pytest.mark.parametrize("name,kind,n,h,v,inter", CASES, ids=[c[0] for c in CASES])
def test_ring_decode_parity(name, kind, n, h, v, inter):
    say(f"case: decode ring {name} rows={n} h={h} V={v} I={inter}")
    if "split" in name:
        assert not skinny_down(h, n, inter)
    elif kind != W.EXIT_MLP and not name.startswith("norm_"):  # (an MLP exit's gate and up always do)
        assert not skinny_logits(v, n, h)
    w, b = make_case(kind, n, h, v, inter, "bf16", seed=31)
    conf = D.exit_decide(O.exits_from_batch(b)[0], W.decode(b.hidden[0]), 0.5)["confidence"]
    thr = float(np.median(conf)) if n > 1 else 0.5
    check(b, thr, run_decide(b, thr))


FEW_ROWS_CASES = [
    # bf16 products with few rows of W, 32 a block: 16, 8 and 4 waves that
    # share K; two row groups a block (the last one past the vocabulary); passes
    # of 32 tokens; the MLP products
    ("few_16_waves", W.EXIT_NORM, 7, 192, 333, 0),
    ("few_8_waves", W.EXIT_NORM, 16, 64, 8193, 0),
    ("few_4_waves", W.EXIT_NORM, 3, 64, 16401, 0),
    ("few_two_groups", W.EXIT_NORM, 20, 4096, 12300, 0),
    ("few_passes", W.EXIT_EMBEDDING, 300, 128, 1000, 0),
    ("few_mlp_down", W.EXIT_MLP, 70, 64, 100, 64),
    ("few_mlp_down_8", W.EXIT_MLP, 8, 192, 100, 448),
]


@pytest.mark.parametrize("name,kind,n,h,v,inter", FEW_ROWS_CASES, ids=[c[0] for c in FEW_ROWS_CASES])
def test_few_rows_decode_parity(name, kind, n, h, v, inter):
    say(f"case: decode {name} rows={n} h={h} V={v} I={inter}")
    if kind == W.EXIT_MLP:
        assert skinny_down(h, n, inter)
    else:
        assert skinny_logits(v, n, h)
    w, b = make_case(kind, n, h, v, inter, "bf16", seed=33)
    conf = D.exit_decide(O.exits_from_batch(b)[0], W.decode(b.hidden[0]), 0.5)["confidence"]
    thr = float(np.median(conf))
    check(b, thr, run_decide(b, thr))


# Equal rows in tiles that take K in each of the orders (128-row tile t takes order
# t / 8 mod 8, or mod 4 past 64 tokens).
TIED = [140 + 1030 * i for i in range(8)]
TIE_CASES = [(3, 4096, 16500), (3, 8192, 16500), (40, 4096, 8300), (40, 8192, 8300), (90, 4096, 8300), (40, 1088, 8300)]


@pytest.mark.parametrize("rows,h,v", TIE_CASES)
def test_equal_rows_of_different_tiles_tie(rows, h, v):
    """Equal rows of W_out give the same fp32 logit wherever they lie, also
    where the row tiles take K in different orders: the lowest id wins."""
    assert not skinny_logits(v, rows, h)
    assert sorted(i // 128 // 8 % 8 for i in TIED) == list(range(8))
    w, b = make_case(W.EXIT_NORM, rows, h, v, 0, "bf16", seed=32)
    z = O.exit_forward(O.exits_from_batch(b)[0], W.decode(b.hidden[0]))["z"]
    mean = z.mean(axis=0)
    row = W.f32_to_bf16_bits((3.0 * mean / np.abs(mean).max()).astype(np.float32))
    for i in TIED:
        b.exits[0].w_out[i] = row
    say(f"case: decode ties rows={rows} h={h}")
    token, _, _ = run_decide(b, 0.9)
    s = D.exit_decide(O.exits_from_batch(b)[0], W.decode(b.hidden[0]), 0.9)["logits"]
    tied = s[:, 140] == s.max(axis=1)
    assert tied.any()
    assert (token[tied] == 140).all()


@pytest.mark.parametrize("rows,h,v", [(32, 3072, 17000), (64, 3072, 9000), (100, 3072, 9000), (300, 3072, 17000)])
def test_embedding_sums_are_short(rows, h, v):
    """An Embedding exit's logits are products of its inputs as they are, so the
    order of the fp32 sums is all of the confidences' error: K is taken in at most 8
    parts of 512 values or more.  One chain over h 3072 gives 1.8e-6 to 3.3e-6 here,
    parts 2.4e-7 to 4.5e-7 (relative, 2-norm): the bar is twice that."""
    assert not skinny_logits(v, rows, h)
    w, b = make_case(W.EXIT_EMBEDDING, rows, h, v, 0, "bf16", seed=34)
    say(f"case: decode embedding sums rows={rows} h={h} V={v}")
    _, conf, _ = run_decide(b, 0.5)
    ref = D.exit_decide(O.exits_from_batch(b)[0], W.decode(b.hidden[0]), 0.5)["confidence"]
    err = np.linalg.norm(conf - ref) / np.linalg.norm(ref)
    say(f"  relative error {err:.2e}")
    assert err <= 9e-7
