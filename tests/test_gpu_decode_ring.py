"""The decode products' tiles at their edges (bf16): token groups of 32, 64 and
128, more than one group, row tiles cut by the vocabulary or the intermediate
size, K of one stage and K taken in parts (rows a multiple of 8 KB apart), the
split down projection, and rows too long for the norm's registers.  The bars
are those of test_gpu_decode."""

import numpy as np
import pytest

import oracle as O
from oracle import decode as D
import workloads as W
from test_gpu_decode import check, make_case, run_decide, say

pytestmark = pytest.mark.gpu

CASES = [
    ("groups_1_stage", W.EXIT_NORM, 33, 64, 129, 0),
    ("group_64", W.EXIT_NORM, 64, 128, 1000, 0),
    ("group_128", W.EXIT_NORM, 65, 192, 300, 0),
    ("two_groups", W.EXIT_NORM, 129, 128, 257, 0),
    ("many_blocks", W.EXIT_NORM, 260, 64, 128 * 130 + 1, 0),
    ("group_chunks", W.EXIT_NORM, 64 * 128 + 3, 64, 70, 0),
    ("parts_8_group_32", W.EXIT_NORM, 5, 4096, 500, 0),
    ("parts_8_group_64", W.EXIT_NORM, 40, 4096, 1300, 0),
    ("parts_4_group_128", W.EXIT_NORM, 100, 4096, 300, 0),
    ("embedding_parts", W.EXIT_EMBEDDING, 17, 4096, 1100, 0),
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
    w, b = make_case(kind, n, h, v, inter, "bf16", seed=31)
    conf = D.exit_decide(O.exits_from_batch(b)[0], W.decode(b.hidden[0]), 0.5)["confidence"]
    thr = float(np.median(conf)) if n > 1 else 0.5
    check(b, thr, run_decide(b, thr))


@pytest.mark.parametrize("rows,h", [(3, 4096), (40, 4096), (90, 4096), (40, 1088)])
def test_equal_rows_of_different_tiles_tie(rows, h):
    """Equal rows of W_out give the same fp32 logit wherever they lie, also
    where the row tiles take K in different orders: the lowest id wins."""
    w, b = make_case(W.EXIT_NORM, rows, h, 5000, 0, "bf16", seed=32)
    z = O.exit_forward(O.exits_from_batch(b)[0], W.decode(b.hidden[0]))["z"]
    mean = z.mean(axis=0)
    row = W.f32_to_bf16_bits((3.0 * mean / np.abs(mean).max()).astype(np.float32))
    for i in (140, 1200, 2300, 3400, 4999):
        b.exits[0].w_out[i] = row
    say(f"case: decode ties rows={rows} h={h}")
    token, _, _ = run_decide(b, 0.9)
    s = D.exit_decide(O.exits_from_batch(b)[0], W.decode(b.hidden[0]), 0.9)["logits"]
    tied = s[:, 140] == s.max(axis=1)
    assert tied.any()
    assert (token[tied] == 140).all()
