"""The products' tiles at their edges, every tile of each data type: one, two and
three stages of K, K that ends inside a stage (operands read MN-major), operands
of a fraction of a tile, and a workspace that holds NaN before the step (nothing
the products multiply may be left over from it).  The bars are those of
test_gpu_parity."""

import pytest
import torch

import workloads as W
from routes import f32_loops, f32_parts, f32_small, mid_tile, split_tail
from test_gpu_parity import compare_full, gpu, say, small  # noqa: F401 (gpu: the module's GPU fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # bf16, 128 x 128 tiles.  name, kind, N, h, V, I: stages of the logits
    # product h / 64, of dW_out ceil(N / 64), of dZ ceil(V / 64), of dW_down ceil(N / 64)
    ("pipe_one_stage", W.EXIT_NORM, 5, 64, 65, 0),
    ("pipe_two_stages", W.EXIT_NORM, 65, 128, 257, 0),
    ("pipe_three_stages", W.EXIT_NORM, 129, 192, 1000, 0),
    ("pipe_mlp_one_stage", W.EXIT_MLP, 9, 64, 64, 64),
    ("pipe_mlp_tail_1", W.EXIT_MLP, 65, 64, 129, 64),
    ("pipe_mlp_tail_63", W.EXIT_MLP, 191, 192, 319, 128),
    ("pipe_mlp_tails_wide", W.EXIT_MLP, 300, 576, 1000, 320),
]


@pytest.mark.parametrize("name,kind,n,h,v,inter", CASES, ids=[c[0] for c in CASES])
def test_pipeline_edges(name, kind, n, h, v, inter):
    from paper_2402_00518_amd.session import Session
    say(f"case: {name} N={n} h={h} V={v} I={inter}")
    assert all(mid_tile(t) for t in big_tiles(n, h, v, inter).values())
    b = small(kind, n, h, v, inter, seed=9, name=name)
    s = Session.from_batch(b)
    s.ws.fill_(0xFF)
    s.step()
    torch.cuda.synchronize()
    s.check_device_error()
    compare_full(s, b, case=name)


def big_tiles(n, h, v, inter):
    """256 x 256 tiles of each launch of a step (splits not counted)."""
    def t(a, b):
        return -(-a // 256) * -(-b // 256)
    tiles = {"logits": t(n, v), "dW_out": t(h, v)}
    if inter:
        tiles.update(gate_up=t(n, 2 * inter), down=t(n, h), dZ=t(-(-n // 64) * 64, h), dA_dW_down=t(n, inter) + t(h, inter),
                     dW_gate_up=2 * t(h, inter))
    return tiles


BIG_TILE_CASES = [
    # bf16, 256 x 256 tiles, and the products that take them: one, two and three
    # stages of K
    ("big_one_stage", W.EXIT_NORM, 5, 64, 130 * 256 + 1, 0, ("logits", "dW_out")),
    ("big_two_stages", W.EXIT_NORM, 65, 128, 130 * 256 + 1, 0, ("logits", "dW_out")),
    ("big_three_stages", W.EXIT_NORM, 129, 192, 130 * 256 + 255, 0, ("logits", "dW_out")),
    ("big_gate_up", W.EXIT_MLP, 300, 64, 100, 8320, ("gate_up",)),
    # dZ, both operands MN-major: one stage that ends inside K, two and three;
    # the down projection of one stage
    ("big_dz_tail_33", W.EXIT_MLP, 1030, 8192, 33, 64, ("down", "dZ")),
    ("big_dz_tail_65", W.EXIT_MLP, 1030, 8192, 65, 64, ("down", "dZ")),
    ("big_dz_tail_129", W.EXIT_MLP, 1030, 8192, 129, 64, ("down", "dZ")),
    # its tokens past 2048 as four slices, the last one with a ragged end
    ("big_dz_split", W.EXIT_MLP, 2310, 8192, 1999, 64, ("down", "dZ")),
    # dW_down over a single stage that ends inside K, beside dA; the gate and up pair
    ("big_down_one_stage", W.EXIT_MLP, 40, 8192, 65, 1088, ("dA_dW_down", "dW_gate_up")),
    ("big_down_two_stages", W.EXIT_MLP, 70, 8192, 65, 1088, ("dA_dW_down", "dW_gate_up")),
]


@pytest.mark.parametrize("name,kind,n,h,v,inter,big", BIG_TILE_CASES, ids=[c[0] for c in BIG_TILE_CASES])
def test_big_tile_edges(name, kind, n, h, v, inter, big):
    from paper_2402_00518_amd.session import Session
    say(f"case: {name} N={n} h={h} V={v} I={inter}")
    tiles = big_tiles(n, h, v, inter)
    assert not any(mid_tile(tiles[p]) for p in big)
    if "dZ" in big:
        assert (split_tail(False, n, h, v)[2] > 1) == ("split" in name)
    b = small(kind, n, h, v, inter, seed=11, name=name)
    s = Session.from_batch(b)
    s.ws.fill_(0xFF)
    s.step()
    torch.cuda.synchronize()
    s.check_device_error()
    compare_full(s, b, case=name)


SMALL_TILE_CASES = [
    # bf16 on 128 x 128 tiles: one stage and ragged tails; both operands
    # MN-major with a K tail (dZ, dW_down); the split tail of dZ
    ("mid_one_stage", W.EXIT_NORM, 130, 64, 300, 0, "bf16"),
    ("mid_mlp_tails", W.EXIT_MLP, 333, 320, 1111, 448, "bf16"),
    ("mid_split", W.EXIT_MLP, 700, 256, 2100, 1216, "bf16"),
    # fp32: 64 x 64 tiles with waves that share K (K of one stage, K tails, the
    # split products); 128 x 128 tiles K-major, with an interleaved pair, and
    # MN-major with a K tail
    ("f32_small", W.EXIT_NORM, 65, 64, 129, 0, "f32"),
    ("f32_small_mlp", W.EXIT_MLP, 100, 192, 203, 320, "f32"),
    ("f32_split", W.EXIT_MLP, 150, 128, 1100, 576, "f32"),
    # the slices of dZ limited by the room behind it
    ("f32_split_narrow", W.EXIT_MLP, 150, 512, 1100, 64, "f32"),
    ("f32_big_logits", W.EXIT_NORM, 100, 64, 32700, 0, "f32"),
    ("f32_big_gate_up", W.EXIT_MLP, 500, 64, 100, 4096, "f32"),
    ("f32_big_dz", W.EXIT_MLP, 4000, 1024, 100, 64, "f32"),
    # 128 x 128 tiles in a loop, all with ragged last tiles: logits and dW_out; with
    # K in four parts gate and up, and dZ (K tail)
    ("f32_loop_logits_dw", W.EXIT_NORM, 100, 128, 74001, 0, "f32"),
    ("f32_loop_parts_gate_up", W.EXIT_MLP, 100, 64, 100, 33088, "f32"),
    ("f32_loop_parts_dz", W.EXIT_MLP, 4100, 2048, 100, 64, "f32"),
    # K in four parts without the loop: fewer stages than parts, a ragged last part
    ("f32_parts_logits", W.EXIT_NORM, 1036, 64, 2862, 0, "f32"),
    ("f32_parts_dw", W.EXIT_NORM, 300, 384, 7440, 0, "f32"),
]


def f32_tiles(a, b):
    return [-(-a // t) * -(-b // t) for t in (128, 64)]


@pytest.mark.parametrize("name,kind,n,h,v,inter,dtype", SMALL_TILE_CASES, ids=[c[0] for c in SMALL_TILE_CASES])
def test_tile_choice_edges(name, kind, n, h, v, inter, dtype):
    from paper_2402_00518_amd.session import Session
    say(f"case: {name} N={n} h={h} V={v} I={inter} {dtype}")
    products = {"logits": (n, v, h), "dw": (h, v, -(-n // 64) * 64), "gate_up": (n, 2 * inter, h), "dz": (-(-n // 64) * 64, h, v)}
    for p, (rows, cols, k) in products.items():
        if name.startswith(("f32_big", "f32_loop", "f32_parts")) and p in name:
            tiles = f32_tiles(rows, cols)
            assert not f32_small(*tiles, k) and f32_loops(tiles[0]) == ("loop" in name)
            assert f32_parts(*tiles) == (4 if "parts" in name else 1)
    b = small(kind, n, h, v, inter, dtype, seed=10, name=name)
    s = Session.from_batch(b)
    s.ws.fill_(0xFF)
    s.step()
    torch.cuda.synchronize()
    s.check_device_error()
    if dtype == "f32":
        compare_full(s, b, loss_rtol=1e-5, grad_rtol=1e-4, case=name)
    else:
        compare_full(s, b, case=name)


@pytest.mark.parametrize("kind,n,inter", [(W.EXIT_NORM, 70, 0), (W.EXIT_NORM, 513, 0), (W.EXIT_MLP, 150, 192)],
                         ids=["norm_70", "norm_513", "mlp_150"])
def test_f32_padding_is_written(kind, n, inter):
    """fp32: the token columns between N and its padding take part in the
    weight-gradient product (times zeros), so the logits product writes them:
    NaN left in the workspace must not reach a gradient."""
    from paper_2402_00518_amd.session import Session
    say(f"case: f32 padding N={n} I={inter}")
    b = small(kind, n, 128, 300, inter, "f32", seed=6, name="f32_padding")
    s = Session.from_batch(b)
    s.ws.fill_(0xFF)
    s.step()
    torch.cuda.synchronize()
    compare_full(s, b, loss_rtol=1e-5, grad_rtol=1e-4, case="f32_padding")
