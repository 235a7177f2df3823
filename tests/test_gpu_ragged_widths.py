"""Widths that the chosen tiles do not divide, and the plan's tile choice around its limits.

Without a tile tuning the last column block of a GEMM may be narrower than
its tile: the loads of columns past the end are clamped and their stores
skipped.  Every tile family that a plan chooses meets such widths here (with
one 64-column remainder, and narrower than one tile; tiles of 64 columns and
widths they divide beside them), in every mode against the sequential mode's
bits and the fp64 oracle; Y stands between guard rows that must stay as they
were.  Each case names the tile it is about, so a change of the choice cannot
take it away unseen.
"""
import pytest
import torch

from oracle import mlp2_oracle as O
from paper_2607_07862_amd import binding as B
from paper_2607_07862_amd import inputs as I

from _gpu import assert_bit_equal, assert_matches_oracle, device_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # M, H, F, act, the tile it is about: rows, columns of GEMM1 and GEMM2, ring, waves
    (5, 1088, 4416, 1, (32, 64, 64, 4, 4)),
    (50, 192, 1472, 2, (32, 64, 64, 4, 4)),
    (20, 704, 16448, 1, (32, 128, 64, 4, 4)),
    (60, 8256, 3520, 0, (64, 128, 128, 4, 4)),
    (100, 8256, 3520, 1, (128, 128, 128, 4, 8)),
    (120, 1088, 2112, 2, (64, 64, 128, 4, 4)),
    (250, 1088, 1472, 1, (128, 128, 128, 4, 8)),
    (250, 1600, 1472, 2, (128, 64, 128, 4, 4)),
    (300, 320, 192, 1, (128, 64, 64, 4, 4)),
    (300, 320, 192, 2, (128, 64, 128, 2, 4)),
    (2100, 2112, 1344, 0, (128, 128, 128, 4, 8)),
    (1030, 1344, 5440, 2, (128, 64, 128, 2, 4)),
    (600, 8256, 8256, 1, (128, 128, 128, 2, 4)),
    # quadrant tiles; the last gated GEMM2 block's second half lies past H, wholly or exactly
    (2048, 2112, 5440, 0, (256, 256, 256, 2, 8)),
    (2048, 2112, 5440, 2, (256, 128, 256, 2, 8)),
    (2048, 2176, 5440, 2, (256, 128, 256, 2, 8)),
    (1030, 8256, 3520, 0, (256, 256, 256, 2, 8)),
    # pair tiles
    (1024, 8256, 8256, 1, (256, 128, 128, 3, 8)),
]


@pytest.mark.parametrize("M,H,F,act,tile", CASES, ids=["x".join(map(str, c[:4])) for c in CASES])
def test_ragged_widths_in_every_mode(lib, M, H, F, act, tile):
    d = I.make_inputs(M, H, F, act, seed=M + H + F + act)
    g = device_inputs(d)
    plan = B.Plan(M, H, F, act)
    info = plan.info()
    print(f"\n[ragged] {M}x{H}x{F} act={act} {info['bm']}x{info['bn1']} {info['bn2']} splits {info['splitk1']} {info['splitk2']}", flush=True)
    if info["num_cus"] == 256:  # the choices are drawn for 256 CUs
        assert tuple(info[k] for k in ("bm", "bn1", "bn2", "stages", "waves")) == tile, info
    outs = {}
    for mode in ("sequential", "tile_pipelined", "workqueue", "sentinel"):
        box = torch.full((M + 2, H), 7.0, dtype=torch.bfloat16, device="cuda")
        plan.run(g["X"], g["W1"], g["W2"], box[1:-1], mode)
        torch.cuda.synchronize()
        assert plan.check() == B.OK
        assert bool((box[0] == 7).all()) and bool((box[-1] == 7).all()), f"{mode} wrote outside Y"
        outs[mode] = box[1:-1].clone()
    for mode, Y in outs.items():
        assert_bit_equal(outs["sequential"], Y, f"sequential vs {mode}")
    rows = None if M < 500 else I.sample_rows(M, 48, 3)
    ref = O.mlp2(I.bits(d["X"]), I.bits(d["W1"]), I.bits(d["W2"]), M, H, F, act, rows=rows)
    Y = outs["sequential"] if rows is None else outs["sequential"][torch.as_tensor(rows, device="cuda")]
    assert_matches_oracle(Y, ref, "Y")
    plan.close()


def test_a_named_width_must_still_divide(lib):
    for tuning in ({"bm": 128, "bn1": 128, "bn2": 128, "stages": 2}, {"bm": 256, "bn1": 256, "bn2": 256, "stages": 2, "waves": 8}):
        with pytest.raises(B.Mlp2Error) as e:
            B.Plan(777, 2112, 5440, 1, tuning)
        assert e.value.code == B.ERR_UNSUPPORTED


def test_noalloc_takes_less_workspace_where_the_chosen_plan_is_too_large(lib):
    M, H, F, act = 512, 4096, 14336, 2  # quadrant tiles: 64 MiB of GEMM2 partials alone
    plan = B.Plan(M, H, F, act)
    info = plan.info()
    own = 2 * info["row_blocks"] * info["bm"] * F * 2  # the sentinel mode's two buffers, which the allocation-free entry has not
    assert info["workspace_bytes"] - own > (64 << 20), info
    plan.close()
    d = I.make_inputs(M, H, F, act, seed=5)
    g = device_inputs(d)
    Y = torch.empty(M, H, dtype=torch.bfloat16, device="cuda")
    B.run_noalloc(g["X"], g["W1"], g["W2"], Y, act, B.MODE_TILE_PIPELINED)
    torch.cuda.synchronize()
    rows = I.sample_rows(M, 24, 5)
    ref = O.mlp2(I.bits(d["X"]), I.bits(d["W1"]), I.bits(d["W2"]), M, H, F, act, rows=rows)
    assert_matches_oracle(Y[torch.as_tensor(rows, device="cuda")], ref, "Y")
