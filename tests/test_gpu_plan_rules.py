"""Which tiles the plans take, at both sides of the rules' lines."""
import pytest
import torch

from oracle import mlp2_oracle as O
from paper_2607_07862_amd import binding as B
from paper_2607_07862_amd import inputs as I

from _gpu import assert_matches_oracle

pytestmark = pytest.mark.gpu


# (M, H, F, activation, tile rows, columns of GEMM1 and GEMM2, ring, waves)
PLANS = [
    # 129 to 256 rows, gated: 128-row tiles from the smallest product on
    (200, 64, 1472, 2, (128, 64, 128, 4, 4)),
    (129, 1024, 1024, 2, (128, 64, 128, 4, 4)),
    (256, 4096, 14336, 2, (256, 128, 256, 2, 8)),
    # up to 32 rows: 64-column GEMM1 tiles up to one per CU
    (32, 8192, 16384, 1, (32, 64, 128, 4, 4)),
    (32, 8192, 16448, 1, (32, 128, 128, 4, 4)),
    # beyond 256 rows: 128 x 64 tiles up to one per CU and GEMM, for an odd multiple of 64 or SwiGLU
    (300, 128, 192, 1, (128, 64, 64, 4, 4)),
    (1000, 2048, 704, 2, (128, 64, 64, 4, 4)),
    (300, 256, 512, 2, (128, 64, 64, 4, 4)),
    (600, 320, 64, 2, (128, 64, 128, 2, 4)),
    (1024, 1984, 1984, 1, (128, 64, 64, 4, 4)),
    (1024, 2048, 2112, 1, (128, 128, 128, 4, 8)),
    (512, 256, 512, 1, (128, 128, 128, 2, 4)),
]


@pytest.mark.parametrize("M,H,F,act,want", PLANS, ids=["x".join(map(str, c[:4])) for c in PLANS])
def test_plan_tiles(lib, M, H, F, act, want):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines are drawn for 256 CUs")
    plan = B.Plan(M, H, F, act)
    info = plan.info()
    assert tuple(info[k] for k in ("bm", "bn1", "bn2", "stages", "waves")) == want, info
    plan.close()


@pytest.mark.parametrize("M,H,F,built", [(129, 256, 256, True), (198, 6400, 2048, True), (256, 4096, 14336, True),
                                         (100, 4096, 14336, False), (300, 1024, 3584, False), (200, 6400, 2112, False)])
def test_the_forced_weight_hint_takes_the_tiles_built_with_it(lib, M, H, F, built):
    """Gated plans of 129 to 256 rows whose widths the hinted tile divides, at any size; refused elsewhere."""
    if not built:
        with pytest.raises(B.Mlp2Error) as e:
            B.Plan(M, H, F, 2, {"weights_nt": 1})
        assert e.value.code == B.ERR_UNSUPPORTED
        return
    plan = B.Plan(M, H, F, 2, {"weights_nt": 1})
    info = plan.info()
    assert (info["bm"], info["bn1"], info["bn2"], info["weights_nt"]) == (256, 128, 256, 1), info
    plan.close()


@pytest.mark.parametrize("M,parts", [(64, 2), (65, 3), (128, 3)])
def test_plan_splits_a_lone_tile(lib, M, parts):
    """One GEMM2 column block over 1472 rows of W2: ranges of at least 512, of 448 beyond 64 rows."""
    plan = B.Plan(M, 64, 1472, 1)
    assert plan.info()["splitk2"] == parts, plan.info()
    plan.close()


# (M, equal widths, work-groups per CU of the chain's tile: 64 x 64 and 128 x 128 tiles two, 256 x 128 one)
CHAINS = [
    (64, 24576, 2),   # 64 x 64: few rows
    (65, 24576, 1),   # 192 tiles of 256 x 128, three quarters of the CUs
    (64, 32768, 1),   # few rows, but 64 x 64 tiles are no alternative
    (128, 40960, 2),  # 320 tiles of 256 x 128 would be a second round, 320 of 128 x 128 fit one
    (256, 40960, 1),  # 640 of 128 x 128: two rounds either way
]


@pytest.mark.parametrize("M,D,per_cu", CHAINS, ids=[f"{c[0]}x{c[1]}" for c in CHAINS])
def test_chain_tile(lib, M, D, per_cu):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the lines are drawn for 256 CUs")
    print(f"\n[chain tile] {M} x {D}", flush=True)
    plan = B.ChainPlan(M, [D, D, D], 1)
    tiles128 = 2 * -(-M // 128) * (D // 128)
    assert plan.grid() == (cus if per_cu == 1 else min(2 * cus, tiles128 * (4 if tiles128 < 2 * cus else 1)))
    plan.close()


def test_chain_whose_256_row_padding_would_pass_4_gb(lib):
    """126080 rows are 985 blocks of 128, an odd number: with 256-row tiles the intermediate's padded rows reach 4 GB."""
    M, dims = 126080, [128, 17024, 128]
    assert M * dims[1] * 2 < 1 << 32 <= -(-M // 256) * 256 * dims[1] * 2
    print(f"\n[chain padding] {M} {dims}", flush=True)
    plan = B.ChainPlan(M, dims, 1)
    d = I.chain_inputs(M, dims, seed=5)
    X, Ws = d["X"].to("cuda"), [w.to("cuda") for w in d["Ws"]]
    Y = torch.empty(M, dims[-1], dtype=torch.bfloat16, device="cuda")
    plan.run(X, Ws, Y, B.MODE_TILE_PIPELINED)
    torch.cuda.synchronize()
    assert plan.check() == B.OK
    rows = sorted({0, 1, M - 1, M - 129, *I.sample_rows(M, 24, 5)})
    ref = O.chain(I.bits(d["X"]), [I.bits(w) for w in d["Ws"]], M, dims, 1, rows=rows)
    assert_matches_oracle(Y[torch.as_tensor(rows, device="cuda")], ref, "chain Y")
    plan.close()
