"""Which tiles the plans take, at both sides of the rules' lines."""
import pytest
import torch

from oracle import mlp2_oracle as O
from paper_2607_07862_amd import binding as B
from paper_2607_07862_amd import inputs as I

from _gpu import assert_matches_oracle

pytestmark = pytest.mark.gpu


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
