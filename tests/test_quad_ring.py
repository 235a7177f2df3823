"""The ping-pong mainloops (256 x 256 quadrant tiles, 256 x 128 pair tiles): ring protocol on the CPU, stage counts on the GPU.

* CPU: a model of the slot program (the half-tile requests, waits, reads and
  barriers of the leading and the trailing waves) shows, for every stage
  count, that no half tile is read before every wave's pieces of it have
  arrived and a barrier has passed, and that no ring slot is requested again
  before every wave's reads of it are complete and a barrier has passed.
* GPU: items of one, two, three and more stages (split-K ranges) of both
  operand forms, ragged rows, every mode bit-equal and within the oracle's bound.
"""
import pytest

HALVES = ("A0", "B0", "B1", "A1")


def program(nk, blocks):
    """One wave's slots: each a list of ("req", half, stage) / ("read", half, stage) / ("vm", n) / ("lgkm",);
    every slot ends in a barrier."""
    two = nk > 1
    if blocks:
        pro = [[("req", "B0", 0), ("req", "B1", 0)] + ([("req", "B0", 1), ("req", "B1", 1)] if two else [])]
        pro.append([("req", "A0", 0), ("req", "A1", 0)] + ([("req", "A0", 1)] if two else []) + [("vm", 0)])
    else:
        pro = [[("req", h, 0) for h in HALVES] + ([("req", h, 1) for h in HALVES[:3]] if two else []) + [("vm", 10 if two else 4)]]
    body = [[("read", "A0", 0), ("lgkm",)]]  # joined to the first memory slot below
    for it in range(nk):
        left = min(2, nk - 1 - it)
        m0 = ([("req", "A1", it + 1)] if left else []) + [("read", "B0", it), ("vm", 10 if left else 2)]
        m1 = ([("req", "A0", it + 2)] if left == 2 else []) + [("read", "B1", it), ("vm", (0, 8, 10)[left])]
        m2 = ([("req", "B0", it + 2)] if left == 2 else []) + [("read", "A1", it)] + ([("vm", 10 if left == 2 else 6)] if left else [])
        m3 = ([("req", "B1", it + 2)] if left == 2 else []) + ([("read", "A0", it + 1), ("vm", 10 if left == 2 else 4)] if left else [])
        for m in (m0, m1, m2, m3):
            body += [m, [("lgkm",)]]
    first = body.pop(0)
    return pro, first, body


def pair_program(nk, blocks):
    """The same of the 256 x 128 tile: two phases a stage, three stages of each half tile."""
    if blocks:
        pro = [[("req", "B0", st) for st in range(min(nk, 2))],
               [("req", h, st) for st in range(min(nk, 2)) for h in ("A0", "A1")] + ([("req", "A0", 2)] if nk > 2 else []) + [("vm", 0)]]
    else:
        pro = [[("req", h, st) for st in range(min(nk, 2)) for h in ("A0", "B0", "A1")] + ([("req", "A0", 2)] if nk > 2 else [])
               + [("vm", 10 if nk > 2 else 8 if nk == 2 else 2)]]
    body = []
    for it in range(nk):
        left = min(3, nk - 1 - it)
        m0 = ([("req", "B0", it + 2)] if left >= 2 else []) + [("read", "B0", it), ("vm", (0, 4, 8, 8)[left])]
        m1 = ([("req", "A1", it + 2)] if left >= 2 else []) + ([("req", "A0", it + 3)] if left >= 3 else []) + [("read", "A1", it)]
        m1 += [("read", "A0", it + 1), ("vm", (0, 2, 8, 10)[left])] if left else []
        body += [m0, [("lgkm",)], m1, [("lgkm",)]]
    return pro, [("read", "A0", 0), ("lgkm",)], body


def timeline(nk, blocks, trailing, pair):
    """(real slot, op) in order: the trailing waves pass one extra barrier after the first read."""
    pro, first, body = (pair_program if pair else program)(nk, blocks)
    slots = [list(s) for s in pro]
    if trailing:
        slots += [first] + body
    else:
        slots += [first + body[0]] + body[1:]
    return [(i, op) for i, s in enumerate(slots) for op in s]


def check(nk, blocks, pair):
    halves = ("A0", "B0", "A1") if pair else HALVES
    deep = 3 if pair else 2  # stages of a half tile in the ring
    reads, arrived, done, req = {}, {}, {}, {}
    for wave in (0, 1):
        pending, unread = [], []
        for slot, op in timeline(nk, blocks, wave == 1, pair):
            if op[0] == "req":
                pending += [(op[1], op[2])] * 2  # two pieces per wave and half tile
                req[wave, op[1], op[2]] = slot
            elif op[0] == "vm":
                while len(pending) > op[1]:
                    arrived[(wave, *pending.pop(0))] = slot
            elif op[0] == "read":
                reads[wave, op[1], op[2]] = slot
                unread.append((wave, op[1], op[2]))
            else:  # lgkm: the fragment reads so far are in registers
                for r in unread:
                    done[r] = slot
                unread = []
        assert not pending, (nk, blocks, pending)  # nothing lands after the loop
        assert not unread
    want = {(w, h, s) for w in (0, 1) for h in halves for s in range(nk)}
    assert set(reads) == want and set(req) == want and set(done) == want
    for (w, h, s), at in reads.items():
        for other in (0, 1):
            assert arrived[other, h, s] < at, f"{h} of stage {s} read in slot {at}, arrives in {arrived[other, h, s]}"
            if s + deep < nk:
                assert done[w, h, s] < req[other, h, s + deep], f"{h} of stage {s} overwritten while read"
    return True


@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("blocks", [False, True])
def test_the_ring_protocol_for_every_stage_count(blocks, pair):
    assert all(check(nk, blocks, pair) for nk in range(1, 14))


CASES = [
    # H, F, act, splitk1, splitk2: stages per item (GEMM1, GEMM2)
    (256, 256, 1, 4, 4),    # 1, 1
    (256, 512, 0, 2, 4),    # 2, 2
    (768, 768, 1, 4, 4),    # 3, 3
    (1024, 768, 1, 4, 3),   # 4, 4
    (512, 1280, 1, 1, 3),   # 8, and parts of 7, 7 and 6
    (256, 256, 2, 4, 2),    # gated: 1, 2
    (512, 768, 2, 1, 2),    # gated: 8, 6
]


@pytest.mark.gpu
@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("H,F,act,s1,s2", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_stage_counts_on_the_gpu(lib, H, F, act, s1, s2, pair):
    if pair and act == 2:
        pytest.skip("the pair tile has one weight operand")
    from oracle import mlp2_oracle as O
    from paper_2607_07862_amd import binding as B
    from paper_2607_07862_amd import inputs as I

    from _gpu import assert_bit_equal, assert_matches_oracle, both_modes, device_inputs, sentinel_mode, workqueue_mode

    M = 300  # two row blocks, the second ragged
    print(f"\n[quad] M={M} H={H} F={F} act={act} splits {s1} {s2}", flush=True)
    bn = 128 if pair else 256
    tuning = {"waves": 8, "bm": 256, "bn1": 128 if act == 2 else bn, "bn2": bn, "stages": 3 if pair else 2, "splitk1": s1, "splitk2": s2}
    d = I.make_inputs(M, H, F, act, seed=H + F + s1)
    g = device_inputs(d)
    plan = B.Plan(M, H, F, act, tuning)
    info = plan.info()
    assert (info["splitk1"], info["splitk2"]) == (s1, s2), info
    Ys, Zs, Yp, Zp = both_modes(plan, g)
    Yq, _ = workqueue_mode(plan, g)
    Yn = sentinel_mode(plan, g)
    assert_bit_equal(Ys, Yp, "Y sequential vs pipelined")
    assert_bit_equal(Zs, Zp, "Z sequential vs pipelined")
    assert_bit_equal(Ys, Yq, "Y sequential vs workqueue")
    assert_bit_equal(Ys, Yn, "Y sequential vs sentinel")
    ref = O.mlp2(I.bits(d["X"]), I.bits(d["W1"]), I.bits(d["W2"]), M, H, F, act)
    assert_matches_oracle(Yp, ref, "Y")
    plan.close()


@pytest.mark.gpu
def test_chain_of_pair_tiles_matches_the_oracle(lib):
    """700 rows and widths past 8192: three row blocks of 64 and 65 pair tiles, ragged rows, two to 64 stages an item."""
    import torch

    from oracle import mlp2_oracle as O
    from paper_2607_07862_amd import binding as B
    from paper_2607_07862_amd import inputs as I

    from _gpu import assert_bit_equal, assert_matches_oracle

    M, dims = 700, [128, 8192, 8320]
    d = I.chain_inputs(M, dims, seed=21)
    X, Ws = d["X"].to("cuda"), [w.to("cuda") for w in d["Ws"]]
    plan = B.ChainPlan(M, dims, 1)
    assert plan.grid() == torch.cuda.get_device_properties(0).multi_processor_count  # one work-group per CU
    out = {}
    for mode in (B.MODE_SEQUENTIAL, B.MODE_TILE_PIPELINED):
        out[mode] = torch.empty(M, dims[-1], dtype=torch.bfloat16, device="cuda")
        plan.run(X, Ws, out[mode], mode)
        torch.cuda.synchronize()
        assert plan.check() == B.OK
    assert_bit_equal(out[B.MODE_SEQUENTIAL], out[B.MODE_TILE_PIPELINED], "chain modes")
    rows = I.sample_rows(M, 48, 21)
    ref = O.chain(I.bits(d["X"]), [I.bits(w) for w in d["Ws"]], M, dims, 1, rows=rows)
    assert_matches_oracle(out[B.MODE_TILE_PIPELINED][torch.as_tensor(rows, device="cuda")], ref, "chain Y")
    plan.close()
