"""The quadrant tile's ping-pong mainloop: its ring protocol on the CPU, its stage counts on the GPU.

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


def timeline(nk, blocks, trailing):
    """(real slot, op) in order: the trailing waves pass one extra barrier after the first read."""
    pro, first, body = program(nk, blocks)
    slots = [list(s) for s in pro]
    if trailing:
        slots += [first] + body
    else:
        slots += [first + body[0]] + body[1:]
    return [(i, op) for i, s in enumerate(slots) for op in s]


def check(nk, blocks):
    reads, arrived, done, req = {}, {}, {}, {}
    for wave in (0, 1):
        pending, unread = [], []
        for slot, op in timeline(nk, blocks, wave == 1):
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
    want = {(w, h, s) for w in (0, 1) for h in HALVES for s in range(nk)}
    assert set(reads) == want and set(req) == want and set(done) == want
    for (w, h, s), at in reads.items():
        for other in (0, 1):
            assert arrived[other, h, s] < at, f"{h} of stage {s} read in slot {at}, arrives in {arrived[other, h, s]}"
            if s + 2 < nk:
                assert done[w, h, s] < req[other, h, s + 2], f"{h} of stage {s} overwritten while read"
    return True


@pytest.mark.parametrize("blocks", [False, True])
def test_the_ring_protocol_for_every_stage_count(blocks):
    assert all(check(nk, blocks) for nk in range(1, 12))


CASES = [
    # H, F, act, splitk1, splitk2: stages per item (GEMM1, GEMM2)
    (256, 256, 1, 4, 4),    # 1, 1
    (256, 512, 0, 2, 4),    # 2, 2
    (768, 768, 1, 4, 4),    # 3, 3
    (512, 1280, 1, 1, 3),   # 8, and parts of 7, 7 and 6
    (256, 256, 2, 4, 2),    # gated: 1, 2
    (512, 768, 2, 1, 2),    # gated: 8, 6
]


@pytest.mark.gpu
@pytest.mark.parametrize("H,F,act,s1,s2", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_stage_counts_on_the_gpu(lib, H, F, act, s1, s2):
    from oracle import mlp2_oracle as O
    from paper_2607_07862_amd import binding as B
    from paper_2607_07862_amd import inputs as I

    from _gpu import assert_bit_equal, assert_matches_oracle, both_modes, device_inputs, sentinel_mode, workqueue_mode

    M = 300  # two row blocks, the second ragged
    print(f"\n[quad] M={M} H={H} F={F} act={act} splits {s1} {s2}", flush=True)
    tuning = {"waves": 8, "bm": 256, "bn1": 128 if act == 2 else 256, "bn2": 256, "stages": 2, "splitk1": s1, "splitk2": s2}
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
