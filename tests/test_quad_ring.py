"""The ping-pong mainloops (256 x 256 quadrant tiles, 256 x 128 pair tiles): ring protocol on the CPU, stage counts on the GPU.

* CPU: the loops' slot program (the half-tile requests, waits, reads and
  barriers of the leading and the trailing waves) is read from the kernel
  source and shows, for every stage count, that no half tile is read before every wave's pieces of it have
  arrived and a barrier has passed, and that no ring slot is requested again
  before every wave's reads of it are complete and a barrier has passed.
* GPU: items of one, two, three and more stages (split-K ranges) of both
  operand forms, ragged rows, every mode bit-equal and within the oracle's bound.
"""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2607_07862_amd", "csrc", "mlp2_device.hpp")


# ------------------------------------------------------------------ the loops, read from the kernel source

def closing(text, i):
    """Index of the bracket that closes the one at text[i]."""
    pairs = {"{": "}", "(": ")"}
    depth = 0
    for j in range(i, len(text)):
        depth += (text[j] == text[i]) - (text[j] == pairs[text[i]])
        if depth == 0:
            return j
    raise ValueError("unbalanced")


def loop_source(name):
    """(stage lambda's body, what follows it up to the function's end), without comments."""
    text = re.sub(r"//[^\n]*", "", open(SRC).read())
    start = text.index("{", text.index(f"void {name}("))
    body = text[start + 1:closing(text, start)]
    at = body.index("auto stage = [&]")
    o = body.index("{", at)
    c = closing(body, o)
    return body[o + 1:c], body[c + 2:]


def parse(text):
    """Statements as ("if", condition, then, else), ("for", condition, body) and ("do", text)."""
    out, i = [], 0

    def unit(i):  # one statement or block from i: (statements, next index)
        while text[i].isspace():
            i += 1
        if text[i] == "{":
            c = closing(text, i)
            return parse(text[i + 1:c]), c + 1
        m = re.match(r"(if\s*(?:constexpr)?|for)\s*\(", text[i:])
        if m:
            o = i + m.end() - 1
            c = closing(text, o)
            head = text[o + 1:c]
            then, j = unit(c + 1)
            if m.group(1) == "for":
                return [("for", head, then)], j
            e = re.match(r"\s*else\b", text[j:])
            if not e:
                return [("if", head, then, [])], j
            other, j = unit(j + e.end())
            return [("if", head, then, other)], j
        j = text.index(";", i)
        return [("do", " ".join(text[i:j].split()))], j + 1

    while text[i:].strip():
        part, i = unit(i)
        out += part
    return out


def value(expr, env):
    """A C expression of integers and conditions."""
    expr = expr.replace("Wait::kBlocks", "blocks")
    m = re.match(r"([^?]*)\?([^:]*):(.*)$", expr)
    if m:
        return value(m.group(2), env) if value(m.group(1), env) else value(m.group(3), env)
    expr = re.sub(r"!(?!=)", " not ", expr.replace("&&", " and ").replace("||", " or "))
    return int(eval(expr.strip(), {}, dict(env)))


def program(source, nk, blocks, trailing, pair):
    """One wave's operations in order: ("req", half, stage, ring slot), ("read", half, ring slot), ("vm", n), ("lgkm",), ("bar",)."""
    stage_body, rest = (parse(t) for t in source)
    ops = []
    env = {"nk": nk, "blocks": int(blocks), "trailing": int(trailing), "wave": 4 if trailing else 0, "r": 0}

    def call(name, args):
        v = [value(a, env) if re.fullmatch(r"[\w\s+\-]+", a) and not re.match(r"[xw][ab01]?$", a.strip()) else None for a in args]
        if name == "load_a":
            ops.append(("req", f"A{v[0]}", v[1], v[2] if pair else v[1] & 1))
        elif name == "load_b":
            ops.append(("req", "B0", v[0], v[1]) if pair else ("req", f"B{v[0]}", v[1], v[1] & 1))
        elif name == "read_a":
            ops.append(("read", f"A{v[1]}", v[2] if pair else v[2] & 1))
        elif name == "read_b":
            ops.append(("read", "B0", v[0]) if pair else ("read", f"B{v[1]}", v[2] & 1))
        elif name == "slot_end":
            ops.append(("bar",))
        elif name == "products_begin":
            ops.append(("lgkm",))
        elif name == "products_end":
            ops.append(("bar",))
        elif name == "products":
            ops.extend([("lgkm",), ("bar",)])
        elif name not in ("mma", "__syncthreads"):
            raise ValueError(f"unknown call {name}")

    def do(t):
        m = re.match(r"stage\((.*), int_constant<(\d)>\(\)\)$", t)
        if m:
            env["it"], env["LEFT"] = value(m.group(1), env), int(m.group(2))
            run(stage_body)
            return
        m = re.match(r"vm_traced\(int_constant<(.*)>\(\)\)$", t) or re.match(r"wait_vm<(\d+)>\(\)$", t)
        if m:
            # the ternary's conditions hold ">=": the constant is what stands between the outer angle brackets
            ops.append(("vm", value(m.group(1), env)))
            return
        if t.startswith("wait.") or t.startswith("constexpr int LEFT") or t.startswith("const int k ="):
            return
        if t == "__builtin_amdgcn_s_waitcnt(0xC07F)":
            ops.append(("lgkm",))
            return
        m = re.match(r"(?:const (?:int|bool) |int )?(\w+ = .*)$", t)
        if m:
            for a in m.group(1).split(","):
                k, e = a.split("=", 1)
                env[k.strip()] = value(e, env)
            return
        m = re.match(r"(\w+)\((.*)\)$", t)
        call(m.group(1), m.group(2).split(","))

    def run(nodes):
        for n in nodes:
            if n[0] == "do":
                do(n[1])
            elif n[0] == "if":
                run(n[2] if value(n[1], env) else n[3])
            else:
                init, cond, step = n[1].split(";")
                assert step.strip() == "++it" and init.strip() == "int it = 0", n[1]
                i = 0
                while value(cond, {**env, "it": i}):
                    assert len(n[2]) == 1
                    do(n[2][0][1].replace("(it,", f"({i},"))
                    i += 1

    run(rest)
    return ops


def check(source, nk, blocks, pair):
    """Every half tile is read once, after every wave's pieces of it have arrived and a barrier, and its ring slot
    requested again only after every wave's reads are complete and a barrier."""
    halves = ("A0", "B0", "A1") if pair else ("A0", "B0", "B1", "A1")
    deep = 3 if pair else 2  # stages of a half tile in the ring
    reads, arrived, done, req = {}, {}, {}, {}
    bars = []
    for wave in (0, 1):
        slot, pending, unread, holds = 0, [], [], {}
        for op in program(source, nk, blocks, wave == 1, pair):
            if op[0] == "bar":
                slot += 1
            elif op[0] == "req":
                assert op[3] == op[2] % deep, op
                pending += [(op[1], op[2])] * 2  # two pieces per wave and half tile
                req[wave, op[1], op[2]] = slot
                holds[op[1], op[3]] = op[2]
            elif op[0] == "vm":
                while len(pending) > op[1]:
                    arrived[(wave, *pending.pop(0))] = slot
            elif op[0] == "read":
                key = (wave, op[1], holds[op[1], op[2]])
                assert key not in reads, f"{key} read twice"
                reads[key] = slot
                unread.append(key)
            else:  # lgkm: the fragment reads so far are in registers
                for r in unread:
                    done[r] = slot
                unread = []
        assert not pending, (nk, blocks, pending)  # nothing lands after the loop
        assert not unread
        bars.append(slot)
    assert bars[0] == bars[1], bars  # every wave passes as many barriers
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
    source = loop_source("mainloop_pair" if pair else "mainloop_quad")
    assert all(check(source, nk, blocks, pair) for nk in range(1, 14))


@pytest.mark.parametrize("pair", [False, True])
def test_no_looser_wait_keeps_the_ring_protocol(pair):
    """Each wait of the stage, loosened by one half tile (two pieces) in the text, breaks the protocol."""
    stage, rest = loop_source("mainloop_pair" if pair else "mainloop_quad")
    waits = [m for m in re.finditer(r"vm_traced\(int_constant<(.*?)>\(\)\)", stage)]
    assert len(waits) == (2 if pair else 4)
    broken = 0
    for m in waits:
        looser = stage[:m.start(1)] + re.sub(r"(?<=[?:] )\d+", lambda d: str(int(d.group()) + 2), m.group(1)) + stage[m.end(1):]
        try:
            for nk in range(1, 14):
                check((looser, rest), nk, False, pair)
        except (AssertionError, KeyError):
            broken += 1
    assert broken == len(waits)


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
