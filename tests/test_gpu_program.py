"""Parity of the control-flow runtime (non-blocking scheduler over the GPU
kernels) with the sequential interpreter of the oracle: every output's shares
or public values, every sigma_i and the verdict, bit for bit, and the number of
block entries; plus the public-operand kernel and the runtime's errors."""
import numpy as np
import pytest
import torch

import oracle.fast as F
from oracle.program import Exec, parse, run_program
from tests._util import dev, host, ints_of_sigma, share_to_dev
from workloads import P61, P127, P_PAPER, programs as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_11112_amd import spdz
    spdz.lib()


def ctx_for(p, n, seed, check_seed):
    from paper_2512_11112_amd.spdz import Context, deal_alpha
    return Context(n, p, deal_alpha(p, n, seed), check_seed)


PROGRAMS = [("pipeline", P.pipeline(3001)), ("branch", P.branch(777)), ("loop", P.loop(1000, 5)),
            ("nested", P.nested(257, 3)), ("select_shl_load", P.select_shl_load(4099, 1000, 77)),
            ("revealed_branch", P.revealed_branch(513)), ("opened_operand", P.opened_operand(3001)),
            ("layer", P.layer(300, 70, 16)), ("layer_public_bias", P.layer_public_bias(300, 70, 16)),
            ("loop_program", P.loop_program(2048, 4)), ("one_block_loop", P.one_block_loop(1000, 5)),
            ("phi_swap", P.phi_swap(777, 4)), ("public_div_mod", P.public_div_mod(1001)),
            ("public_phi_swap", P.public_phi_swap(999, 6)), ("broadcast", P.broadcast(3001)),
            ("loop_reads_source", P.loop_reads_source(1000, 4)), ("lane_constants", P.lane_constants(333)),
            ("concatenation", P.concatenation(1001))]


@pytest.mark.parametrize("handoff", [True, False])
@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("p,n", [(P_PAPER, 2), (P61, 3), (P127, 2)])
@pytest.mark.parametrize("name,text", PROGRAMS)
def test_program_matches_oracle(name, text, p, n, fuse, handoff):
    """Fused element-wise runs (default) and node-by-node execution, phis that take their
    sources' buffers (default) and phis that copy: all match the oracle."""
    from paper_2512_11112_amd.spdz import Program
    if name.startswith("layer") and p == P127:
        pytest.skip("layers need a single-limb field")
    print(f"case {name} p-bits={p.bit_length()} n={n} fuse={fuse} handoff={handoff}", flush=True)
    seed, check = 21, 22
    ref = run_program(text, p, n, seed, check)
    ctx = ctx_for(p, n, seed, check)
    prog = Program(ctx, text, fuse=fuse, handoff=handoff)
    ok, sigma, ms = prog.run(seed)
    check_run(prog, ref, ok, sigma, ms, name)
    prog.close()


def check_run(prog, ref, ok, sigma, ms, name):
    """Every output (shares and MAC shares, or public values), the verdict, every sigma_i,
    the block entries and the number of opened values equal the oracle's."""
    for o, v in ref["outputs"].items():
        got = prog.output(o)
        if isinstance(v, F.Shares):
            assert np.array_equal(host(got.val), v.val), f"{name}: output {o} values"
            assert np.array_equal(host(got.mac), v.mac), f"{name}: output {o} MAC shares"
        else:
            assert np.array_equal(host(got), v), f"{name}: public output {o}"
    assert ok == ref["ok"] and ok
    assert sigma == ints_of_sigma(ref["sigma"])
    st = prog.stats()
    assert st["block_entries"] == ref["entries"]
    assert st["opened"] == sum(o.shape[1] for o in ref["opened"])
    assert ms > 0


@pytest.mark.parametrize("seed", range(160))
def test_random_program_matches_oracle(seed):
    """Seeded random programs (public branches merged by phis that may mix a public and a
    secret value, loops of one block whose phis may take each other's values, zero-trip
    header loops, nested regions, opens fed back as public operands, sums broadcast back)
    at widths 1 .. 4099 over the three fields and 2, 3, 4 or 8 parties: fused and node by node,
    phis handing off their buffers and copying, each equal to the oracle."""
    from paper_2512_11112_amd.spdz import Program
    p, n = [(P_PAPER, 2), (P61, 3), (P127, 2), (P_PAPER, 3), (P61, 4), (P_PAPER, 8)][seed % 6]
    W = [1, 63, 64, 65, 1000, 4099][seed // 6 % 6]
    text = P.random_program(seed, W, regions=4 + seed % 5, depth=3 if seed % 3 == 0 else 2)
    ref = run_program(text, p, n, seed, seed + 1)
    for fuse, handoff in ((True, True), (True, False), (False, True), (False, False)):
        print(f"case random seed={seed} W={W} p-bits={p.bit_length()} n={n} fuse={fuse} handoff={handoff}",
              flush=True)
        ctx = ctx_for(p, n, seed, seed + 1)
        prog = Program(ctx, text, fuse=fuse, handoff=handoff)
        ok, sigma, ms = prog.run(seed)
        check_run(prog, ref, ok, sigma, ms, f"random {seed}")
        prog.close()
        ctx.close()


def test_program_reruns_are_identical():
    """A second run of the same program object (new MAC-check epoch) matches the oracle at epoch 1."""
    from paper_2512_11112_amd.spdz import Program
    p, n, text = P_PAPER, 2, P.loop(64, 3)
    ctx = ctx_for(p, n, 5, 6)
    prog = Program(ctx, text)
    r1 = prog.run(5)
    r2 = prog.run(5)
    ref1 = run_program(text, p, n, 5, 6, epoch=0)
    ref2 = run_program(text, p, n, 5, 6, epoch=1)
    assert r1[1] == ints_of_sigma(ref1["sigma"]) and r2[1] == ints_of_sigma(ref2["sigma"])
    assert r1[0] and r2[0]
    out = prog.output(6)   # the loop's result (a phi that took its source's buffer) after two runs
    assert np.array_equal(host(out.val), ref2["outputs"][6].val) and np.array_equal(host(out.mac), ref2["outputs"][6].mac)


@pytest.mark.parametrize("p,n", [(P_PAPER, 3), (P127, 2)])
def test_public_op_modes(p, n):
    """x + v, x * v (vector and scalar v) and share(v) against the oracle's definitions."""
    from paper_2512_11112_amd.spdz import SPDZ_PUB_ADD, SPDZ_PUB_MUL, SPDZ_PUB_SHARE, ShareTensor, public_op
    W = 5000
    text = f"input 1 private {W} 0\ninput 2 public {W} 1\ninput 3 public 1 2\nblock 0\nret\n"
    ex = Exec(parse(text, p), p, n, 9, 9)
    ex.run()
    x, v, s = ex.val[1], ex.val[2], ex.val[3]
    ctx = ctx_for(p, n, 9, 9)
    xd, vd, sd = share_to_dev(x), dev(v), dev(s)
    L = ex.f.L
    for mode, pub, want in [(SPDZ_PUB_ADD, vd, ex.add_pub(x, v)), (SPDZ_PUB_MUL, vd, ex.mul_pub(x, v)),
                            (SPDZ_PUB_ADD, sd, ex.add_pub(x, ex.pub(3, W))),
                            (SPDZ_PUB_MUL, sd, ex.mul_pub(x, ex.pub(3, W)))]:
        out = public_op(ctx, mode, xd, pub, ShareTensor.empty(n, L, W))
        torch.cuda.synchronize()
        assert np.array_equal(host(out.val), want.val) and np.array_equal(host(out.mac), want.mac)
    out = public_op(ctx, SPDZ_PUB_SHARE, None, vd, ShareTensor.empty(n, L, W))
    torch.cuda.synchronize()
    want = ex.share_pub(v)
    assert np.array_equal(host(out.val), want.val) and np.array_equal(host(out.mac), want.mac)


@pytest.mark.parametrize("p,n", [(P_PAPER, 3), (P127, 2)])
def test_public_op_in_place(p, n):
    """out may be x: x + v and x * v written over x give the same shares as into a fresh buffer."""
    from paper_2512_11112_amd.spdz import SPDZ_PUB_ADD, SPDZ_PUB_MUL, ShareTensor, public_op
    W = 3001
    text = f"input 1 private {W} 0\ninput 2 public {W} 1\nblock 0\nret\n"
    ex = Exec(parse(text, p), p, n, 9, 9)
    ex.run()
    x, v = ex.val[1], ex.val[2]
    ctx = ctx_for(p, n, 9, 9)
    vd = dev(v)
    for mode, want in [(SPDZ_PUB_ADD, ex.add_pub(x, v)), (SPDZ_PUB_MUL, ex.mul_pub(x, v))]:
        xd = share_to_dev(x)
        out = public_op(ctx, mode, xd, vd, xd)
        torch.cuda.synchronize()
        assert np.array_equal(host(out.val), want.val) and np.array_equal(host(out.mac), want.mac)


def test_program_errors():
    from paper_2512_11112_amd.spdz import Program, ProgramError, SpdzError
    ctx = ctx_for(P_PAPER, 2, 1, 1)
    with pytest.raises(ProgramError, match="secret"):
        Program(ctx, P.secret_branch(8))
    with pytest.raises(ProgramError, match="widths"):
        Program(ctx, "input 1 private 4 0\ninput 2 private 5 1\nblock 0\n3 = add 1 2\nret\n")
    # a load whose public start runs past its base: a run-time error, nothing left enqueued
    bad = "input 1 private 10 0\nconst 2 1 8\nblock 0\n3 = load 1 2 5\nret\n"
    prog = Program(ctx, bad)
    with pytest.raises(SpdzError, match="beyond"):
        prog.run(1)
    prog.close()


@pytest.mark.parametrize("pool_seed", [31, 99])
def test_predealt_triples_give_the_same_run(pool_seed):
    """Triples dealt ahead for the first two executions (or for another seed, then unused):
    the run still matches the oracle bit for bit."""
    from paper_2512_11112_amd.spdz import Program
    p, n, text = P_PAPER, 2, P.loop_program(1000, 5)
    ref = run_program(text, p, n, 31, 32)
    ctx = ctx_for(p, n, 31, 32)
    prog = Program(ctx, text)
    prog.predeal(pool_seed, 2)
    ok, sigma, _ = prog.run(31)
    got = prog.output(6)
    assert np.array_equal(host(got.val), ref["outputs"][6].val)
    assert np.array_equal(host(got.mac), ref["outputs"][6].mac)
    assert ok and sigma == ints_of_sigma(ref["sigma"])


@pytest.mark.parametrize("p,n", [(P_PAPER, 2), (P61, 4), (P127, 2), (P61, 8), (P_PAPER, 8)])
def test_fused_groups_formed_and_identical(p, n):
    """The loop body's chain (3 products, 2 additions) is one fused run where the slots fit
    (none at 8 parties: a product needs 3 slots); fused and unfused runs give the same bits."""
    from paper_2512_11112_amd.spdz import Program
    text = P.loop_program(3001, 3)
    # one context each: every run starts a new MAC-check epoch of its context
    a, b = Program(ctx_for(p, n, 4, 5), text, fuse=True), Program(ctx_for(p, n, 4, 5), text, fuse=False)
    word = 4 if p == P_PAPER else 8
    assert (a.n_groups >= 1) == (n * (2 if p == P127 else 1) * 2 * word * 256 * 3 <= 61440)
    ra, rb = a.run(4), b.run(4)
    assert ra[0] and rb[0] and ra[1] == rb[1]
    for o in (6, 15):
        ga, gb = a.output(o), b.output(o)
        if hasattr(ga, "val"):
            assert np.array_equal(host(ga.val), host(gb.val)) and np.array_equal(host(ga.mac), host(gb.mac))
        else:
            assert np.array_equal(host(ga), host(gb))
    if a.n_groups:
        assert a.stats()["launches"] < b.stats()["launches"]
    else:
        assert a.stats()["launches"] == b.stats()["launches"]
    ref = run_program(text, p, n, 4, 5)
    assert ra[1] == ints_of_sigma(ref["sigma"])
    a.close()
    b.close()


def test_fused_public_operands():
    """Fused runs with public scalars and vectors on either side of +, - and *."""
    from paper_2512_11112_amd.spdz import Program
    W = 777
    text = f"""
input 1 private {W} 0
input 2 private {W} 1
input 3 public {W} 2
const 4 1 7
output 12
block 0
5 = mul 1 2
6 = sub 5 3
7 = sub 3 6
8 = mul 7 4
9 = add 4 8
10 = sub 9 4
11 = mul 3 10
12 = mul 11 1
ret
"""
    for p, n in [(P_PAPER, 2), (P61, 3), (P127, 2)]:
        ref = run_program(text, p, n, 8, 9)
        ctx = ctx_for(p, n, 8, 9)
        prog = Program(ctx, text)
        assert prog.n_groups == 1
        ok, sigma, _ = prog.run(8)
        got = prog.output(12)
        assert np.array_equal(host(got.val), ref["outputs"][12].val)
        assert np.array_equal(host(got.mac), ref["outputs"][12].mac)
        assert ok and sigma == ints_of_sigma(ref["sigma"])
        prog.close()


@pytest.mark.timeout(600)
@pytest.mark.parametrize("fuse", [True, False])
def test_program_full_size(fuse):
    """The runtime at the benchmark's configuration (loop program, width 2^22, 16 iterations,
    2 parties, p = 2^32 - 5, triples dealt ahead): every element of the accumulator
    reconstructs to acc <- acc y + x iterated 16 times from acc = x (values below 2^32, so
    uint64 arithmetic is exact), its MAC shares to alpha times it, the opened sum to the sum of
    all elements, and the MAC check accepts."""
    from paper_2512_11112_amd.spdz import Program
    p, n, W, T, seed = P_PAPER, 2, 1 << 22, 16, 1
    print(f"case loop program W={W} T={T} fuse={fuse}", flush=True)
    ctx = ctx_for(p, n, seed, seed)
    prog = Program(ctx, P.loop_program(W, T), fuse=fuse)
    prog.predeal(seed, T)
    ok, sigma, _ = prog.run(seed)
    assert ok and sum(sigma) % p == 0
    f = F.Field(p)
    x = f.deal_values(seed, 0, W)[0]
    y = f.deal_values(seed, 1, W)[0]
    acc = x.copy()
    P64 = np.uint64(p)
    for _ in range(T):
        acc = (acc * y + x) % P64
    got = prog.output(6)
    v, m = host(got.val).reshape(n, W), host(got.mac).reshape(n, W)
    assert np.array_equal((v[0] + v[1]) % P64, acc)
    alpha = np.uint64(sum(int(a) for a in f.alpha_shares(n, seed)[:, 0]) % p)
    assert np.array_equal((m[0] + m[1]) % P64, (acc * alpha) % P64)
    s = host(prog.output(15))
    assert int(s.reshape(-1)[0]) == int(acc.astype(object).sum() % p)
    prog.close()


# --------------------------------------------------------------------------
# programs emitted by the LLVM front end from annotated C (tests/frontend/), run by the
# runtime fused and node by node, against the oracle's interpreter on the same text
# --------------------------------------------------------------------------
def frontend_programs():
    import os
    from paper_2512_11112_amd import frontend as FE
    here = os.path.join(os.path.dirname(os.path.abspath(__file__)), "frontend")
    src = lambda n: open(os.path.join(here, n)).read()
    return [
        ("fig2_layer", FE.translate(src("fig2_layer.c"), "linear_layer", sizes={0: 300, 1: 300 * 70, 2: 70},
                                    defines={"DIN": 300, "DOUT": 70}, slice_size=4800).text),
        ("dot_loop_vw16", FE.translate(src("dot_loop.c"), "dot", sizes={0: 4096, 1: 4096}, bind={2: 4000},
                                       vector_width=16, interleave=2).text),
        ("dot_runtime_vw16", FE.translate(src("dot_runtime.c"), "dot_rt", sizes={0: 4096, 1: 4096},
                                          vector_width=16, interleave=2).text),
        ("matvec_rows", FE.translate(src("matvec.c"), "matvec_sum", sizes={0: 512 * 48, 1: 512},
                                     defines={"DIN": 512, "DOUT": 48}, vector_width=16).text),
        ("axpy_bcast", FE.translate(src("axpy.c"), "axpy_dot", sizes={0: 64, 1: 64}, vector_width=8).text),
        ("branch_runtime_condition", FE.translate(src("branch.c"), "branchy", sizes={0: 64, 1: 64},
                                                  vector_width=8).text),
        ("poly_select", FE.translate(src("poly.c"), "poly", sizes={0: 4}).text),
    ]


@pytest.fixture(scope="module")
def fe_programs():
    return dict(frontend_programs())


@pytest.mark.parametrize("fuse", [True, False])
@pytest.mark.parametrize("name", ["fig2_layer", "dot_loop_vw16", "dot_runtime_vw16", "matvec_rows", "axpy_bcast",
                                  "branch_runtime_condition", "poly_select"])
def test_frontend_program_matches_oracle(fe_programs, name, fuse):
    from paper_2512_11112_amd.spdz import Program
    text = fe_programs[name]
    p, n, seed, check = P_PAPER, 2, 31, 32
    print(f"case front-end program {name} fuse={fuse}", flush=True)
    ref = run_program(text, p, n, seed, check)
    ctx = ctx_for(p, n, seed, check)
    prog = Program(ctx, text, fuse=fuse)
    ok, sigma, ms = prog.run(seed)
    for o, v in ref["outputs"].items():
        got = prog.output(o)
        if isinstance(v, F.Shares):
            assert np.array_equal(host(got.val), v.val), f"{name}: output {o} values"
            assert np.array_equal(host(got.mac), v.mac), f"{name}: output {o} MAC shares"
        else:
            assert np.array_equal(host(got), v), f"{name}: public output {o}"
    assert ok == ref["ok"] and ok
    assert sigma == ints_of_sigma(ref["sigma"])
    prog.close()
    ctx.close()


def test_random_c_functions_on_the_runtime():
    """The seeded random C functions the front end accepts (tests/frontend/random_c.py; lane
    picks, constant vectors with a lane inserted, selects of pointers, vector reductions) run by
    the device runtime, fused and node by node, equal to the oracle's run."""
    import os
    import sys
    from paper_2512_11112_amd import frontend as FE
    from paper_2512_11112_amd.spdz import Program
    sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "frontend"))
    from random_c import random_c
    ran = 0
    for seed in range(40):
        try:
            text = FE.translate(random_c(seed), "fz", sizes={0: 64, 1: 64}, vector_width=[None, 4, 8][seed % 3]).text
        except FE.FrontendError:
            continue
        ref = run_program(text, P_PAPER, 2, seed, seed + 1)
        for fuse in (True, False):
            print(f"case random C seed={seed} fuse={fuse}", flush=True)
            ctx = ctx_for(P_PAPER, 2, seed, seed + 1)
            prog = Program(ctx, text, fuse=fuse)
            ok, sigma, ms = prog.run(seed)
            check_run(prog, ref, ok, sigma, ms, f"random C {seed}")
            prog.close()
            ctx.close()
        ran += 1
    assert ran >= 30


@pytest.mark.parametrize("p,n,W", [(P_PAPER, 2, 65536), (P_PAPER, 2, 65537), (P61, 3, 32768), (P61, 3, 32769),
                                   (P61, 4, 33), (P61, 5, 17), (P61, 8, 1), (P_PAPER, 8, 300), (P_PAPER, 2, 63)])
def test_narrow_and_wide_runs_match_node_by_node(p, n, W):
    """Fused runs on both sides of the width at which they change kernels, and at partial blocks of each number
    of lanes per element: outputs and sigma as with every node its own kernel."""
    from paper_2512_11112_amd import spdz as S
    got = []
    for fuse in (True, False):
        ctx = S.Context(n, p, S.deal_alpha(p, n, 5), 5)
        prog = S.Program(ctx, P.loop_program(W, 3), fuse=fuse)
        ok, sigma, _ = prog.run(5)
        assert ok
        acc = prog.output(6)
        got.append((sigma, acc.val, acc.mac, prog.output(15)))
        prog.close()
        ctx.close()
    assert got[0][0] == got[1][0]
    assert all(torch.equal(a, b) for a, b in zip(got[0][1:], got[1][1:]))


def joining_program(W, trips):
    """A loop of two values carried in one fused run: every kind of instruction of a fused run, a public operand
    of full width and of one element, a value read again in the next iteration, one read only after the loop."""
    return f"""
input 1 private {W} 0
input 2 private {W} 1
input 20 public {W} 7
const 3 1 {trips}
const 4 1 0
const 5 1 1
const 21 1 77
output 6
output 18
output 14
block 0
br 1
block 1
6 = phi 1 0 9 2
18 = phi 2 0 17 2
7 = phi 4 0 10 2
8 = lt 7 3
cbr 8 2 3
block 2
11 = mul 6 2
9 = add 11 1
12 = sub 20 9
13 = mul 12 21
14 = sub 13 20
15 = mul 14 9
16 = add 15 21
17 = sub 16 18
10 = add 7 5
br 1
block 3
ret
"""


@pytest.mark.parametrize("trips", [1, 7, 8, 25])  # 8 and more: several launches of joined runs
@pytest.mark.parametrize("p,n,W", [(P_PAPER, 2, 1), (P_PAPER, 2, 32769), (P61, 2, 1000), (P61, 3, 16384), (P61, 3, 16385),
                                   (P61, 8, 130), (P127, 2, 77), (P127, 2, 32769)])
def test_joined_runs_match_node_by_node(p, n, W, trips):
    """Iterations of a loop that share a launch, both kernels: outputs and sigma as with every node its own kernel,
    and, at small sizes, the oracle's."""
    from paper_2512_11112_amd import spdz as S
    text, got = joining_program(W, trips), []
    for fuse, ahead in ((True, True), (True, False), (False, True)):
        ctx = S.Context(n, p, S.deal_alpha(p, n, 5), 5)
        prog = S.Program(ctx, text, fuse=fuse)
        if ahead:
            prog.predeal(5, trips)
        sigma = []
        for _ in range(2):  # a second run starts anew (and a new epoch of the check)
            ok, s, _ = prog.run(5)
            assert ok
            sigma.append(s)
        outs = [prog.output(o) for o in (6, 18, 14)]
        got.append((sigma, [t for o in outs for t in (o.val, o.mac)]))
        prog.close()
        if W * trips <= 2000:
            ref = run_program(text, p, n, 5, 5)
            assert sigma[0] == ints_of_sigma(ref["sigma"])
            assert np.array_equal(host(outs[1].val), ref["outputs"][18].val)
        ctx.close()
    for g in got[:2]:
        assert g[0] == got[2][0]
        assert all(torch.equal(a, b) for a, b in zip(g[1], got[2][1]))


@pytest.mark.parametrize("p,n", [(P61, 3), (P127, 2)])
@pytest.mark.parametrize("layout", ["dense", "padded", "parties_apart", "limbs_apart"])
def test_output_into_strided_shares(p, n, layout):
    """spdz_prog_output into every spacing of planes: one copy, one per limb, one per plane."""
    import ctypes
    from paper_2512_11112_amd import spdz as S
    W, L = 301, 2 if p == P127 else 1
    ps, ls = {"dense": (L * W, W), "padded": (L * (W + 5), W + 5), "parties_apart": (L * W + 9, W + 2 if L > 1 else W),
              "limbs_apart": (W, n * W)}[layout]
    ctx = ctx_for(p, n, 4, 5)
    prog = S.Program(ctx, P.loop_program(W, 2), fuse=True)
    assert prog.run(4)[0]
    ref = prog.output(6)
    size = n * ps + L * ls
    val, mac = (torch.zeros(size, dtype=torch.int64, device="cuda") for _ in range(2))
    d = S.Shares(val=val.data_ptr(), mac=mac.data_ptr(), len=W, party_stride=ps, limb_stride=ls)
    assert S.lib().spdz_prog_output(prog._h, 6, ctypes.byref(d), None) == 0
    for got, want in ((host(val), host(ref.val)), (host(mac), host(ref.mac))):
        want, left = want.reshape(n, L, W), got.copy()
        for i in range(n):
            for l in range(L):
                at = i * ps + l * ls
                assert np.array_equal(got[at:at + W], want[i, l])
                left[at:at + W] = 0
        assert not left.any()
    prog.close()
    ctx.close()


@pytest.mark.parametrize("p,n,W,trips", [(P_PAPER, 2, 64, 20), (P61, 2, 70000, 9), (P127, 2, 77, 1)])
@pytest.mark.parametrize("fuse", [True, False])
def test_launch_counter_counts_launches(p, n, W, trips, fuse):
    """spdz_prog_stats counts a launch of several fused runs, and a sum, as the one launch it is: the kernel timer
    of the same run, which brackets each launch, saw as many (triples dealt ahead, phis handed over)."""
    from paper_2512_11112_amd import spdz as S
    ctx = S.Context(n, p, S.deal_alpha(p, n, 5), 5)
    prog = S.Program(ctx, P.loop_program(W, trips), fuse=fuse)
    prog.predeal(5, trips)
    ctx.spdz_timing_enable(True)
    assert prog.run(5)[0]
    timed = {k: ctx.spdz_timing_get(k)[1] for k in ("fused", "beaver", "linear", "reduce", "open")}
    assert timed["reduce"] == timed["open"] == 1 and (timed["fused"] > 0) == fuse
    assert prog.stats()["launches"] == sum(timed.values())
    prog.close()
    ctx.close()


@pytest.mark.parametrize("apart", [(1 << 28) - 1, 1 << 28])
def test_output_into_shares_far_apart(apart):
    """spdz_prog_output where the parties' planes lie as far apart as the rows of one copy may (2^31 - 1 bytes on
    this device), and further."""
    import ctypes
    from paper_2512_11112_amd import spdz as S
    W, n = 300, 2
    ctx = ctx_for(P_PAPER, n, 4, 5)
    prog = S.Program(ctx, P.loop_program(W, 2), fuse=True)
    assert prog.run(4)[0]
    ref = prog.output(6)
    val, mac = (torch.zeros((n - 1) * apart + W, dtype=torch.int64, device="cuda") for _ in range(2))
    d = S.Shares(val=val.data_ptr(), mac=mac.data_ptr(), len=W, party_stride=apart, limb_stride=W)
    assert S.lib().spdz_prog_output(prog._h, 6, ctypes.byref(d), None) == 0
    for got, want in ((val, ref.val), (mac, ref.mac)):
        for i in range(n):
            assert torch.equal(got[i * apart:i * apart + W], want[i, 0])
        assert int((got != 0).sum()) == int((want != 0).sum())
    prog.close()
    ctx.close()


@pytest.mark.parametrize("past", [0, 1])
@pytest.mark.parametrize("p,n,lanes", [(P_PAPER, 2, 4), (P61, 2, 4), (P127, 2, 4), (P61, 3, 8), (P_PAPER, 4, 8),
                                       (P61, 5, 16), (P_PAPER, 8, 16)])
def test_fused_runs_where_the_kernels_change(p, n, lanes, past):
    """The largest width of the narrow kernel (two blocks of 256 lanes per CU) and the smallest of the wide one, for
    each number of lanes per element: outputs and sigma as with every node its own kernel."""
    from paper_2512_11112_amd import spdz as S
    W = 2 * torch.cuda.get_device_properties(0).multi_processor_count * 256 // lanes + past
    for text, outs in ((P.loop_program(W, 4), (6, 15)), (joining_program(W, 4), (6, 18, 14))):
        got = []
        for fuse in (True, False):
            ctx = S.Context(n, p, S.deal_alpha(p, n, 5), 5)
            prog = S.Program(ctx, text, fuse=fuse)
            assert prog.n_groups > 0
            prog.predeal(5, 4)
            ok, sigma, _ = prog.run(5)
            assert ok
            vals = [prog.output(o) for o in outs]
            got.append((sigma, [t for v in vals for t in ((v.val, v.mac) if hasattr(v, "val") else (v,))]))
            prog.close()
            ctx.close()
        assert got[0][0] == got[1][0]
        assert all(torch.equal(a, b) for a, b in zip(got[0][1], got[1][1]))


@pytest.mark.parametrize("p,n,W", [(P61, 5, 1), (P61, 5, 130), (P_PAPER, 8, 17), (P_PAPER, 8, 130)])
def test_joined_runs_of_sixteen_lanes(p, n, W):
    """Runs that share a launch with 16 lanes per element, at partial blocks: the oracle's outputs and sigma."""
    from paper_2512_11112_amd import spdz as S
    trips = 9
    text = joining_program(W, trips)
    ref = run_program(text, p, n, 5, 5)
    for ahead in (True, False):
        ctx = S.Context(n, p, S.deal_alpha(p, n, 5), 5)
        prog = S.Program(ctx, text)
        assert prog.n_groups > 0
        if ahead:
            prog.predeal(5, trips)
        ok, sigma, _ = prog.run(5)
        assert ok and sigma == ints_of_sigma(ref["sigma"])
        if ahead:
            assert prog.stats()["launches"] < trips  # (dealt on the fly, each iteration is its own launch)
        for o in (6, 18, 14):
            out = prog.output(o)
            assert np.array_equal(host(out.val), ref["outputs"][o].val) and np.array_equal(host(out.mac), ref["outputs"][o].mac)
        prog.close()
        ctx.close()
