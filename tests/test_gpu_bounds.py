"""GPU kernels at the bounds that keep their fp64 sums of residues exact: inputs made so that a partial sum is as large
as it can get, against the CPU oracle (whole numbers: every comparison is exact)."""
import sys

import numpy as np
import pytest

from oracle import bgv as B
from oracle import circuit as CI
from oracle import compiler as OC
from oracle import nt

pytestmark = pytest.mark.gpu
T = 65537


def say(*a):
    print("[gpu-test]", *a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module")
def C():
    from paper_2104_09583_amd import copse
    return copse


def same(exported, oct_):
    assert exported["level"] == oct_.level and len(exported["polys"]) == len(oct_.polys)
    for a, b in zip(exported["polys"], oct_.polys):
        assert a.shape == b.shape and (a == b).all()


def one_branch_forest(C, log_n, n_data, bits):
    """One prime a digit and a tree of one branch over one bit: an evaluation without ciphertext products, so that
    rotations are its only key switches (on the split rings the chain's small q_0 keeps the switches unmerged)."""
    data, q0, sp = (1 << b for b in bits)
    text = "no yes\nB 1 1 L 0 L 1\n"
    oc = OC.compile_forest(text, 3, 1)
    ctx = C.Context(log_n, n_data, q0, data, 1, sp)
    sc = B.BGV(nt.make_chain(log_n, T, n_data, q0, data, 1, sp))
    comp, meta = C.forest_compile(text, 3, 1, log_n)
    pl = CI.make_plan(oc, sc.N, sc.L)
    seed = b"\x41" * 32
    rots = C.compiled_rotations(meta)
    assert 1 in rots
    return ctx, sc, ctx.model_encode(comp), CI.encode_model(sc, pl), pl, \
        ctx.keygen(seed, rots, False), sc.keygen(seed, pl.rotations(), False)


def random_poly(sc, rng):
    return np.stack([rng.integers(0, q, sc.N, dtype=np.uint64) for q in sc.primes[:sc.L + 1]])


@pytest.mark.parametrize("n_data", [9, 10, 17, 18])
def test_rotations_of_many_digits(C, n_data):
    """The fused rotations at the digit counts at which they fold their sums, without a separate column pass."""
    ctx, sc, model, omodel, pl, keys, okeys = one_branch_forest(C, 13, n_data, (49, 44, 49))
    rng = np.random.default_rng(n_data)
    polys = [random_poly(sc, rng) for _ in range(2)]
    query = ctx.import_(polys, ctx.L)
    want = CI.Evaluator(sc, okeys, pl).run([B.Ciphertext(polys, sc.L)], omodel)["result"]
    say("evaluate,", n_data - 1, "digits in the reshuffle")
    cols = (C.PROF_NTT_FWD_COLS, C.PROF_NTT_INV_COLS)
    ctx.profile_enable()
    for kind in cols:
        ctx.profile_read(kind, True)
    same(ctx.export(ctx.evaluate(model, keys, query))[0], want)
    assert [ctx.profile_read(kind)["launches"] for kind in cols] == [0, 0]
