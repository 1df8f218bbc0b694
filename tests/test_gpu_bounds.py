"""GPU kernels at the bounds that keep their fp64 sums of residues exact: inputs made so that a partial sum is as large
as it can get, against the CPU oracle (whole numbers: every comparison is exact)."""
import sys

import numpy as np
import pytest

from oracle import bgv as B
from oracle import circuit as CI
from oracle import compiler as OC
from oracle import nt
from paper_2104_09583_amd import synth

import test_gpu_kernel_edges as edges

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
def lazy_product(a, b, q):
    """The kernels' product a b - rint(fl(a b) fl(1 / q)) q, in whole numbers."""
    return a * b - int(np.rint(float(a) * float(b) * (1.0 / q))) * q


@pytest.mark.parametrize("log_n,bits", [(10, (49, 49, 49)), (13, (49, 44, 49))])
@pytest.mark.parametrize("row", [5, 47])
def test_key_switch_sums_of_46_digits(C, log_n, bits, row):
    """The longest sum of digit x key that an evaluation has, 46 products modulo a 49-bit prime, made as large as it can
    be in one slot of one row (a data row, the special row): added up without a fold it passes 2^53 and loses its last
    bit.  The digits are constants, so that every slot of every row holds them: the query is the constant that the
    reshuffle is to rotate, divided by what the comparison multiplies with."""
    ctx, sc, model, omodel, pl, keys, okeys = one_branch_forest(C, log_n, 47, bits)
    key, q, slot = okeys.rot[sc.galois(1)], sc.primes[row], 77
    v, products = [], []
    for j in range(46):
        k = int(key.b_ntt[j][row][slot])
        r = q * 47 // 100 // 2 * 2 + (j == 45)   # even, the last one odd
        while True:
            a = r * pow(k, -1, q) % q
            if a < sc.primes[j] and lazy_product(a, k, q) == r:
                break
            r -= 2
        v.append(a)
        products.append(r)
    total = np.float64(0.0)
    for r in products:
        total += np.float64(r)
    assert int(total) != sum(products)   # without a fold
    idx = sc.data_idx(sc.L)
    factor = sc.plain_ntt(omodel.G[0], sc.L)
    c1 = np.zeros((sc.L + 1, sc.N), dtype=np.uint64)
    for i in idx[:-1]:   # the limb that the comparison's switch drops stays zero
        qi = sc.primes[i]
        top = v[i] * sc.primes[sc.L] % qi
        c1[i] = np.array([top * pow(int(f), -1, qi) % qi for f in factor[i]], dtype=np.uint64)
    polys = [random_poly(sc, np.random.default_rng(9)), sc.intt(c1, idx)]
    x = B.Ciphertext(polys, sc.L)
    dec = CI.Evaluator(sc, okeys, pl).seccomp([x], omodel)
    assert all(dec.polys[1][i][0] == v[i] and not dec.polys[1][i][1:].any() for i in idx[:-1])
    want = CI.Evaluator(sc, okeys, pl).run([x], omodel)["result"]
    say("evaluate, 46 digits in the reshuffle, log_n", log_n, "row", row)
    same(ctx.export(ctx.evaluate(model, keys, ctx.import_(polys, ctx.L)))[0], want)


@pytest.mark.parametrize("bits", [20, 21, 22])
def test_encrypted_matmul_of_small_primes(C, bits):
    """The unreduced sums of an encrypted model's products with primes of 17 to 22 bits, on both sides of the size (20
    bits) below which their fold interval would not fit its type."""
    log_n, t = 6, 257
    text, n_data, seed = "no yes\nB 1 1 L 0 L 1\n", 4, b"\x43" * 32
    top = 1 << bits
    ctx = C.Context(log_n, n_data, top, top, 1, top, t=t)
    sc = B.BGV(nt.make_chain(log_n, t, n_data, top, top, 1, top))
    comp, meta = C.forest_compile(text, 3, 1, log_n)
    pl = CI.make_plan(OC.compile_forest(text, 3, 1), sc.N, sc.L, encrypted_model=True)
    keys, okeys = ctx.keygen(seed, C.compiled_rotations(meta)), sc.keygen(seed, pl.rotations())
    model, omodel = ctx.model_encode(comp, keys, True, seed), CI.encrypt_model(sc, okeys, pl, seed)
    rng = np.random.default_rng(bits)
    polys = [[random_poly(sc, rng) for _ in range(2)] for _ in range(8)]
    say("evaluate an encrypted model, primes of", bits, "bits")
    got = ctx.evaluate_batch(model, keys, [ctx.import_(p, ctx.L) for p in polys])
    for r, p in zip(got, polys):
        same(ctx.export(r)[0], CI.Evaluator(sc, okeys, pl).run([B.Ciphertext(p, sc.L)], omodel)["result"])


# jobs x limbs x tiles above the count from which a relinearization's finish forms its own inner products: plain rows (a
# prime of 49 bits), and two to eight digits, whose tiles take turns in one buffer; merged with the switch (products) and
# not (an encrypted model's inner sums)
@pytest.mark.parametrize("bits,alpha,enc,groups,spare",
                         [((48, 49, 49), 4, False, 64, 0), ((49, 49, 49), 3, True, 40, 0), ((48, 49, 49), 1, False, 56, 0),
                          ((48, 48, 48), 1, False, 64, 1), ((49, 49, 49), 1, True, 40, 0), ((42, 44, 44), 2, False, 48, 5),
                          ((49, 49, 49), 2, False, 32, 9)])
def test_relinearizations_by_prime_size_and_digit_count(C, bits, alpha, enc, groups, spare):
    edges.evaluate_groups(C, synth.ForestShape(3, 3, 0.9, 3, 4, 3), 74, 13, bits, alpha, enc, groups, spare=spare)
