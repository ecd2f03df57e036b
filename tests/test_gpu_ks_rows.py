"""The fused kernels of key switching (k_ks_rows): sums of a ciphertext and its
rotation, and outputs that overlap another item's operands, for every
row-pass length, both digit arrangements, and full, ragged and lowest levels;
bit-exact against the oracle."""

import ctypes

import pytest

import synth as S
from oracle import ckks as C
from paper_1908_06972_amd import native as N

from .ks_split_host import split
from .test_gpu_modup_fused import CASES, STEPS, World, world

pytestmark = pytest.mark.gpu


@pytest.fixture(params=list(CASES))
def fused(request):
    w = world(request.param)
    w.ctx.ntt_set_schedule(False, [c for c in w.col16 if c[1] == 0][0])
    yield w
    w.ctx.bconv_mode(True)
    w.ctx.ntt_set_schedule(False, None)


def levels(w):
    return sorted({w.op.L, w.op.L - 1, 1})


@pytest.mark.parametrize("pairs", [True, False])
def test_rotate_and_sum(fused, pairs):
    """ct + ROTATE(ct, 1): the addend enters through the accumulators."""
    w = fused
    w.ctx.bconv_mode(True, pairs=pairs)
    for level in levels(w):
        cts = [w.enc_pair(300 + 10 * level + i, level) for i in range(2)]
        for g, (_, o) in zip(w.ctx.total_sum_batch([c[0] for c in cts], 2), cts):
            w.assert_same(g, C.hadd(w.op, o, C.rotate(w.op, o, 1, w.rot[1])))


def test_outputs_over_other_items_operands(fused):
    """Each output is the next item's operand: the operands are read as they
    were before the call."""
    w = fused
    for level in levels(w):
        a, b = ([w.enc_pair(s + 10 * level + i, level) for i in range(3)] for s in (400, 500))
        want = [C.hmul_relin(w.op, x[1], y[1], w.rlk) for x, y in zip(a, b)]
        out = w.ctx.mul_relin_batch([x[0] for x in a], [y[0] for y in b], out=[a[1][0], b[0][0], a[0][0]])
        for g, o in zip(out, want):
            w.assert_same(g, o)
        a = [w.enc_pair(600 + 10 * level + i, level) for i in range(3)]
        want = [C.rotate(w.op, x[1], 5, w.rot[5]) for x in a]
        for g, o in zip(w.ctx.rotate_batch([x[0] for x in a], 5, out=[a[1][0], a[2][0], a[0][0]]), want):
            w.assert_same(g, o)


@pytest.mark.parametrize("bits", [51, 55, 59])
def test_integer_rows_of_other_sizes(bits):
    """Every prime on the 64-bit integer path and below 60 bits: products with
    relinearisation and their rescale under every transform schedule."""
    w = World(dict(log_n=12, n_q=4, q0_bits=bits, q_bits=bits, n_p=2, p_bits=bits, dnum=2, scale=2 ** 40))
    (ga, oa), (gb, ob) = w.enc_pair(1, 4), w.enc_pair(2, 4)
    prod = C.hmul_relin(w.op, oa, ob, w.rlk)
    low = C.rescale(w.op, prod)
    for sched in w.ctx.ntt_candidates():
        for inverse in (False, True):
            w.ctx.ntt_set_schedule(inverse, sched)
        g = w.ctx.mul_relin(ga, gb)
        w.assert_same(g, prod)
        w.assert_same(w.ctx.rescale(g), low)


@pytest.mark.parametrize("name,n_q,n_p,items", [("a6_n12", 36, 6, 64), ("a3_n13", 18, 3, 64), ("a2_n14", 10, 2, 64),
                                                ("a4_n15", 10, 5, 64)])
def test_large_launches_equal_small_ones(name, n_q, n_p, items):
    """Enough items for the 8-residue forms of the fused kernels (a launch of
    more than 2^23 words; the last case's special rows too), against the same
    calls one item at a time."""
    w = World(dict(CASES[name], n_q=n_q, n_p=n_p, dnum=n_q // n_p))
    L = w.op.L
    assert items * L * w.n > 2 ** 23 >= 2 * L * w.n
    a, b = ([w.ctx.encrypt_seeded(S.plaintext_coeffs(S.rng(s + i), w.n, 2 ** 30), L, w.op.scale, s + i)
             for i in range(items)] for s in (3000, 4000))
    prod = w.ctx.mul_relin_batch(a, b)
    for big, one in ((prod, lambda i: w.ctx.mul_relin(a[i], b[i])),
                     (w.ctx.rotate_batch(a, 5), lambda i: w.ctx.rotate(a[i], 5)),
                     (w.ctx.total_sum_batch(b, 2), lambda i: w.ctx.total_sum(b[i], 2)),
                     (w.ctx.rescale_batch(prod), lambda i: w.ctx.rescale(prod[i]))):
        for i in range(items):
            assert bool((big[i].data == one(i).data).all())


@pytest.mark.parametrize("n_q,n_p,dnum,q_bits,p_bits", [(5, 1, 5, 40, 60), (8, 1, 8, 40, 60), (6, 2, 3, 55, 60),
                                                        (7, 3, 3, 45, 50)])
def test_small_launches_in_parts(n_q, n_p, dnum, q_bits, p_bits):
    """Special rows in two to four parts of one or two digits (integer and
    fp64), none to all of the ciphertext rows on the integer path, at every
    level."""
    w = World(dict(log_n=12, n_q=n_q, q0_bits=60, q_bits=q_bits, n_p=n_p, p_bits=p_bits, dnum=dnum, scale=2 ** 40))
    for level in range(w.op.L, 0, -1):
        (ga, oa), (gb, ob) = w.enc_pair(10 + level, level), w.enc_pair(30 + level, level)
        w.assert_same(w.ctx.mul_relin(ga, gb), C.hmul_relin(w.op, oa, ob, w.rlk))
        rot = C.rotate(w.op, oa, 1, w.rot[1])
        w.assert_same(w.ctx.rotate(ga, 1), rot)
        w.assert_same(w.ctx.total_sum(ga, 2), C.hadd(w.op, oa, rot))


@pytest.mark.parametrize("log_n", [13, 16])
def test_fp64_special_rows_in_parts(log_n):
    """50-bit special primes in three and four parts where the inverse row
    pass (9 and 12 stages) ends on a stage that does not reduce."""
    w = World(dict(log_n=log_n, n_q=4, q0_bits=50, q_bits=50, n_p=1, p_bits=50, dnum=4, scale=2 ** 40))
    for level in (4, 3):
        assert split(1, level, 1, 1, 0, log_n) == (level, 1, False)
        (ga, oa), (gb, ob) = w.enc_pair(50 + level, level), w.enc_pair(70 + level, level)
        w.assert_same(w.ctx.mul_relin(ga, gb), C.hmul_relin(w.op, oa, ob, w.rlk))
        w.assert_same(w.ctx.rotate(ga, 5), C.rotate(w.op, oa, 5, w.rot[5]))


@pytest.mark.parametrize("n_q,n_p,dnum", [(36, 12, 3), (50, 12, 5)])
def test_conversions_of_many_rows(n_q, n_p, dnum):
    """Digits of 12 limbs, 12 special primes and long chains, whose operands
    and constants pass 64 KB of LDS: on the fused kernels, one item and a
    batch, against the oracle."""
    w = World(dict(log_n=12, n_q=n_q, q0_bits=60, q_bits=40, n_p=n_p, p_bits=60, dnum=dnum, scale=2 ** 40))
    for level in (n_q, n_q - 1, 1):
        pairs = [(w.enc_pair(50 + 3 * level + i, level), w.enc_pair(300 + 3 * level + i, level)) for i in range(3)]
        prod = [C.hmul_relin(w.op, x[1], y[1], w.rlk) for x, y in pairs]
        N.check(w.ctx.lib.pft_prof_enable(w.ctx.handle, 1 << 3))  # the key inner product's kernels
        w.assert_same(w.ctx.mul_relin(pairs[0][0][0], pairs[0][1][0]), prod[0])
        var = (ctypes.c_uint32 * 16)()
        k = w.ctx.lib.pft_prof_read_variants(w.ctx.handle, 3, 16, var, None, None, None, None)
        N.check(w.ctx.lib.pft_prof_enable(w.ctx.handle, 0))
        assert k > 0 and min(var[:k]) >= 1024  # k_ks_rows
        for g, o in zip(w.ctx.mul_relin_batch([x[0] for x, _ in pairs], [y[0] for _, y in pairs]), prod):
            w.assert_same(g, o)
        rot = C.rotate(w.op, pairs[0][0][1], 5, w.rot[5])
        w.assert_same(w.ctx.rotate(pairs[0][0][0], 5), rot)


@pytest.mark.parametrize("cache", [0, 1])
def test_op_list_rotations_of_many_steps(cache):
    """One wave of rotations by different steps at two levels, more of them
    than a launch takes, the identity among them, and their sums in place;
    with and without a limited key cache."""
    w = World(CASES["a2_n12"])
    ctx = w.ctx
    if cache:
        ctx = type(ctx)(w.lp)
        ctx.set_key_cache(cache)
        ctx.keygen(31, STEPS)
    x = [w.enc_pair(900 + i, lv) for i, lv in enumerate((4, 3))]
    cts, ops, want = [g for g, _ in x], [], []
    rot = {(i, st): o if st == 0 else C.rotate(w.op, o, st, w.rot[st]) for i, (_, o) in enumerate(x) for st in (0, 1, 5)}
    for i in range(240):
        src, st = (i // 2) % 2, (0, 1, 5)[i % 3]
        cts.append(ctx.empty_ct(x[src][0].level))
        ops.append(("rotate", src, 0, len(cts) - 1, st, 0))
        want.append((src, st))
    ops += [("add", 2 + i, want[i][0], 2 + i, 0, 0) for i in range(240)]
    ctx.exec_batch(cts, ops)
    for i, key in enumerate(want):
        if i < 12 or i > 230:
            w.assert_same(cts[2 + i], C.hadd(w.op, rot[key], x[key[0]][1]))
        else:
            assert bool((cts[2 + i].data == cts[2 + want.index(key)].data).all())


@pytest.mark.parametrize("n_slots", [1, 2, 4])
def test_total_sum_over_its_inputs(n_slots):
    """Outputs that are the inputs, in order and shifted by one: read before
    they are written."""
    w = world("a2_n12")
    ctx = type(w.ctx)(w.lp)
    ctx.keygen(31, [1, 2])
    enc = [lambda i=i: ctx.encrypt_seeded(S.plaintext_coeffs(S.rng(950 + i), w.n, 2 ** 30), 3, w.op.scale, 950 + i)
           for i in range(3)]
    want = [ctx.total_sum(e(), n_slots) for e in enc]
    for shift in (0, 1):
        x = [e() for e in enc]
        out = ctx.total_sum_batch(x, n_slots, out=[x[(i + shift) % 3] for i in range(3)])
        for g, o in zip(out, want):
            assert bool((g.data == o.data).all())
