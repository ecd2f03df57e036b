"""Key switches whose integer ciphertext rows are taken early beside whole
special rows (csrc/ks_split.h): more special primes than a digit has limbs,
several integer rows, and both together, so that the sums of the early rows
and of the special rows crowd the workspace; products, rotations and
rotate-and-sum, bit-exact against the oracle."""

from unittest import mock

import pytest

import synth as S
from oracle import ckks as C

from .ks_split_host import split
from .test_gpu_modup_fused import World

pytestmark = pytest.mark.gpu


def _case(log_n, bits, n_p, dnum, n, level):
    """bits: of each ciphertext prime, descending."""
    two_n, q = 2 << log_n, []
    for b in bits:
        q += C.largest_primes(two_n, b, 1, exclude=set(q))
    p = C.largest_primes(two_n, 60, n_p, exclude=set(q))
    return dict(log_n=log_n, q=q, p=p, dnum=dnum, n=n, level=level)


CASES = {
    "k2a1_n12": _case(12, [60, 40, 40, 40], 2, 4, 40, 2),
    "k4a2_n14": _case(14, [60] + 5 * [40], 4, 3, 6, 3),
    "k2a2_n14": _case(14, [60] + 5 * [40], 2, 3, 9, 3),   # room in any layout
    "ints_n14": _case(14, 6 * [60], 3, 3, 6, 3),
    "two_ints_n15": _case(15, [60, 60, 40, 40], 2, 2, 5, 3),
    "k4a3_n15": _case(15, [60] + 5 * [40], 4, 2, 3, 4),
    "k6a5_n16": _case(16, [60] + 9 * [40], 6, 2, 2, 6),
}


def split_of(c):
    """(parts, digits a part, early) of the case's launches."""
    alpha = -(-len(c["q"]) // c["dnum"])
    return split(c["n"], c["level"], alpha, len(c["p"]), sum(q >= 2 ** 50 for q in c["q"][:c["level"]]), c["log_n"])


def _world(c):
    import paper_1908_06972_amd.ckks as L
    spec = dict(log_n=c["log_n"], n_q=len(c["q"]), q0_bits=0, q_bits=0, n_p=len(c["p"]), p_bits=0, dnum=c["dnum"],
                scale=2 ** 40)
    lp = L.Params.from_primes(c["log_n"], c["q"], c["p"], c["dnum"], 2 ** 40)
    with mock.patch.object(C, "prime_chain", lambda *a: (c["q"], c["p"])), mock.patch.object(L, "Params", lambda *a: lp):
        return World(spec)


@pytest.mark.parametrize("name", list(CASES))
def test_early_rows_beside_whole_special_rows(name):
    c = CASES[name]
    parts, _, early = split_of(c)
    assert early and parts == 1
    w, n, level = _world(c), c["n"], c["level"]
    enc = lambda s: w.ctx.encrypt_seeded(S.plaintext_coeffs(S.rng(s), w.n, 2 ** 30), level, w.op.scale, 500 + s)  # noqa: E731
    checked = sorted({0, n // 2, n - 1})
    pairs = {i: (w.enc_pair(100 + i, level), w.enc_pair(200 + i, level)) for i in checked}
    a = [pairs[i][0][0] if i in pairs else enc(100 + i) for i in range(n)]
    b = [pairs[i][1][0] if i in pairs else enc(200 + i) for i in range(n)]
    prod, rot, total = w.ctx.mul_relin_batch(a, b), w.ctx.rotate_batch(a, 1), w.ctx.total_sum_batch(a, 2)
    for i in checked:
        oa, ob = pairs[i][0][1], pairs[i][1][1]
        w.assert_same(prod[i], C.hmul_relin(w.op, oa, ob, w.rlk))
        o = C.rotate(w.op, oa, 1, w.rot[1])
        w.assert_same(rot[i], o)
        w.assert_same(total[i], C.hadd(w.op, oa, o))
    for i in range(n):  # one item at a time
        assert bool((prod[i].data == w.ctx.mul_relin(a[i], b[i]).data).all())
        assert bool((rot[i].data == w.ctx.rotate(a[i], 1).data).all())
