"""The plaintext and encrypted-weight dot products (k_pt_dot_multi_b,
k_ct_dot_multi_b) at the edges of their item groups, term folds and output
groups, on a chain with 60-bit and 40-bit rows; bit-exact against the oracle."""

import numpy as np
import pytest

import synth as S
from oracle import ckks as C
from oracle import training as T

from .test_gpu_modup_fused import CASES, World, world

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("docs,terms,outs", [(1, 1, 1), (2, 8, 9), (3, 9, 3), (5, 17, 8), (4, 16, 17)])
def test_plaintext_dot(docs, terms, outs):
    w = world("a2_n12")
    level, bound = 3, 2 ** 30
    coeffs = np.stack([np.stack([S.plaintext_coeffs(S.rng(7000 + 100 * k + j), w.n, bound) for j in range(terms)])
                       for k in range(outs)])
    mat = w.ctx.ptdot_from_coeffs(coeffs, level, 2.0 ** 30)
    cts = [[w.enc_pair(900 + 20 * d + j, level) for j in range(terms)] for d in range(docs)]
    got = w.ctx.ptdot_apply(mat, [[c[0] for c in doc] for doc in cts])
    for d, doc in enumerate(cts):
        for k in range(outs):
            o = None
            for j, (_, x) in enumerate(doc):
                t = C.hmul_plain(w.op, x, coeffs[k, j], 2.0 ** 30)
                o = t if o is None else C.hadd(w.op, o, t)
            w.assert_same(got[d][k], o)


def test_encrypted_dot_groups():
    """Documents alone, in a pair and in a group with a remainder give the
    same products (one document is pinned to the oracle elsewhere)."""
    spec = dict(CASES["a2_n14"], log_n=12)
    w = World(spec)
    n_o, n_i, level = 4, 16, 4
    w.ctx.keygen(31, [1, 2, 4, 8])
    b, G = 2, 2
    diags = [w.enc_pair(40 + i, level)[0] for i in range(b * G)]
    docs = [[w.ctx.encrypt_seeded(S.plaintext_coeffs(S.rng(60 + d), w.n, 2 ** 30), level, w.op.scale, 700 + d)]
            for d in range(3)]
    one = [w.ctx.export(w.ctx.ctmatvec(diags, n_o, n_i, 1, [d])[0]) for d in docs]
    for n in (2, 3):
        for a, g in zip(one, w.ctx.ctmatvec(diags, n_o, n_i, 1, docs[:n])):
            assert np.array_equal(a, w.ctx.export(g))


@pytest.mark.parametrize("n_o,n_i", [(1, 2), (2, 2)])
@pytest.mark.parametrize("docs", [1, 2, 3])
def test_encrypted_dot_of_one_giant_step(n_o, n_i, docs):
    w, level = world("a2_n12"), 4
    diags = [w.enc_pair(80 + i, level) for i in range(n_o)]
    ins = [w.enc_pair(90 + d, level) for d in range(docs)]
    got = w.ctx.ctmatvec([g for g, _ in diags], n_o, n_i, 1, [[g] for g, _ in ins])
    for g, (_, x) in zip(got, ins):
        w.assert_same(g, T.ctmatvec(w.op, [x], [[[o for _, o in diags]]], n_o, n_i, w.rlk, w.rot))
