"""The key switch's inner product on every kind of limb at N = 2^16, against the oracle, bit for bit: ciphertext and
special primes on either arithmetic path (the dropped limb of a rescale among them), digit counts on both sides of a
round of four, digits shared by several rotations and digits of one, results that overlap a factor of a Mult."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

_Q50 = tuple(2**50 - d for d in (3014655, 4718591, 19529727))
_Q55 = tuple(2**55 - d for d in (4587519, 5636095, 8519679))
SETS = {
    # 55- and 50-bit ciphertext primes in turn, one special prime on the integer path, six digits
    "mixed": wl.Params("mixed", 16, tuple(v for pair in zip(_Q55, _Q50) for v in pair), (2**60 - 262143,), 6),
    # 40-bit ciphertext primes, the special prime on the floating-point path, five digits
    "float": wl.Params("float", 16, tuple(2**40 - d for d in (1572863, 3932159, 5111807, 7077887, 7733247)), (2**50 - 3014655,), 5),
}


@pytest.fixture(scope="module", params=sorted(SETS))
def env(request, oracle_mod):
    import paper_2210_02574_amd as pkg

    p = SETS[request.param]
    he, o = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum)
    evk = wl.uniform_evk(7, p)
    return he, o, p, evk


@pytest.mark.parametrize("level", [1, 4, 5, 6])
def test_rotations(env, level):
    he, o, p, evk = env
    level = min(level, p.L)
    ct = wl.uniform_ct(20 + level, p, level)
    shifts = [1, 3, -2]
    keys = [he.evk_from_host(evk, he.galois_element(r)) for r in shifts]
    want = [o.hrot(ct, evk, r) for r in shifts]
    d = he.to_device(ct)
    assert np.array_equal(he.to_host(he.hrot(keys[0], d)), want[0])
    for got, w in zip(he.hrot_many(keys, d), want):
        assert np.array_equal(he.to_host(got), w)


@pytest.mark.parametrize("level", [2, 5, 6])
def test_mult(env, level):
    he, o, p, evk = env
    level, count = min(level, p.L), 2
    key = he.evk_from_host(evk, 1)
    a, b = [np.stack([wl.uniform_ct(40 + 10 * k + level + o_, p, level) for o_ in range(count)]) for k in range(2)]
    prod = [o.hmult_relin(x, y, evk) for x, y in zip(a, b)]
    resc = [o.rescale(x) for x in prod]
    da, db = he.to_device(a), he.to_device(b)
    assert np.array_equal(he.to_host(he.hmult_relin_batch(key, da, db)), np.stack(prod))
    assert np.array_equal(he.to_host(he.hmult_relin_rescale_batch(key, da, db)), np.stack(resc))
    # results in the place of a factor, of the other, and of a square's only one
    short = p.N * 2 * (level - 1) * count
    for which in (0, 1):
        f = [he.to_device(a), he.to_device(b)]
        he.hmult_relin_batch(key, f[0], f[1], out=f[which])
        assert np.array_equal(he.to_host(f[which]), np.stack(prod)), which
        f = [he.to_device(a), he.to_device(b)]
        out = f[which].view(-1)[:short].view(count, 2, level - 1, p.N)
        he.hmult_relin_rescale_batch(key, f[0], f[1], out=out)
        assert np.array_equal(he.to_host(out), np.stack(resc)), which
    sq = he.to_device(a)
    he.hmult_relin_batch(key, sq, sq, out=sq)
    assert np.array_equal(he.to_host(sq), np.stack([o.hmult_relin(x, x, evk) for x in a]))
