"""Base conversions of the key switch at N = 2^16 and 2^17 against the oracle, bit for bit: digits of one to eight limbs and a last digit
that is shorter, special primes on either arithmetic path, operations of several levels in one launch, one operation (its targets
shared out among several work-groups) and a few, uniform residues and the largest ones."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

SETS = {
    "three16": wl.Params("three16", 16, wl.N16.q[:7], wl.N16.p[:2], 3),  # digits of 3, 3, 1
    "two16": wl.Params("two16", 16, wl.N16.q[:6], wl.N16.q[10:13], 3),  # special primes below 2^50
    "one16": wl.Params("one16", 16, wl.N16.q[:3], (wl.N16.p[0],), 3),  # digits of 1
    "five16": wl.Params("five16", 16, wl.N16.q[:9], wl.W16.p, 2),  # digits of 5, 4; five special primes
    "eight16": wl.Params("eight16", 16, wl.N16.q[:8], wl.N16.p + wl.N16.q[10:14], 1),  # one digit of 8, special primes of both kinds
    "four17": wl.Params("four17", 17, wl.P17.q[:6], wl.P17.p[:3], 2),  # digits of 3, 3
    "mixed17": wl.Params("mixed17", 17, wl.P17.q[:5], (wl.P17.p[0], wl.P17.q[9]), 2),  # special primes of both kinds
}


@pytest.fixture(scope="module", params=sorted(SETS))
def env(request, oracle_mod):
    import paper_2210_02574_amd as pkg

    p = SETS[request.param]
    he, o = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum)
    return he, o, p, wl.uniform_evk(11, p)


def _largest(p, level):
    """Every NTT value of both components is q - 1."""
    return np.stack([np.stack([np.full(p.N, p.q[i] - 1, dtype=np.uint64) for i in range(level)])] * 2)


def test_rotations_of_every_level(env):
    he, o, p, evk = env
    key = he.evk_from_host(evk, he.galois_element(3))
    levels = list(range(1, p.L + 1))
    cts = [wl.uniform_ct(60 + lv, p, lv) for lv in levels]
    want = [o.hrot(ct, evk, 3) for ct in cts]
    for ct, w in zip(cts, want):
        assert np.array_equal(he.to_host(he.hrot(key, he.to_device(ct))), w)
    # in one launch, the buffers laid out for the largest level
    packed = he.to_device(np.concatenate([ct.reshape(-1, p.N) for ct in cts]))
    got = he.to_host(he.hrot_batch_levels([key] * len(levels), levels, packed))
    assert np.array_equal(got, np.concatenate([w.reshape(-1, p.N) for w in want]))


def test_products(env):
    he, o, p, evk = env
    key, count = he.evk_from_host(evk, 1), 3
    for level in (2, p.L):
        a = np.stack([wl.uniform_ct(80 + level, p, level), _largest(p, level), wl.uniform_ct(81 + level, p, level)])
        b = np.stack([wl.uniform_ct(90 + level, p, level), _largest(p, level), a[2]])
        prod = [o.hmult_relin(x, y, evk) for x, y in zip(a, b)]
        da, db = he.to_device(a), he.to_device(b)
        assert np.array_equal(he.to_host(he.hmult_relin_batch(key, da, db)), np.stack(prod))
        resc = np.stack([o.rescale(x) for x in prod])
        assert np.array_equal(he.to_host(he.hmult_relin_rescale_batch(key, da, db)), resc)
        for i in range(count):
            assert np.array_equal(he.to_host(he.hmult_relin_rescale(key, da[i], db[i])), resc[i])


@pytest.mark.parametrize("params", ["N16", "P17"])
def test_buffers_that_start_at_an_odd_word(params, oracle_mod):
    """Transforms and rescales take buffers aligned to words, not to the 16 bytes that a pair of them has."""
    import torch

    import paper_2210_02574_amd as pkg

    p = getattr(wl, params)
    he, o = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum)

    def odd(x):
        t = he.to_device(np.concatenate([np.zeros(1, dtype=np.uint64), x.reshape(-1)]))[1:].view(x.shape)
        assert t.data_ptr() % 16 == 8 and t.is_contiguous()
        return t

    mods = [0, p.L]  # one limb on either arithmetic path
    x = np.stack([wl.rng(5).integers(0, p.moduli[i], size=p.N, dtype=np.uint64) for i in mods])
    want = o.ntt(x, mods)
    d = odd(x)
    assert np.array_equal(he.to_host(he.ntt(d, mods)), want)
    assert np.array_equal(he.to_host(he.intt(d, mods)), x)
    ct = wl.uniform_ct(6, p, 3)
    out = torch.zeros(2 * 2 * p.N + 1, dtype=torch.int64, device="cuda:0")[1:].view(2, 2, p.N)
    assert np.array_equal(he.to_host(he.rescale(odd(ct), out=out)), o.rescale(ct))


def test_more_digits_than_unreduced_sums_hold(oracle_mod):
    """29 digits: the special limb's 128-bit sums of values below 8q are folded on the way (28 and fewer fit)."""
    import paper_2210_02574_amd as pkg

    p = wl.Params("many16", 16, wl.P17.q[:29], (wl.P17.p[0],), 29)
    he, o = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum)
    evk = wl.uniform_evk(12, p)
    key = he.evk_from_host(evk, he.galois_element(5))
    for level in (28, 29):
        ct = wl.uniform_ct(40 + level, p, level)
        assert np.array_equal(he.to_host(he.hrot(key, he.to_device(ct))), o.hrot(ct, evk, 5))


# name -> (parameters, levels of the operations of one call, whether the inverse column passes run apart from the conversions)
_ONES16 = wl.Params("ones16", 16, wl.N16.q[:5], wl.N16.p[:1], 5)  # digits of 1, one special prime
FORMS = {
    "few targets on average": (wl.W16, [12] + [2] * 15, True),  # by its largest level it would have many
    "many targets on average": (wl.W16, [12] * 8 + [2], False),
    "wide digits": (wl.W16, [5] * 8, True),
    "one source": (_ONES16, [5] * 16, True),
    "one source, one round": (_ONES16, [1] * 4, False),
}


@pytest.mark.parametrize("name", FORMS)
def test_batches_in_either_form(name, oracle_mod):
    import torch

    import paper_2210_02574_amd as pkg

    p, levels, apart = FORMS[name]
    he, o, evk = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum), wl.uniform_evk(13, p)
    key, relin = he.evk_from_host(evk, he.galois_element(3)), he.evk_from_host(evk, 1)
    cts = {lv: [wl.uniform_ct(70 + 2 * lv + k, p, lv) for k in range(2)] for lv in set(levels)}
    want = {lv: [o.hrot(ct, evk, 3) for ct in pair] for lv, pair in cts.items()}
    packed = he.to_device(np.concatenate([cts[lv][i % 2].reshape(-1, p.N) for i, lv in enumerate(levels)]))
    he.profile_start()
    got = he.to_host(he.hrot_batch_levels([key] * len(levels), levels, packed))
    assert ("k_ntt_inv_cols" in he.profile_stop()) == apart
    assert np.array_equal(got, np.concatenate([want[lv][i % 2].reshape(-1, p.N) for i, lv in enumerate(levels)]))
    lv = levels[0]
    if set(levels) != {lv} or lv < 2:
        return
    a = np.stack([cts[lv][i % 2] for i in range(len(levels))])
    da, db = he.to_device(a), torch.roll(he.to_device(a), 1, 0).contiguous()
    assert np.array_equal(he.to_host(he.hrot_batch(key, da)), np.stack([want[lv][i % 2] for i in range(len(levels))]))
    prod = o.hmult_relin(cts[lv][0], cts[lv][1], evk)
    got = he.to_host(he.hmult_relin_batch(relin, da, db))
    assert all(np.array_equal(g, prod) for g in got)
    got, resc = he.to_host(he.hmult_relin_rescale_batch(relin, da, db)), o.rescale(prod)
    assert all(np.array_equal(g, resc) for g in got)
