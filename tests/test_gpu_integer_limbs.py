"""Ciphertext primes of 2^50 and above (the integer path of the device kernels) at every ring size, alone and in turn with
smaller ones, through every form of the key switch: rotations one by one, hoisted, summed, with keys and levels of their
own, with both kinds of base conversion, and products whose result lies over a factor.  Against the oracle, bit for bit."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

_A16 = tuple(2**55 - d for d in (4587519, 5636095, 8519679))  # = 1 mod 2^17
_B16 = tuple(2**50 - d for d in (3014655, 4718591, 19529727))
_P16 = tuple(2**60 - d for d in (262143, 8126463))
_A17 = tuple(2**55 - d for d in (13107199, 17825791))  # = 1 mod 2^18
_B17 = tuple(2**50 - d for d in (4718591, 20447231))
_P17 = tuple(2**60 - d for d in (262143, 8126463))


def _alternate(a, b):
    return tuple(v for pair in zip(a, b) for v in pair)


SETS = {
    "M12": wl.M12,
    "I12": wl.I12,
    # digits of two primes, one on either path; five limbs leave the last digit partial
    "mixed16": wl.Params("mixed16", 16, _alternate(_A16, _B16), _P16, 3),
    "int16": wl.Params("int16", 16, _A16, _P16, 2),
    "mixed17": wl.Params("mixed17", 17, _alternate(_A17, _B17), _P17, 2),
}


@pytest.fixture(scope="module", params=[(n, ex) for n in SETS for ex in (False, True)], ids=lambda v: v[0] + ("-corrected" if v[1] else ""))
def env(request, oracle_mod):
    import paper_2210_02574_amd as pkg

    name, exact = request.param
    p = SETS[name]
    he, o = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum)
    he.set_exact_conversion(exact)
    o.set_exact(exact)
    yield he, o, p, wl.uniform_evk(9, p)
    o.set_exact(False)


def _levels(p):
    return [p.L, p.L - 1, 1]


def test_rotations_of_one_level(env):
    import torch

    he, o, p, evk = env
    shifts = [1, 6]
    keys = [he.evk_from_host(evk, he.galois_element(r)) for r in shifts]
    for level in _levels(p):
        cts = [wl.uniform_ct(30 + 3 * level + k, p, level) for k in range(2)]
        d = [he.to_device(c) for c in cts]
        want = [o.hrot(cts[0], evk, r) for r in shifts]
        assert np.array_equal(he.to_host(he.hrot(keys[0], d[0])), want[0]), level
        for got, w in zip(he.hrot_many(keys, d[0]), want):
            assert np.array_equal(he.to_host(got), w), level
        both = he.hrot_batch_keys(keys, torch.stack(d))
        assert np.array_equal(he.to_host(both[0]), want[0]), level
        assert np.array_equal(he.to_host(both[1]), o.hrot(cts[1], evk, shifts[1])), level
    doubling = [he.evk_from_host(evk, he.galois_element(r)) for r in (2, 4, 8)]
    for n_rot in (2, 3):  # the result ends in the caller's buffer, or in the workspace and is copied
        sums = torch.stack(d)
        he.rotate_sum_batch(doubling[:n_rot], sums)
        for k in range(2):
            assert np.array_equal(he.to_host(sums[k]), o.rotate_sum(cts[k], [evk] * n_rot, 2)), (level, n_rot, k)


def test_rotations_of_mixed_levels(env):
    import torch

    he, o, p, evk = env
    levels, shifts = [2, p.L, p.L, 1, p.L - 1], [1, 1, 6, 6, 3]
    keys = {r: he.evk_from_host(evk, he.galois_element(r)) for r in set(shifts)}
    cts = [wl.uniform_ct(60 + k, p, lv) for k, lv in enumerate(levels)]
    packed = torch.cat([he.to_device(c).reshape(-1, p.N) for c in cts])
    got = he.to_host(he.hrot_batch_levels([keys[r] for r in shifts], levels, packed))
    at = 0
    for lv, r, ct in zip(levels, shifts, cts):
        assert np.array_equal(got[at:at + 2 * lv].reshape(2, lv, p.N), o.hrot(ct, evk, r)), (lv, r)
        at += 2 * lv


def test_products_over_their_factors(env):
    """Results in fresh memory, in a factor's place, from the start of a factor on, and across the end of the first factor
    into the second."""
    import torch

    he, o, p, evk = env
    key = he.evk_from_host(evk, 1)
    count = 2
    for level in _levels(p)[:2]:
        a, b = [np.stack([wl.uniform_ct(80 + 10 * k + level + i, p, level) for i in range(count)]) for k in range(2)]
        prod = np.stack([o.hmult_relin(x, y, evk) for x, y in zip(a, b)])
        resc = np.stack([o.rescale(x) for x in prod])
        words = a.size
        both = torch.empty(2 * words, dtype=torch.int64, device="cuda:0")
        fa, fb = both[:words].view(a.shape), both[words:].view(b.shape)

        def factors():
            fa.copy_(he.to_device(a))
            fb.copy_(he.to_device(b))

        factors()
        assert np.array_equal(he.to_host(he.hmult_relin_batch(key, fa, fb)), prod), level
        assert np.array_equal(he.to_host(he.hmult_relin_rescale_batch(key, fa, fb)), resc), level
        for first in (0, p.N, words // 2, words):  # words before the result
            factors()
            out = both[first:first + resc.size].view(resc.shape)
            he.hmult_relin_rescale_batch(key, fa, fb, out=out)
            assert np.array_equal(he.to_host(out), resc), (level, first)
        for f in (fa, fb):
            factors()
            he.hmult_relin_batch(key, fa, fb, out=f)
            assert np.array_equal(he.to_host(f), prod), level


# name -> (parameters, levels, counts, levels whose digits are finished ahead in the larger count's products with rescale): launches of the special
# limbs on both sides of the 1024 work-groups from which one or two digits are finished ahead (64 per limb and operation at N = 2^16); three keep three
# of the four waves busy and are not
BATCHES = {
    "N16": (wl.N16, (4, 7), (3, 4), (4, 7)),
    "mixed16": (SETS["mixed16"], (3, 4, 5, 6), (5, 8), (3, 4)),  # a dropped limb on either path
    "float16": (wl.Params("float16", 16, wl.N16.q[:3], (wl.N16.q[3],), 3), (3,), (16,), ()),  # no special limb on the integer path
}


@pytest.mark.parametrize("name", BATCHES)
def test_special_limbs_of_small_and_large_launches(oracle_mod, name):
    import torch

    import paper_2210_02574_amd as pkg

    p, levels, counts, ahead = BATCHES[name]
    he, o, evk = pkg.HE.from_params(p, device=0), oracle_mod.Oracle(p.logN, p.q, p.p, p.dnum), wl.uniform_evk(9, p)
    relin, rot = he.evk_from_host(evk, 1), he.evk_from_host(evk, he.galois_element(3))
    for level in levels:
        host = [wl.uniform_ct(200 + 20 * level + i, p, level) for i in range(max(counts))]
        dev = torch.stack([he.to_device(c) for c in host])
        rotated = [o.hrot(c, evk, 3) for c in host]
        products = [o.rescale(o.hmult_relin(host[i], host[i - 1], evk)) for i in range(len(host))]
        for count in counts:
            got = he.to_host(he.hrot_batch(rot, dev[:count]))
            assert all(np.array_equal(got[i], rotated[i]) for i in range(count)), (level, count)
            shifted = torch.roll(dev, 1, 0)[:count].contiguous()
            he.profile_start()
            got = he.to_host(he.hmult_relin_rescale_batch(relin, dev[:count], shifted))
            assert ("k_inner_finished" in he.profile_stop()) == (count == counts[-1] and level in ahead), (level, count)
            assert all(np.array_equal(got[i], products[i]) for i in range(count)), (level, count)
        for count in (2, 3):  # shared digits
            for got in he.hrot_many([rot] * count, dev[0]):
                assert np.array_equal(he.to_host(got), rotated[0]), (level, count)


# launches of up to 1280 work-groups of a rescale's last pass (40 limbs at N = 2^16, 20 at 2^17) and larger ones, on either arithmetic path
@pytest.mark.parametrize("params,level,count", [(wl.N16, 21, 1), (wl.N16, 22, 1), (SETS["mixed16"], 6, 4), (SETS["mixed16"], 6, 5), (wl.P17, 11, 1), (wl.P17, 12, 1)],
                         ids=lambda v: getattr(v, "name", v))
def test_rescales_of_small_and_large_launches(oracle_mod, params, level, count):
    import paper_2210_02574_amd as pkg

    he, o = pkg.HE.from_params(params, device=0), oracle_mod.Oracle(params.logN, params.q, params.p, params.dnum)
    cts = np.stack([wl.uniform_ct(350 + i, params, level) for i in range(count)])
    cts[0, 0] = np.array(params.q[:level], dtype=np.uint64)[:, None] - 1  # the largest residues
    got = he.to_host(he.rescale_batch(he.to_device(cts)))
    assert all(np.array_equal(got[i], o.rescale(cts[i])) for i in range(count))


def test_product_over_a_factor_in_a_graph():
    """The copy that such a result takes can be captured: three replays with eager work in between."""
    import torch

    import paper_2210_02574_amd as pkg

    p = SETS["int16"]
    he = pkg.HE.from_params(p, device=0)
    relin = he.evk_from_host(wl.uniform_evk(9, p), 1)
    a, b = [he.to_device(wl.uniform_ct(300 + k, p, p.L)) for k in range(2)]
    want = he.hmult_relin_rescale(relin, a, b)
    work = a.clone()
    out = work.view(-1)[: want.numel()].view(want.shape)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        he.hmult_relin_rescale(relin, work, b, out=out)  # the workspace of the capture stream exists before the capture starts
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        he.hmult_relin_rescale(relin, work, b, out=out)
    for replay in range(3):
        work.copy_(a)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), replay
        assert torch.equal(he.hmult_relin_rescale(relin, a, b), want)
