"""GPU calls that leave the route first planned for them, or sit at the edge of a rule that picks
one: against the CPU oracle or the same sum computed in parts, bit for bit (coefficients are small
integers or halves, so every sum is exact in any order)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from helpers import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def pk():
    import paper_2410_09654_amd as pk
    pk._lib.load()
    return pk


def raw(pk, h, dtype=0):
    return pk.PauliOp.from_raw(h.n_qubits, h.x, h.z, h.coef, dtype=dtype)


def same(got, want, what):
    g, w = got.as_dict(), want.as_dict()
    assert len(g) == got.n, f"{what}: strings repeat"
    assert set(g) == set(w), f"{what}: {len(set(w) - set(g))} missing, {len(set(g) - set(w))} extra"
    off = [k for k in w if g[k] != w[k]]
    assert not off, f"{what}: {len(off)} coefficients differ"


def small_ints(n, x, z, seed):
    rng = np.random.default_rng(seed)
    c = rng.integers(1, 9, len(x)) * rng.choice([1.0, -1.0], len(x))
    return wl.HostOp(n, np.asarray(x, np.uint64).reshape(-1, 1),
                     np.asarray(z, np.uint64).reshape(-1, 1), c.astype(complex))


def ring(n):
    """Representative of every string of an n-site ring, as (x << n | z) -> (x << n | z)."""
    rot = lambda v, r: ((v >> r) | (v << (n - r))) & ((1 << n) - 1)
    rep = np.zeros(4 ** n, np.int64)
    for s in range(4 ** n):
        x, z = s >> n, s & ((1 << n) - 1)
        _, rx, rz = min((rot(x | z, r), rot(x, r), rot(z, r)) for r in range(n))
        rep[s] = rx << n | rz
    return rep


def ring_operands(pk, n, nh):
    """H0 and O of a dense ring: O all representatives but the identity, H0 the nh of them whose
    translates make most records of the fullest of the 2^8 key ranges."""
    rep = ring(n)
    reps = np.unique(rep)
    reps = reps[reps > 0]
    m = (1 << n) - 1
    every = np.arange(4 ** n)
    keys = pk.order_keys(pk.PauliOp.from_raw(n, (every >> n).astype(np.uint64).reshape(-1, 1),
                                             (every & m).astype(np.uint64).reshape(-1, 1),
                                             np.ones(4 ** n)))
    bucket = (keys[:, 0].cpu().numpy().view(np.uint64) >> np.uint64(56)).astype(np.int64)
    rot = lambda v, r: ((v >> r) | (v << (n - r))) & m
    count = np.zeros((len(reps), 256), np.int64)
    for i, h in enumerate(reps):
        for r in range(n):
            hx, hz = rot(int(h) >> n, r), rot(int(h) & m, r)
            ox, oz = reps >> n, reps & m
            anti = (np.bitwise_count(hx & oz) + np.bitwise_count(hz & ox)) & 1 == 1
            p = rep[((ox ^ hx) << n | (oz ^ hz))[anti]]
            count[i] += np.bincount(bucket[p], minlength=256)
    b = count.sum(0).argmax()
    pick = np.sort(np.argsort(-count[:, b], kind="stable")[:nh])
    H0, O = reps[pick], reps
    return (small_ints(n, H0 >> n, H0 & m, n), small_ints(n, O >> n, O & m, n + 1),
            int(count[pick].sum(0).max()))


# a translation-symmetric call of at most 2^18 possible records whose fullest bucket overflows is
# redone with its count read first: H0 has to be expanded over its translations once, not twice
# (200 x 5 strings twice over are more than a bucket holds, 46 x 6 are not)
@pytest.mark.parametrize("n,nh", [(5, 200), (6, 46)])
def test_crowded_symmetric_call(pk, n, nh):
    H0, O, fullest = ring_operands(pk, n, nh)
    print(f"ring n={n} |H0|={nh} |O|={O.n} fullest bucket {fullest}", flush=True)
    assert nh * n * O.n + O.n <= 1 << 18 and 1408 < fullest
    ws = pk.Workspace(256 << 20)
    dH, dO = raw(pk, H0), raw(pk, O)
    got = pk.commutator_ts1d(dH, dO, ws=ws)
    assert pk.last_stats()["host_syncs"] == 2  # the redone call reads its count
    same(got.to_host(), oracle.commutator_ts(H0, O), "commutator")
    prev = oracle.canonicalize(small_ints(n, O.x[::3], O.z[::3], n + 2))
    want, b, _ = oracle.lanczos_step_ts(H0, prev, O, 0.5)
    got, bg, broke = pk.lanczos_step(dH, raw(pk, prev), dO, 0.5, ws=ws, ts1d=True)
    assert pk.last_stats()["host_syncs"] == 2
    assert not broke and bg == b
    same(got.to_host(), want, "Lanczos step")
