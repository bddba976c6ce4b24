"""GPU parity of small and middle-sized calls at the edges of their planning rules, bit for bit
against the CPU oracle: both sum each string's contributions in ascending H index, so equal
inputs give equal bits (tolerance 0)."""
import numpy as np
import pytest

import oracle
import workloads as wl
from helpers import assert_canonical_unique, gpu_available

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
    assert_canonical_unique(got)
    g, w = got.as_dict(), want.as_dict()
    assert set(g) == set(w), f"{what}: {len(set(w) - set(g))} missing, {len(set(g) - set(w))} extra"
    off = [k for k in w if g[k] != w[k]]
    assert not off, f"{what}: {len(off)} coefficients differ"


# tiles of 1024 strings shared out over H (up to 256 workgroups, at least 8 entries of H each),
# pruned to site windows above 32 tiles; 2^10, 2^12 and 2^14 bins (bounds of 2^18 and 2^22
# pairs), H indices kept aside above 127 and 511
@pytest.mark.parametrize("n,nh,no", [(12, 7, 1), (12, 16, 1), (30, 8, 1023), (64, 15, 1025),
                                     (40, 127, 2064), (40, 128, 2049), (64, 17, 32 * 1024),
                                     (64, 33, 32 * 1024 + 5), (100, 64, 3001), (70, 511, 600),
                                     (70, 512, 600), (64, 40, 104858), (64, 41, 104858)])
def test_tiles_shared_over_h(pk, n, nh, no):
    print(f"commutator n={n} nh={nh} no={no}", flush=True)
    H = wl.random_local_strings(n, nh, 3 if nh < 100 else 5, seed=nh)
    O = wl.random_local_strings(n, no, 12, seed=no)
    ws = pk.Workspace(256 << 20)
    tr = dict(max_len=14, max_strings=20000)
    got = pk.commutator(raw(pk, H), raw(pk, O), pk.Trunc(**tr), ws=ws).to_host()
    want = oracle.truncate(oracle.commutator(H, O), oracle.Trunc(**tr))
    same(got, want, "commutator")


@pytest.mark.parametrize("n,nh,no", [(12, 9, 1), (30, 17, 1025), (70, 24, 3001)])
def test_products_shared_over_h(pk, n, nh, no):
    print(f"product n={n} nh={nh} no={no}", flush=True)
    H = wl.random_operator(n, nh, seed=nh, density=0.2)
    O = wl.random_local_strings(n, no, 8, seed=no)
    ws = pk.Workspace(256 << 20)
    same(pk.multiply(raw(pk, H), raw(pk, O), ws=ws).to_host(), oracle.product(H, O), "product")


# powers of a chain: many pairs meet in one string, so the largest buckets are far above the mean
# (16-19: few buckets, 24: more than run at once, one pass), and the same size without long runs
@pytest.mark.parametrize("n", [16, 19, 24])
@pytest.mark.parametrize("runs", [True, False])
def test_products_with_long_runs(pk, n, runs):
    print(f"long runs n={n} runs={runs}", flush=True)
    H = wl.ising_chain(n, 0.5, 2.0)
    ws = pk.Workspace(1 << 30)
    A = pk.multiply(raw(pk, H), pk.multiply(raw(pk, H), raw(pk, H), ws=ws), ws=ws)
    if not runs:
        A = raw(pk, wl.random_operator(n, A.size, seed=n, density=0.7))
    same(pk.multiply(raw(pk, H), A, ws=ws).to_host(), oracle.product(H, A.to_host()), "product")


# minibatches that end inside a 32-row block, longer than the 256 rows whose mask is read ahead,
# and a workspace with no room for the transposed weights: the same bits as with it
@pytest.mark.parametrize("n,batch", [(31, 32), (300, 256), (700, 300), (513, 512)])
def test_training_without_transposed_weights(pk, n, batch):
    import torch
    from paper_2410_09654_amd import surrogate
    print(f"train n={n} batch={batch}", flush=True)
    g = torch.Generator().manual_seed(n)
    x = 1.0 + 0.2 * torch.randn((n, 16), generator=g)
    t = 1.0 + 0.2 * torch.randn((n, 16), generator=g)
    m = (torch.rand((n, 16), generator=g) < 0.7).float()
    nblk = (batch + 31) // 32
    least = -(-nblk * surrogate.param_offsets()[1] * 4 // 256) * 256 + -(-nblk * 16 // 256) * 256

    class Least:  # exactly the gradient shares and the loss shares
        def __init__(self):
            self.buf = torch.empty(least, dtype=torch.uint8, device="cuda")

        def c_struct(self):
            return pk._lib.PauliWsC(self.buf.data_ptr(), least, 0)

    nets = [surrogate.BnSurrogate(seed=1), surrogate.BnSurrogate(seed=1, ws=Least())]
    hist = [net.train(x, t, m, epochs=3, batch=batch, seed=2) for net in nets]
    assert hist[0] == hist[1]
    assert torch.equal(nets[0].params, nets[1].params)
    assert hist[0][-1] < hist[0][0]


# products whose operands are both read along k in 16-byte words (k in whole words), at the edges
# of a block's 64 rows and 64 columns and with k tails: the same bits as the kernel that takes any
# layout, which the same product with B laid out by rows goes to; k = 20 has no whole words
@pytest.mark.parametrize("M,N,K", [(16, 16, 8), (48, 80, 24), (64, 64, 32), (80, 48, 40),
                                   (112, 256, 256), (1040, 16, 264), (32, 32, 20)])
def test_gemm_along_k(pk, M, N, K):
    import torch
    from paper_2410_09654_amd import surrogate
    print(f"gemm along k {M}x{N}x{K}", flush=True)
    g = torch.Generator().manual_seed(M + N + K)
    A = torch.randn((M, K), generator=g).bfloat16().view(torch.int16).cuda()
    B = torch.randn((N, K), generator=g).bfloat16().view(torch.int16).cuda()
    got = surrogate.gemm_bf16(A, B, False, True)
    assert torch.equal(got, surrogate.gemm_bf16(A, B.t().contiguous(), False, False))
    exact = A.view(torch.bfloat16).double() @ B.view(torch.bfloat16).double().t()
    scale = A.view(torch.bfloat16).double().abs() @ B.view(torch.bfloat16).double().abs().t()
    assert bool(((got.double() - exact).abs() <= 2e-6 * scale).all())


# appended buckets of 2^F (bound of 2^(10 + F) records): filled to their room of 1408 one-word or
# 1344 two-word records, one above it, and above it but within the merge's 1984; every pair of
# the product with a single string is one record, half of the key range is left empty
@pytest.mark.parametrize("n,count", [(40, 1408), (40, 1409), (40, 1700), (100, 1344), (100, 1345)])
def test_appended_bucket_at_its_room(pk, n, count):
    print(f"append n={n} count={count}", flush=True)
    pool = wl.random_local_strings(n, 4 * count, 12, seed=count)
    one = wl.from_terms(n, [(1.0, [("X", 3)])])
    # strings whose product with X_3 has a key in the lower half
    x = pool.x.copy()
    x[:, 0] ^= np.uint64(4)
    moved = pk.order_keys(pk.PauliOp.from_raw(n, x, pool.z, pool.coef))[:, 0].cpu().numpy()
    pick = np.flatnonzero(moved >= 0)[:count]
    assert len(pick) == count
    O = wl.HostOp(n, pool.x[pick], pool.z[pick], pool.coef[pick])
    ws = pk.Workspace(256 << 20)
    got = pk.multiply(raw(pk, one), raw(pk, O), ws=ws).to_host()
    same(got, oracle.product(one, O), "product")
    room = 1408 if n <= 64 else 1344
    assert (pk.last_stats()["host_syncs"] == 1) == (count <= room)


# term runs found by one pass over the terms: no bucket bits (n <= 1033), empty buckets at both
# ends, terms of one string, and unsorted input (redone by emission)
@pytest.mark.parametrize("na,nb,shuffle", [(1, 1, False), (1, 1033, False), (700, 334, False),
                                           (40000, 3, False), (5, 600000, False),
                                           (3000, 2000, True)])
def test_add_streamed_bounds(pk, na, nb, shuffle):
    print(f"add na={na} nb={nb} shuffle={shuffle}", flush=True)
    A = wl.random_local_strings(50, na, 12, seed=1)
    B = wl.random_local_strings(50, nb, 12, seed=2)
    ws = pk.Workspace(256 << 20)
    dev = [raw(pk, h) if shuffle else pk.PauliOp.from_host(h, ws=ws) for h in (A, B)]
    got = pk.add(dev[0], 2.0 - 0.5j, dev[1], 0.25, ws=ws).to_host()
    same(got, oracle.add(A, 2.0 - 0.5j, B, 0.25), "add")


# groups of equal |c| around the 64 that one wave ranks, the 2048 that one block takes, and more
# (the multi-level select); the cut falls inside the group and is settled by the keys
@pytest.mark.parametrize("n", [24, 100])
@pytest.mark.parametrize("tied", [1, 64, 65, 1025, 2048, 2049])
def test_threshold_among_ties(pk, n, tied):
    print(f"ties n={n} tied={tied}", flush=True)
    O = wl.random_local_strings(n, 6000, 12, seed=tied)
    rng = np.random.default_rng(tied)
    mag = np.where(np.arange(6000) < tied, 1.0, 2.0 ** rng.integers(1, 4, 6000))
    mag[3000 + tied // 2:] = 2.0 ** -rng.integers(1, 9, 6000 - 3000 - tied // 2)
    phase = np.array([1, 1j, -1, -1j])[rng.integers(0, 4, 6000)]
    O = wl.HostOp(n, O.x, O.z, mag * phase)
    above = int((mag > 1.0).sum())
    ws = pk.Workspace(256 << 20)
    for cut in sorted({above + 1, above + (tied + 1) // 2, above + tied}):
        tr = dict(max_strings=cut)
        got = pk.truncate(pk.PauliOp.from_host(O, ws=ws), pk.Trunc(**tr), ws=ws).to_host()
        same(got, oracle.truncate(O, oracle.Trunc(**tr)), f"top {cut}")


# key search by interpolation: operators of 1 to 3 strings and more, members and others; 768
# results fit the pinned block, 769 do not; 131072 strings fill one round of the reductions
@pytest.mark.parametrize("n", [30, 90])
@pytest.mark.parametrize("na,nq", [(1, 3), (2, 5), (3, 768), (5000, 769), (131073, 2000)])
def test_lookups_and_reductions(pk, n, na, nq):
    print(f"lookups n={n} na={na} nq={nq}", flush=True)
    A = wl.random_local_strings(n, na, 12, seed=na)
    B = wl.random_local_strings(n, nq, 12, seed=nq + 1)
    k = min(na, nq // 2)  # half of Q's strings are A's
    Q = wl.HostOp(n, np.concatenate([A.x[:k], B.x[k:]]), np.concatenate([A.z[:k], B.z[k:]]),
                  B.coef)
    ws = pk.Workspace(64 << 20)
    dA = pk.PauliOp.from_host(A, ws=ws)
    assert np.array_equal(pk.coefficients(dA, raw(pk, Q), ws=ws), oracle.coefficients(A, Q))
    assert pk.norm2(dA, ws=ws) == oracle.norm2(A)
    dB = pk.PauliOp.from_host(oracle.canonicalize(Q), ws=ws)
    want = oracle.inner(A, oracle.canonicalize(Q))
    got = pk.inner(dA, dB, ws=ws)
    assert got == want
    s = pk.correlator(dA, dA, ws=ws)
    assert s == 1.0


def dyadic(h, seed):
    """The strings of h with small integer coefficients: every sum of products is exact, so any
    order of summation gives the same bits."""
    rng = np.random.default_rng(seed)
    c = rng.integers(1, 9, h.n) * rng.choice([1.0, -1.0], h.n) + 1j * rng.integers(-8, 9, h.n)
    return wl.HostOp(h.n_qubits, h.x, h.z, c)


# calls too large for one pass over 2^14 bins, binned over 2^15 or (more than 55 M one-word or
# 37 M two-word records expected) 2^17 at once, against the sum of the same call on quarters of O
# (each within 2^14 bins); the last case puts 400 records of one string into one workgroup's bin,
# more than a byte counts, and goes back to the partitions
@pytest.mark.parametrize("n,chain,count,dtype,crowd", [(64, "ising", 2500003, 0, 0),
                                                       (64, "ising", 3700003, 0, 0),
                                                       (100, "xxz", 1200001, 1, 0),
                                                       (100, "xxz", 1900001, 0, 0),
                                                       (100, "xxz", 1900001, 1, 0),
                                                       (48, "random", 640000, 0, 400)])
def test_one_pass_over_wide_bins(pk, n, chain, count, dtype, crowd):
    print(f"wide bins n={n} {chain} count={count} dtype={dtype} crowd={crowd}", flush=True)
    O = wl.random_local_strings(n, count, 13, seed=count)
    if crowd:
        H, P = wl.same_key_runs(n, np.ones(crowd))
        keep = ~np.isin(O.x[:, 0] ^ (O.z[:, 0] << np.uint64(1)), P.x[:, 0] ^ (P.z[:, 0] << np.uint64(1)))
        O = wl.HostOp(n, np.concatenate([P.x, O.x[keep]]), np.concatenate([P.z, O.z[keep]]),
                      np.concatenate([P.coef, O.coef[keep]]))
    else:
        H = wl.ising_chain(n, 0.5, 2.0) if chain == "ising" else wl.xxz_random_field(n, 0.5, 0.0)[0]
        H = wl.HostOp(n, H.x[H.coef != 0], H.z[H.coef != 0], H.coef[H.coef != 0])
    H = wl.HostOp(n, H.x, H.z, np.where(np.arange(H.n) % 3, 0.5, 2.0))
    O = dyadic(O, 7)
    assert H.n * O.n > 7 * (1 << 14) * (1984 if n <= 64 else 1344)
    ws = pk.Workspace(1 << 30)
    dH = raw(pk, H)
    got = pk.commutator(dH, raw(pk, O, dtype), ws=ws)
    stats = pk.last_stats()
    assert stats["passes"] == 1 or crowd
    q = -(-O.n // 4)
    total = None
    for k in range(4):
        part = wl.HostOp(n, O.x[k * q:(k + 1) * q], O.z[k * q:(k + 1) * q], O.coef[k * q:(k + 1) * q])
        c = pk.commutator(dH, raw(pk, part, dtype), ws=ws)
        total = c if total is None else pk.add(total, 1.0, c, 1.0, ws=ws)
    m = got.size
    assert m == total.size
    import torch
    assert torch.equal(got.x[:, :m], total.x[:, :m]) and torch.equal(got.z[:, :m], total.z[:, :m])
    assert torch.equal(got.coef[:m], total.coef[:m])
