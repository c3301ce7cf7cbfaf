"""LSD and global OSD at the edges of their shapes: numbers of faults and of checks around the
64-bit words of the bases and fault sets, more flipped checks than a wavefront has lanes, dependent
checks (syndromes outside the image), ties, NaN and empty syndromes.  Every result is a whole
number and equals the oracle's."""
import numpy as np
import pytest

from paper_2406_18655_amd import binding

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()


def _graph(m, n, seed):
    """Columns of weight 1 to 6; the last check repeats the first, the two before it share their faults."""
    rng = np.random.default_rng(seed)
    H = np.zeros((m, n), dtype=np.uint8)
    for j in range(n):
        H[rng.choice(m - 3, size=min(m - 3, int(rng.choice([1, 2, 3, 4, 6], p=[.05, .25, .45, .2, .05]))),
                     replace=False), j] = 1
    for i in np.nonzero(H[:m - 3].sum(1) < 2)[0]:
        H[i, rng.choice(np.nonzero(H[i] == 0)[0], size=2, replace=False)] = 1
    H[m - 3, rng.choice(n, size=3, replace=False)] = 1
    H[m - 2] = H[m - 3]
    H[m - 1] = H[0]
    return H


def _shots(H, seed, dense):
    """Sparse and dense errors, syndromes outside the image, soft information with and without ties."""
    rng = np.random.default_rng(seed)
    m, n = H.shape
    rates = np.repeat([0.01, 0.03, 0.1, 0.3], 16)
    E = (rng.random((len(rates), n)) < rates[:, None]).astype(np.int64)
    S = (E @ H.T % 2).astype(np.uint8)
    off = S[::4].copy()
    off[np.arange(len(off)), rng.integers(m, size=len(off))] ^= 1
    S = np.concatenate([S, off, np.zeros((2, m), np.uint8), np.ones((2, m), np.uint8),
                        (rng.random((dense, m)) < 0.5).astype(np.uint8)])
    L = (rng.normal(2.0, 2.0, size=(len(S), n))).astype(np.float32)
    L[::3] = np.rint(L[::3] / 2)
    L[1::9, ::4] = -0.0
    return np.ascontiguousarray(S), np.ascontiguousarray(L)


@pytest.mark.parametrize("m,n", [(8, 16), (24, 63), (63, 64), (64, 65), (65, 128), (64, 192), (100, 129),
                                 (127, 191), (128, 192), (128, 193), (129, 192)])
def test_lsd_of_small_graphs(oracle_mod, m, n):
    print(f"case lsd_shapes lsd {m}x{n}", flush=True)
    H = _graph(m, n, seed=m + n)
    S, L = _shots(H, seed=m * n, dense=16)
    bc = binding.Code.from_dense(H)
    dec = binding.Decoder(bc, np.full(n, 0.02), len(S), max_iter=5)
    L[5, n - 1] = np.nan
    corr, info, st = dec.lsd_stats(torch.from_numpy(S).cuda(), torch.from_numpy(L).cuda())
    plain, pinfo = dec.lsd(torch.from_numpy(S).cuda(), torch.from_numpy(L).cuda())
    torch.cuda.synchronize()
    assert torch.equal(plain, corr) and torch.equal(pinfo, info)
    c, st, inf = corr.cpu().numpy(), st.cpu().numpy(), binding.parse_info(info)
    oc = oracle_mod.Code.from_dense(H)
    assert inf["status"][5] & binding.ST_BAD_LLR and not c[5].any()
    unsat = 0
    for b in range(len(S)):
        if b == 5:
            continue
        want, ost, stats = oracle_mod.lsd(oc, S[b], L[b].astype(np.float64))
        assert not inf["status"][b] & (binding.ST_OVERFLOW | binding.ST_BAD_LLR), b
        assert (c[b] == want).all(), b
        assert bool(inf["status"][b] & binding.ST_UNSAT) == bool(ost & oracle_mod.ST_UNSAT), b
        assert (inf["n_clusters"][b], inf["max_cluster_cols"][b]) == tuple(stats[:2]), b
        # the oracle also counts a last round in which the clusters only find no fault left
        assert stats[2] - inf["rounds"][b] in ((0, 1) if ost & oracle_mod.ST_UNSAT else (0,)), b
        assert tuple(st[b]) == (stats[0], stats[1], stats[3], stats[6]), b
        unsat += bool(ost & oracle_mod.ST_UNSAT)
    assert unsat


@pytest.mark.parametrize("m,n", [(8, 16), (64, 64), (64, 65), (65, 128), (128, 129), (96, 192), (129, 193),
                                 (192, 256), (193, 257), (255, 300)])
def test_osd_of_every_word_count(oracle_mod, m, n):
    print(f"case lsd_shapes osd {m}x{n}", flush=True)
    H = _graph(m, n, seed=m + 2 * n)
    S, L = _shots(H, seed=m * n + 1, dense=4)
    bc = binding.Code.from_dense(H)
    priors = np.random.default_rng(3).uniform(0.005, 0.1, size=n)
    dec = binding.Decoder(bc, priors, len(S), max_iter=5)
    s, l = torch.from_numpy(S).cuda(), torch.from_numpy(L).cuda()
    c0, i0 = dec.osd0(s, l)
    order = 7
    cs, ics = dec.osd_cs(s, l, order)
    torch.cuda.synchronize()
    c0, cs = c0.cpu().numpy(), cs.cpu().numpy()
    st0, st1 = binding.parse_info(i0)["status"], binding.parse_info(ics)["status"]
    oc = oracle_mod.Code.from_dense(H)
    om = oracle_mod.omega_from_llr(oracle_mod.llr_from_priors(priors))
    for b in range(len(S)):
        L64 = L[b].astype(np.float64)
        want, ost = oracle_mod.osd0(oc, S[b], L64)
        assert (c0[b] == want).all() and bool(st0[b] & binding.ST_UNSAT) == bool(ost & oracle_mod.ST_UNSAT), b
        want, ost = oracle_mod.osd_cs(oc, S[b], L64, order, om)
        assert (cs[b] == want).all() and bool(st1[b] & binding.ST_UNSAT) == bool(ost & oracle_mod.ST_UNSAT), b


def _heavy_graph(m, n, heavy, seed):
    """Columns of weight 1 or 2 and, every ninth, of weight `heavy`; rows of weight 2 to 32."""
    rng = np.random.default_rng(seed)
    H = np.zeros((m, n), dtype=np.uint8)
    load = np.zeros(m, dtype=int)
    for j in range(n):
        room = np.nonzero(load < 32)[0]
        w = min(len(room), heavy if j % 9 == 0 else int(rng.integers(1, 3)))
        rows = rng.choice(room, size=w, replace=False)
        H[rows, j] = 1
        load[rows] += 1
    for i in np.nonzero(load < 2)[0]:
        H[i, rng.choice(np.nonzero(H[i] == 0)[0], size=2, replace=False)] = 1
    return H


# lone growing clusters: columns of up to 1, 2, 8 and 16 checks (the lanes that share a row's edges), rows of
# more edges than are read ahead, keys outside LDS (more than 4096 faults), rounds of all clusters after them
@pytest.mark.parametrize("m,n,heavy,mu", [(90, 200, 1, 0), (150, 400, 2, 0), (140, 600, 7, 0), (130, 400, 15, 0),
                                          (130, 400, 16, 3), (250, 4400, 3, 0), (250, 4400, 4, 2), (130, 200, 3, 5)])
def test_lsd_of_lone_clusters(oracle_mod, m, n, heavy, mu):
    print(f"case lsd_shapes lone {m}x{n} weight {heavy} mu {mu}", flush=True)
    H = _heavy_graph(m, n, heavy, seed=m + n + heavy)
    rng = np.random.default_rng(m * n)
    # a few flipped checks, soft information that leads the growth astray: many rounds of few clusters
    E = (rng.random((48, n)) < (np.arange(48) % 6 + 1)[:, None] / (2.0 * n)).astype(np.int64)
    S = np.ascontiguousarray((E @ H.T % 2).astype(np.uint8))
    S[::5, rng.integers(m)] ^= 1
    L = rng.normal(2.0, 2.0, size=(48, n)).astype(np.float32)
    L[::4] = np.rint(L[::4] / 2)
    L = np.ascontiguousarray(L + 6.0 * E.astype(np.float32))
    bc = binding.Code.from_dense(H)
    priors = np.full(n, 0.02)
    dec = binding.Decoder(bc, priors, 48, max_iter=5, lsd_order=mu)
    corr, info, st = dec.lsd_stats(torch.from_numpy(S).cuda(), torch.from_numpy(L).cuda())
    torch.cuda.synchronize()
    c, st, inf = corr.cpu().numpy(), st.cpu().numpy(), binding.parse_info(info)
    oc = oracle_mod.Code.from_dense(H)
    om = oracle_mod.omega_from_llr(oracle_mod.llr_from_priors(priors))
    most = 0
    for b in range(48):
        want, ost, stats = oracle_mod.lsd(oc, S[b], L[b].astype(np.float64), mu=mu, omega=om)
        assert not inf["status"][b] & (binding.ST_OVERFLOW | binding.ST_BAD_LLR), b
        assert (c[b] == want).all(), b
        assert bool(inf["status"][b] & binding.ST_UNSAT) == bool(ost & oracle_mod.ST_UNSAT), b
        assert tuple(st[b]) == (stats[0], stats[1], stats[3], stats[6]), b
        if not ost & oracle_mod.ST_UNSAT:
            assert inf["rounds"][b] == stats[2], b
        most = max(most, int(inf["rounds"][b]))
    print(f"  rounds up to {most}")


def _blocks(chain, copies, weight):
    """A chain of `chain` checks, two faults between neighbours (a syndrome of odd weight is outside its
    image), beside `copies` blocks of `weight` checks with one fault on each check and one on all."""
    m, n = chain + copies * weight, 2 * (chain - 1) + copies * (weight + 1)
    H = np.zeros((m, n), dtype=np.uint8)
    for i in range(chain - 1):
        H[i:i + 2, 2 * i:2 * i + 2] = 1
    for k in range(copies):
        r, c = chain + k * weight, 2 * (chain - 1) + k * (weight + 1)
        H[r + np.arange(weight), c + np.arange(weight)] = 1
        H[r:r + weight, c + weight] = 1
    return H


# LSD-mu after a cluster that grew alone has found no fault left: its rounds of all other clusters take more
# (cluster, check) pairs than a wavefront has lanes (22 clusters of column weight 3, 5 of weight 16), or fewer
@pytest.mark.parametrize("chain,copies,weight,mu", [(3, 30, 3, 1), (40, 30, 3, 3), (70, 60, 3, 2), (40, 6, 16, 2),
                                                    (9, 12, 16, 5), (40, 4, 3, 2)])
def test_lsd_mu_after_a_frozen_cluster(oracle_mod, chain, copies, weight, mu):
    print(f"case lsd_shapes frozen chain {chain} copies {copies} weight {weight} mu {mu}", flush=True)
    H = _blocks(chain, copies, weight)
    m, n = H.shape
    rng = np.random.default_rng(m + n)
    B, first = 24, 2 * (chain - 1)
    S = np.zeros((B, m), dtype=np.uint8)
    L = rng.normal(3.0, 0.5, size=(B, n)).astype(np.float32)
    starts = chain + weight * np.arange(copies)
    for b in range(B):
        S[b, rng.choice(chain, size=1 + 2 * (b % 2), replace=False)] = 1
        # every block, or all but a few: a check of it, whose own fault is the likeliest of the block
        some = starts[rng.permutation(copies)[b % 3:]]
        S[b, some] = 1
        L[b, first + (some - chain) // weight * (weight + 1)] = 1.0
    L[1::4, first:] = np.rint(L[1::4, first:])
    bc = binding.Code.from_dense(H)
    priors = np.random.default_rng(7).uniform(0.01, 0.2, size=n)
    dec = binding.Decoder(bc, priors, B, max_iter=5, lsd_order=mu)
    corr, info, st = dec.lsd_stats(torch.from_numpy(S).cuda(), torch.from_numpy(L).cuda())
    torch.cuda.synchronize()
    c, st, inf = corr.cpu().numpy(), st.cpu().numpy(), binding.parse_info(info)
    oc = oracle_mod.Code.from_dense(H)
    om = oracle_mod.omega_from_llr(oracle_mod.llr_from_priors(priors))
    for b in range(B):
        want, ost, stats = oracle_mod.lsd(oc, S[b], L[b].astype(np.float64), mu=mu, omega=om)
        assert ost & oracle_mod.ST_UNSAT and inf["status"][b] & binding.ST_UNSAT, b
        assert not inf["status"][b] & (binding.ST_OVERFLOW | binding.ST_BAD_LLR), b
        assert (c[b] == want).all(), b
        assert tuple(st[b]) == (stats[0], stats[1], stats[3], stats[6]), b


# columns of up to 16 checks where the clusters are held by the lanes (at most 128 checks and 192 faults)
@pytest.mark.parametrize("m,n,heavy", [(40, 100, 9), (64, 120, 16), (96, 190, 11), (128, 192, 16)])
def test_lsd_of_small_heavy_graphs(oracle_mod, m, n, heavy):
    print(f"case lsd_shapes small {m}x{n} weight {heavy}", flush=True)
    H = _heavy_graph(m - 1, n, heavy - 2, seed=m + n + heavy)
    H = np.vstack([H, H[:1]])  # a dependent check: syndromes outside the image
    assert 1 <= H.sum(0).min() and 7 <= H.sum(0).max() <= 16 and H.sum(1).max() <= 32
    S, L = _shots(H, seed=m * n, dense=8)
    dec = binding.Decoder(binding.Code.from_dense(H), np.full(n, 0.02), len(S), max_iter=5)
    corr, info, st = dec.lsd_stats(torch.from_numpy(S).cuda(), torch.from_numpy(L).cuda())
    torch.cuda.synchronize()
    c, st, inf = corr.cpu().numpy(), st.cpu().numpy(), binding.parse_info(info)
    oc = oracle_mod.Code.from_dense(H)
    unsat = 0
    for b in range(len(S)):
        want, ost, stats = oracle_mod.lsd(oc, S[b], L[b].astype(np.float64))
        assert not inf["status"][b] & (binding.ST_OVERFLOW | binding.ST_BAD_LLR), b
        assert (c[b] == want).all(), b
        assert bool(inf["status"][b] & binding.ST_UNSAT) == bool(ost & oracle_mod.ST_UNSAT), b
        assert tuple(st[b]) == (stats[0], stats[1], stats[3], stats[6]), b
        unsat += bool(ost & oracle_mod.ST_UNSAT)
    assert unsat
