"""Workgroup shapes of the slot BP kernel: 256 threads with four workgroups per compute unit, 1024
threads with one, and batches smaller than the grid's slots, which spread over the compute units
with fewer slots per workgroup.  BP is the same function of a shot in every shape, so posteriors of
a shot do not depend on its batch; they are checked against the float64 oracle, and the decode
whose BP and LSD share one kernel of 1024 threads against the two-kernel path, byte for byte."""
import numpy as np
import pytest

import _r24
from paper_2406_18655_amd import binding
from paper_2406_18655_amd.workloads import CheckMatrix, bivariate_bicycle, random_34_hgp, sample

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _random_code(m=96, n=640, cw=3, p=0.01, seed=4):
    """m <= 128 checks of weight 20: too many edges for four workgroups per compute unit, few
    enough checks for BP and LSD in one kernel."""
    rng = np.random.default_rng(seed)
    H = np.zeros((m, n), dtype=np.uint8)
    load = np.zeros(m, dtype=int)
    for j in range(n):
        rows = np.lexsort((rng.random(m), load))[:cw]
        H[rows, j] = 1
        load[rows] += 1
    return CheckMatrix(name="random_96x640", H=H, priors=np.full(n, p))


CODES = {"bb144": lambda: bivariate_bicycle(p=0.05), "hgp16": lambda: random_34_hgp(16, p=0.03),
         "random96": _random_code}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("which", list(CODES))
def test_bp_does_not_depend_on_the_batch(oracle_mod, which):
    code = CODES[which]()
    full = 6000
    print(f"case bp_shapes {which}", flush=True)
    e, S = sample(code, full, seed=31)
    bc = binding.Code.from_dense(code.H)
    dec = binding.Decoder(bc, code.priors, full, max_iter=30)
    s = torch.from_numpy(S).cuda()
    L, hard, info = dec.bp(s)
    for B in (1, 2, 255, 256, 257, 1025, 3001):
        print(f"  batch {B}", flush=True)
        l, h, i = dec.bp(s[:B])
        assert torch.equal(l.view(torch.int32), L[:B].view(torch.int32)) and torch.equal(h, hard[:B])
        assert torch.equal(i, info[:B])
    inf = binding.parse_info(info)
    L32, h32 = L[:64].cpu().numpy(), hard[:64].cpu().numpy()
    oc = oracle_mod.Code.from_dense(code.H)
    lam = oracle_mod.llr_from_priors(code.priors)
    for b in range(64):
        _r24.check_shot(oracle_mod, oc, lam, S[b], 30, L32[b], inf["status"][b] & 1, inf["bp_iters"][b], hard32=h32[b])


@pytest.mark.parametrize("B", [1, 300, 5000])
def test_one_kernel_of_wide_workgroups_equals_two(B):
    code = _random_code(p=0.02)
    print(f"case bp_shapes fused {B}", flush=True)
    e, S = sample(code, B, seed=32)
    bc = binding.Code.from_dense(code.H)
    s = torch.from_numpy(S).cuda()
    one = binding.Decoder(bc, code.priors, B, max_iter=20)
    two = binding.Decoder(bc, code.priors, B, max_iter=20, flags=binding.FLAG_SEPARATE_LSD)
    c1, i1 = one.decode(s, want_info=True)
    c2, i2 = two.decode(s, want_info=True)
    torch.cuda.synchronize()
    assert torch.equal(c1, c2) and torch.equal(i1, i2)
    if B >= 300:
        assert (binding.parse_info(i1)["status"] & binding.ST_LSD_RUN).any()


def _weighted_graph(m, n, probs, seed):
    """Columns of weight w with probability probs[w], rows of weight 2 to 32."""
    rng = np.random.default_rng(seed)
    H = np.zeros((m, n), dtype=np.uint8)
    load = np.zeros(m, dtype=np.int64)
    w = rng.choice(len(probs), size=n, p=probs)
    for j in range(n):
        k = min(int(w[j]), int((load < 32).sum()))
        rows = rng.choice(np.nonzero(load < 32)[0], size=k, replace=False)
        H[rows, j] = 1
        load[rows] += 1
    for i in np.nonzero(load < 2)[0]:
        cols = np.nonzero((H.sum(0) < len(probs) - 1) & (H[i] == 0))[0]
        H[i, rng.choice(cols, size=2 - int(load[i]), replace=False)] = 1
    return H, rng.uniform(0.001, 0.05, size=n)


# one workgroup per shot: every instantiation of the fault phase (columns past the first 1024 of
# weight up to 7, or up to 4 with heavier ones first), columns of weight 0, 1024 checks, 9216 faults
LARGE = {"heavy": (700, 3300, [0, 0, .05, .1, .15, .2, .25, .25]),
         "edges": (1024, 9216, [.05, .2, .45, .2, .06, .02, .01, .01]),
         "light": (900, 8000, [0, .1, .9])}


@pytest.mark.parametrize("which", list(LARGE))
@pytest.mark.parametrize("flags", [0, binding.FLAG_NO_EARLY_EXIT])
def test_large_graph_posteriors(oracle_mod, which, flags):
    m, n, probs = LARGE[which]
    H, priors = _weighted_graph(m, n, probs, seed=len(which))
    assert H.sum(1).min() >= 2 and H.sum(1).max() <= 32
    rng = np.random.default_rng(3)
    e = (rng.random((5, n)) < priors / 4).astype(np.uint8)
    S = ((e.astype(np.int64) @ H.T.astype(np.int64)) & 1).astype(np.uint8)
    T = 15
    print(f"case bp_shapes large {which} {flags}", flush=True)
    dec = binding.Decoder(binding.Code.from_dense(H), priors, 5, max_iter=T, flags=flags)
    llr, hard, info = dec.bp(torch.from_numpy(S).cuda())
    torch.cuda.synchronize()
    L32, h32, inf = llr.cpu().numpy(), hard.cpu().numpy(), binding.parse_info(info)
    oc = oracle_mod.Code.from_dense(H)
    lam = oracle_mod.llr_from_priors(priors)
    for b in range(5):
        _r24.check_shot(oracle_mod, oc, lam, S[b], T, L32[b], inf["status"][b] & 1, inf["bp_iters"][b],
                        early_exit=flags == 0, hard32=h32[b])


# as many heavy columns as a layout below 2^15 words holds: the last of weight 7 past position 4096, of 6 past
# 5120, of 5 past 6144 and of 4 past 7168 (each with and without faults past 7 x 1024)
@pytest.mark.parametrize("weight,heavy,n", [(7, 4097, 7650), (7, 4097, 7000), (6, 5121, 6700), (5, 6145, 7750),
                                            (5, 6145, 7168), (4, 7169, 9216), (7, 1025, 9216)])
def test_large_graph_of_heavy_columns(oracle_mod, weight, heavy, n):
    print(f"case bp_shapes large {heavy} of weight {weight} among {n}", flush=True)
    m = 1024
    rng = np.random.default_rng(n + weight)
    H = np.zeros((m, n), dtype=np.uint8)
    load = np.zeros(m)
    at = rng.permutation(n)
    for k, j in enumerate(at):
        rows = np.argsort(load + rng.random(m))[:weight if k < heavy else 1]
        H[rows, j] = 1
        load[rows] += 1
    assert 2 <= load.min() and load.max() <= 32
    assert -(-heavy // 64) * weight + -(-(n - heavy) // 64) < 512  # words of the layout / 64
    priors = rng.uniform(0.001, 0.05, size=n)
    e = (rng.random((4, n)) < priors / 4).astype(np.uint8)
    S = ((e.astype(np.int64) @ H.T.astype(np.int64)) & 1).astype(np.uint8)
    dec = binding.Decoder(binding.Code.from_dense(H), priors, 4, max_iter=12)
    llr, hard, info = dec.bp(torch.from_numpy(S).cuda())
    torch.cuda.synchronize()
    L32, h32, inf = llr.cpu().numpy(), hard.cpu().numpy(), binding.parse_info(info)
    oc = oracle_mod.Code.from_dense(H)
    lam = oracle_mod.llr_from_priors(priors)
    for b in range(4):
        _r24.check_shot(oracle_mod, oc, lam, S[b], 12, L32[b], inf["status"][b] & 1, inf["bp_iters"][b], hard32=h32[b])
