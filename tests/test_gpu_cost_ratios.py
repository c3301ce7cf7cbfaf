"""Ratios of two timings on one device, for calls whose cost has to follow another's: a kernel that falls
off its path (registers in memory, one thread where a wavefront belongs) shows here and in no result."""
import numpy as np
import pytest

from paper_2406_18655_amd import binding
from paper_2406_18655_amd.workloads import bivariate_bicycle, sample, synthetic_dem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()


def _ms(call, passes=1):
    """Shortest of five measurements of `passes` calls, in ms a call."""
    call()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(passes):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / passes)
    return best


def test_lsd_mu_rounds_of_wide_shots():
    """Shots of the detector error model whose clusters outgrow 512 rows: the rounds are nearly all of
    LSD-1's time, so it stays close to LSD-0's (0.9 of it; 1.3 where the sweep's calls cost the rounds
    their registers)."""
    print("case cost wide lsd-mu", flush=True)
    code = synthetic_dem()
    rng = np.random.default_rng(7)
    E = (rng.random((8, code.n)) < 0.003).astype(np.int32)
    s = torch.from_numpy((E @ code.H.T.astype(np.int32) % 2).astype(np.uint8)).cuda()
    llr = torch.from_numpy((rng.normal(3, 2, E.shape) - 3 * E).astype(np.float32)).cuda()
    bc = binding.Code.from_dense(code.H)
    t = [_ms(lambda d=binding.Decoder(bc, code.priors, 8, max_iter=10, lsd_order=mu): d.lsd(s, llr)) for mu in (0, 1)]
    print(f"  LSD-0 {t[0]:.1f} ms, LSD-1 {t[1]:.1f} ms")
    assert t[1] <= 1.15 * t[0]


def _flags(n, rows, weight, B):
    """A call that scores B shots of n faults by logical rows of the given weight."""
    rng = np.random.default_rng(1)
    L = np.zeros((rows, n), dtype=np.uint8)
    for q in range(rows):
        L[q, rng.choice(n, size=weight, replace=False)] = 1
    H = np.zeros((2, n), dtype=np.uint8)
    H[0, ::2] = H[1, 1::2] = 1
    smp = binding.Sampler(binding.Code.from_dense(H), np.full(n, 0.01), L if rows else None)
    e, c = torch.zeros((2, B, n), dtype=torch.uint8, device="cuda")
    f = torch.empty(B, dtype=torch.uint8, device="cuda")
    return lambda: smp.failures_into(e, c, f)


def test_failure_flags_by_logical_rows():
    """6,000 shots of 8,800 faults: one row over half the faults costs what looking at every fault costs
    (1.1 of it; 13 with one thread for the row), twelve rows of 14 a part of it (2,000 shots: 0.4; 1.0 if
    every fault is read)."""
    print("case cost failure flags", flush=True)
    t = [_ms(_flags(8800, *a), passes=30) for a in ((0, 0, 6000), (1, 4400, 6000), (0, 0, 2000), (12, 14, 2000))]
    print("  ms " + " ".join(f"{x:.4f}" for x in t))
    assert t[1] <= 2.0 * t[0] and t[3] <= 0.7 * t[2]


def test_syndromes_of_few_shots():
    """32 shots of the detector error model take one group of bit-sliced shots: their syndromes cost what
    one shot's flags cost, a launch (1.05 of it; 2.1 on one workgroup)."""
    print("case cost few syndromes", flush=True)
    code = synthetic_dem()
    smp = binding.Sampler(binding.Code.from_dense(code.H), code.priors)
    e = torch.zeros((32, code.n), dtype=torch.uint8, device="cuda")
    s = torch.empty((32, code.m), dtype=torch.uint8, device="cuda")
    t = [_ms(_flags(144, 1, 5, 1), passes=100), _ms(lambda: smp.syndromes_into(e, s), passes=100)]
    print("  ms " + " ".join(f"{x:.4f}" for x in t))
    assert t[1] <= 1.5 * t[0]


def test_bp_of_heavy_columns():
    """BP of 1000 x 9000 with one column in four of weight 5 against the detector error model (936 x 8800,
    columns of 1 to 4): 27,000 against 24,643 edges (1.2 times the time; 3.5 with its offsets in memory)."""
    print("case cost heavy columns", flush=True)
    rng = np.random.default_rng(1)
    H = np.zeros((1000, 9000), dtype=np.uint8)
    load = np.zeros(1000)
    for j in range(9000):
        rows = np.argsort(load + 2 * rng.random(1000))[:(2, 2, 3, 5)[j % 4]]
        H[rows, j] = 1
        load[rows] += 1
    t = []
    for M in (H, synthetic_dem().H):
        s = torch.from_numpy((rng.random((512, len(M))) < 0.5).astype(np.uint8)).cuda()
        dec = binding.Decoder(binding.Code.from_dense(M), np.full(M.shape[1], 0.01), 512, max_iter=30)
        t.append(_ms(lambda: dec.bp(s), passes=3))
    print("  ms " + " ".join(f"{x:.4f}" for x in t))
    assert t[0] <= 2.0 * t[1]


def test_decode_of_easy_batches():
    """1,500 shots that BP solves at once: a decode is BP, the end of its kernel and two short launches, 1.5
    times BP as a kernel of its own (2.3 where a thousand wavefronts poll for LSD work that never comes)."""
    print("case cost easy batch", flush=True)
    code = bivariate_bicycle(p=0.003)
    s = torch.from_numpy(sample(code, 1500, seed=5)[1]).cuda()
    dec = binding.Decoder(binding.Code.from_dense(code.H), code.priors, 1500, max_iter=30)
    corr = torch.empty((1500, code.n), dtype=torch.uint8, device="cuda")
    t = [_ms(lambda: dec.bp(s), passes=50), _ms(lambda: dec.decode_into(s, corr), passes=50)]
    print("  ms " + " ".join(f"{x:.4f}" for x in t))
    assert t[1] <= 2.0 * t[0]
