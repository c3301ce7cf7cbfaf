"""Sampler kernels at the edges of their splits: batches around the groups of 32 shots and of up to eight
such groups a workgroup, rows that are no whole words, buffers off the word boundary, and matrices too
wide for bit-sliced rows in LDS.  Bits are compared exactly with the host sampler and with products
formed by torch."""
import numpy as np
import pytest

from paper_2406_18655_amd import binding
from paper_2406_18655_amd.workloads import CheckMatrix, bivariate_bicycle, random_34_hgp, sample, surface_hgp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _wide():
    rng = np.random.default_rng(2)
    H = (rng.random((5, 40001)) < 0.01).astype(np.uint8)
    return CheckMatrix(name="wide", H=H, priors=rng.uniform(0.001, 0.5, size=40001),
                       logicals=(rng.random((3, 40001)) < 0.01).astype(np.uint8))


CODES = {"bb144": bivariate_bicycle, "surface5": lambda: surface_hgp(5, 0.1), "hgp16": lambda: random_34_hgp(16),
         "wide": _wide}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()


def _off(rows, cols, shift):
    """A contiguous uint8 [rows, cols] tensor `shift` bytes into an allocation."""
    return torch.zeros(rows * cols + shift, dtype=torch.uint8, device="cuda")[shift:].view(rows, cols)


@pytest.mark.parametrize("which,B,shift", [("bb144", 1, 0), ("bb144", 31, 0), ("bb144", 33, 1), ("bb144", 40000, 2),
                                           ("bb144", 70001, 0), ("bb144", 270000, 0), ("surface5", 64, 3),
                                           ("hgp16", 515, 0), ("wide", 40, 1)])
def test_sampler(which, B, shift):
    code = CODES[which]()
    print(f"case sampler_shapes {which} {B} {shift}", flush=True)
    smp = binding.Sampler(binding.Code.from_dense(code.H), code.priors, code.logicals)
    e, s = _off(B, code.n, shift), _off(B, code.m, shift)
    smp.sample_into(77, 4090, e, s)
    e_h, s_h = sample(code, B, seed=77, start=4090)
    assert np.array_equal(e.cpu().numpy(), e_h) and np.array_equal(s.cpu().numpy(), s_h)
    c, f = _off(B, code.n, shift), torch.empty(B, dtype=torch.uint8, device="cuda")
    c.copy_(e)
    gen = torch.Generator(device="cuda").manual_seed(3)
    flips = (torch.rand((B, code.n), generator=gen, device="cuda") < 1.0 / code.n).byte()
    flips[: B // 2] = 0
    c ^= flips
    smp.failures_into(e, c, f)
    Lt = torch.from_numpy(code.logicals).cuda().t().contiguous().float()
    want = torch.cat([((flips[a:a + 8192].float() @ Lt).remainder_(2) != 0).any(1) for a in range(0, B, 8192)])
    assert torch.equal(f.bool(), want)
    word = binding.Sampler(binding.Code.from_dense(code.H), code.priors)  # no logicals: word error
    word.failures_into(e, c, f)
    assert torch.equal(f.bool(), flips.any(1))
    smp.syndromes_into(c, s)
    Ht = torch.from_numpy(code.H).cuda().t().contiguous().float()
    for a in range(0, B, 8192):
        assert torch.equal(s[a:a + 8192], (c[a:a + 8192].float() @ Ht).remainder_(2).byte())


# rows of logicals that one thread, several threads and several wavefronts share, and both kernels' sides of
# the line between them
@pytest.mark.parametrize("n,rows,weight,B", [(50, 1, 16, 70001), (50, 40, 17, 3), (50, 40, 17, 70000), (300, 3, 250, 40),
                                             (300, 70, 33, 999), (2000, 1, 2000, 20000), (2000, 12, 14, 300),
                                             (9001, 1, 4400, 33), (9001, 8, 880, 65), (9001, 2, 5, 3000)])
def test_failures_by_rows(n, rows, weight, B):
    print(f"case sampler_shapes rows {n} {rows} {weight} {B}", flush=True)
    rng = np.random.default_rng(n + rows)
    L = np.zeros((rows, n), dtype=np.uint8)
    for q in range(rows):  # the last row is light, the one before it empty
        L[q, rng.choice(n, size=weight if q < rows - 2 or rows < 3 else (0 if q == rows - 2 else 1), replace=False)] = 1
    H = np.ones((1, n), dtype=np.uint8)
    smp = binding.Sampler(binding.Code.from_dense(H), np.full(n, 0.01), L)
    gen = torch.Generator(device="cuda").manual_seed(n)
    e = (torch.rand((B, n), generator=gen, device="cuda") < 0.1).byte()
    r = (torch.rand((B, n), generator=gen, device="cuda") < 2.0 / n).byte()
    f = torch.empty(B, dtype=torch.uint8, device="cuda")
    smp.failures_into(e, e ^ r, f)
    Lt = torch.from_numpy(L).cuda().t().contiguous().float()
    want = torch.cat([((r[a:a + 8192].float() @ Lt).remainder_(2) != 0).any(1) for a in range(0, B, 8192)])
    assert torch.equal(f.bool(), want)


# checks of up to 48 entries and of more, both kernels' sides of the line of 3.5 million entries, and shots that
# are no whole groups or words
@pytest.mark.parametrize("m,n,weight,B", [(20, 41, 4, 41666), (20, 41, 4, 42001), (33, 500, 48, 100), (33, 500, 49, 100),
                                          (33, 500, 48, 2211), (936, 8800, 27, 31), (936, 8800, 27, 159)])
def test_syndromes_by_entries(m, n, weight, B):
    print(f"case sampler_shapes entries {m}x{n} weight {weight} {B}", flush=True)
    rng = np.random.default_rng(m + n)
    H = np.zeros((m, n), dtype=np.uint8)
    for i in range(m):
        H[i, rng.choice(n, size=weight, replace=False)] = 1
    smp = binding.Sampler(binding.Code.from_dense(H), np.full(n, 0.01))
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = (torch.rand((B, n), generator=gen, device="cuda") < 0.1).byte()
    s = torch.empty((B, m), dtype=torch.uint8, device="cuda")
    smp.syndromes_into(x, s)
    Ht = torch.from_numpy(H).cuda().t().contiguous().float()
    for a in range(0, B, 8192):
        assert torch.equal(s[a:a + 8192], (x[a:a + 8192].float() @ Ht).remainder_(2).byte())
