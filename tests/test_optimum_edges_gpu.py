"""Edges of the reference-scale kernel on the GPU, bit for bit against the oracle: blocks whose
breakpoints tie or nearly tie across elements, blocks with zeros, magnitudes over the whole binary32
range, and counts of blocks that do not fill a workgroup's batch."""
import numpy as np
import pytest
import torch

import workloads
from test_parity_gpu import DEV
from test_parity_optimum_gpu import compare_optimum, oracle_blocks

pytestmark = pytest.mark.gpu


def blocks(rng, count, n):
    """Values 4m (the seven midpoints' multiples) times powers of two, some one ulp off, some zero."""
    x = rng.choice([1, 3, 5, 7, 10, 14, 20], (count, n)).astype(np.float32)
    x *= np.exp2(rng.integers(-3, 4, (count, n))).astype(np.float32)
    up = np.nextafter(x, np.float32(np.inf), dtype=np.float32)
    x = np.where(rng.random((count, n)) < 0.3, up, x)
    x = np.where(rng.random((count, n)) < rng.choice([0.0, 0.2, 0.9], (count, 1)), np.float32(0), x)
    return (x * np.where(rng.random((count, n)) < 0.5, -1, 1)).astype(np.float32)


@pytest.mark.parametrize("n", [16, 32, 64, 128])
@pytest.mark.parametrize("count", [1, 2, 3, 5, 37])
def test_optimum_ties_and_partial_batches(n, count):
    import paper_2606_07618_amd as nv
    rng = np.random.default_rng([n, count])
    x = blocks(rng, count, n)
    x[0] = 0.0
    x[-1] = x[-1] * np.exp2(rng.integers(-120, 120, n)).astype(np.float32)
    w = rng.choice([0.0, 0.25, 1.0, 3.0], n).astype(np.float32)
    S = torch.ones(1, device=DEV)
    xt = torch.from_numpy(x).to(DEV)
    for weight in (None, w):
        got = nv.block_optimum(xt, S, n, None if weight is None else torch.from_numpy(weight).to(DEV))
        torch.cuda.synchronize()
        compare_optimum(got, oracle_blocks(workloads.host_array(xt), 1.0, n, weight), f"n {n} count {count}")


# the most blocks of 16 that take a workgroup each, and more of them, four to a workgroup, with remainders
@pytest.mark.parametrize("count", [10240, 10241, 10242, 10243, 10244])
def test_optimum_single_blocks_and_batches(count):
    test_optimum_ties_and_partial_batches(16, count)


@pytest.mark.parametrize("n", [16, 32, 64, 128])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_optimum_nonfinite_elements(n, bad):
    """A block with an infinity or a NaN has that loss, at the all-zero reconstruction; its neighbours are
    what they are without it.  One such element (first, middle, last), several, and a block of nothing else."""
    import paper_2606_07618_amd as nv
    rng = np.random.default_rng([n, 7])
    x = rng.standard_normal((11, n)).astype(np.float32)
    x[9] = 0.0
    S = torch.ones(1, device=DEV)
    clean = [t.cpu().numpy().reshape(-1) for t in nv.block_optimum(torch.from_numpy(x).to(DEV), S, n)]
    rows = [1, 3, 4, 6, 8]
    for r, at in zip(rows, ([0], [n // 2], [n - 1], list(range(0, n, 3)), list(range(n)))):
        x[r, at] = bad
    for weight in (None, torch.ones(n, device=DEV)):
        got = [t.cpu().numpy().reshape(-1) for t in nv.block_optimum(torch.from_numpy(x).to(DEV), S, n, weight)]
        torch.cuda.synchronize()
        for r in range(11):
            if r not in rows:
                assert all(g[r] == c[r] for g, c in zip(got, clean)), r
                continue
            loss, scale, code, fp8 = (g[r] for g in got)
            assert np.isnan(loss) if np.isnan(bad) else loss == np.inf
            assert scale == np.inf and code == 126
            assert np.isnan(fp8) if np.isnan(bad) else fp8 == np.inf
