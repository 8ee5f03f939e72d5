"""Edges of the channel-norm pass on the GPU: tiles of 64 / 32 rows and 64 columns with remainders,
rows that start on 16 bytes and rows that do not (two load paths of one kernel), runs of one row,
runs cut by tiles and chunks, and several chunks; every case against a binary64 sum."""
import numpy as np
import pytest
import torch

import workloads
from test_parity_gpu import DEV

pytestmark = pytest.mark.gpu


def reference(x, grows, groups, div, rep):
    r = torch.arange(x.shape[0], device=x.device)
    g = (r // grows) % groups // div
    out = torch.zeros((groups // div, x.shape[1]), dtype=torch.float64, device=x.device)
    out.index_add_(0, g, x.double().square())
    return out.repeat_interleave(rep, 0).cpu().numpy()


@pytest.mark.parametrize("rows,cols", [(1, 8), (63, 64), (65, 72), (255, 200), (257, 63), (700, 136), (33, 1)])
@pytest.mark.parametrize("args", [(1, 1, 1, 1), (5, 1, 1, 2), (1, 4, 1, 1), (1, 4, 2, 3), (31, 3, 1, 1), (300, 2, 2, 1)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_norms_edges(rows, cols, args, dtype):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 91, rows, cols)
    x = torch.randn((rows, cols), generator=g, device=DEV).to(dtype)
    got = nv.channel_sq_norms(x, *args)
    buf = torch.empty(x.numel() + 1, dtype=dtype, device=DEV)
    buf[1:].copy_(x.reshape(-1))
    shifted = nv.channel_sq_norms(buf[1:].view(rows, cols), *args)   # no row starts on 16 bytes
    torch.cuda.synchronize()
    ref = reference(x, *args)
    # at most 700 additions of rounding 2^-53 each, then one rounding to binary32 (2^-24)
    assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= ref * (2.0 ** -24 + 700 * 2.0 ** -53))
    assert torch.equal(got.view(torch.int32), shifted.view(torch.int32))    # one order of additions


# runs of at least 256 rows on 4096 workgroups (straight from memory), and one chunk fewer (tiles): 2048
# chunks of 256 rows and 2 column tiles, with a ragged last run and last columns
@pytest.mark.parametrize("rows", [2048 * 256, 2048 * 256 - 5, 2047 * 256])
@pytest.mark.parametrize("args", [(256, 3, 1, 1), (1000, 4, 2, 2)])
def test_norms_long_runs(rows, args):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 92, rows)
    x = torch.randn((rows, 72), generator=g, device=DEV).to(torch.bfloat16)
    got = nv.channel_sq_norms(x, *args)
    torch.cuda.synchronize()
    ref = reference(x, *args)
    # at most 2^19 additions of rounding 2^-53 each on either side, then one rounding to binary32
    assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= ref * (2.0 ** -24 + 2.0 ** -33))


# Both forms of the pass (through tiles, and runs straight from memory) add in one order.  A bfloat16
# matrix, its exact binary32 widening, and the same values one element off 16 bytes meet the rule between
# them on both sides: runs of 7, 8, 9, 15, 16, 39 (rows that load singly) and 40 rows, 1 to 257 workgroups
# of 64 columns (the shifted ones go through tiles from 65 on).
@pytest.mark.parametrize("chunks", [1, 63, 64, 65, 257])
@pytest.mark.parametrize("args", [(7, 3, 1, 1), (8, 2, 1, 1), (3, 6, 3, 1), (15, 2, 1, 2), (16, 1, 1, 1), (39, 2, 1, 1), (20, 4, 2, 1), (100, 33, 1, 1), (2, 64, 8, 1)])
def test_norms_forms_agree(chunks, args):
    check_forms(256 * chunks - 3, 64, args)


# 4094 and 4096 workgroups: straight from memory at 4096, shifted rows with runs of 9 rows and more, the others
# of 256 and more; 6 and 7 a CU of 32 groups, of which a CU holds six through tiles (shifted rows)
@pytest.mark.parametrize("chunks,cols", [(768, 128), (769, 128), (2047, 128), (2048, 128)])
@pytest.mark.parametrize("run,groups", [(9, 16), (40, 32), (255, 3), (256, 3), (256, 1)])
def test_norms_forms_agree_on_large_grids(chunks, cols, run, groups):
    check_forms(256 * chunks, cols, (run, groups, 1, 1))


def check_forms(rows, cols, args):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 93, rows, cols)
    x = torch.randn((rows, cols), generator=g, device=DEV).to(torch.bfloat16)
    got = nv.channel_sq_norms(x, *args)
    ref = reference(x, *args)
    # a group's additions, at most one a row, of rounding 2^-53 each, then one rounding to binary32 (2^-24)
    assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= ref * (2.0 ** -24 + rows * 2.0 ** -53))
    for dtype in (torch.bfloat16, torch.float32):
        buf = torch.empty(x.numel() + 1, dtype=dtype, device=DEV)
        buf[1:].copy_(x.reshape(-1))
        for other in (x.to(dtype), buf[1:].view(rows, cols)):
            again = nv.channel_sq_norms(other, *args)
            assert torch.equal(got.view(torch.int32), again.view(torch.int32))
