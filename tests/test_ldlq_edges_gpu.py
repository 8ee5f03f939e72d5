"""Edges of the GPTQ pass on the GPU, nibble for nibble against the oracle: row blocks of 16 and 128 with
remainders, tile counts on both sides of the change from pairs of tiles to single ones, and the values
for which a wave quantizes by the general form (global scales outside [2^-26, 2^26], values of 2^100 and
beyond in some rows), zero scale codes and zero weights among them."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import workloads
from test_parity_gpu import DEV, describe_mismatch
from test_parity_ldlq_gpu import check, synthetic_hessian

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 15, 17, 127, 129])
@pytest.mark.parametrize("tiles", [1, 2, 3, 5])
def test_ldlq_row_blocks(rows, tiles):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 68, rows, tiles)
    w = workloads.llm_weight(rows, 64 * tiles, g, DEV, outlier_frac=0.02).to(torch.bfloat16)
    check(nv, w, synthetic_hessian(64 * tiles, 200, rows))


@pytest.mark.parametrize("tiles", [15, 16, 17, 18, 19, 20, 21, 26])
def test_ldlq_tile_counts(tiles):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 69, tiles)
    w = workloads.llm_weight(19, 64 * tiles, g, DEV, outlier_frac=0.02)
    check(nv, w, synthetic_hessian(64 * tiles, 500, tiles), block=64)


def check_fixed(nv, w, H, sc, S):
    St = torch.tensor([S], dtype=torch.float32, device=DEV)
    got = nv.ldlq(w, H, sc, St, 16).cpu().numpy()
    ref = oracle.ldlq(workloads.host_array(w), H.cpu().numpy(), sc.cpu().numpy(), float(St.item()), 16, 0.01)
    assert np.array_equal(got, ref), describe_mismatch(got, ref, "nibbles")


@pytest.mark.parametrize("S", [2.0 ** -30, 2.0 ** -26, 0.003, 2.0 ** 26, 2.0 ** 26 * 1.0001, 2.0 ** 40])
@pytest.mark.parametrize("factor", [1e-9, 1.0, 1e9])
def test_ldlq_fixed_scales_of_any_size(S, factor):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 70, 1)
    w = workloads.llm_weight(35, 192, g, DEV) * factor
    w[3] = 0.0
    w[4, ::3] = -0.0
    sc = torch.randint(0, 127, (35, 12), generator=g, device=DEV, dtype=torch.uint8)
    sc[5] = 0                                          # zero scales: every nibble a signed zero
    check_fixed(nv, w, synthetic_hessian(192, 300, 3), sc, S)


@pytest.mark.parametrize("at", [(0, 0), (17, 100), (34, 191)])
def test_ldlq_huge_values_in_one_row(at):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 70, 2)
    w = workloads.llm_weight(35, 192, g, DEV)
    w[at] = 2.0 ** 101
    sc = torch.randint(1, 127, (35, 12), generator=g, device=DEV, dtype=torch.uint8)
    check_fixed(nv, w, synthetic_hessian(192, 300, 4), sc, 0.003)


@pytest.mark.parametrize("at", [(0,), (63, 64), (0, 1, 2, 100, 191), tuple(range(192))])
def test_ldlq_nan_on_the_diagonal(at):
    """The order of the columns stays a permutation (the workspace's first ints; filled with other values
    before) and the call reports a Hessian that is not positive definite."""
    import paper_2606_07618_amd as nv
    rows, cols = 35, 192
    g = workloads.generator(DEV, 70, 3)
    w = workloads.llm_weight(rows, cols, g, DEV)
    H = synthetic_hessian(cols, 300, 5)
    H[list(at), list(at)] = float("nan")
    _, sc, S = nv.quantize(w, "absmax", 16)
    nbytes = nv.nvfp4_ldlq_workspace_bytes(rows, cols)
    ws = torch.full((nbytes,), 0x7F, dtype=torch.uint8, device=DEV)
    q = torch.empty((rows, cols // 2), dtype=torch.uint8, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    rc = nv.nvfp4_ldlq(w.data_ptr(), 1, rows, cols, 16, H.data_ptr(), sc.data_ptr(), S.data_ptr(), 0.01,
                       q.data_ptr(), status.data_ptr(), ws.data_ptr(), nbytes,
                       ctypes.c_void_p(torch.cuda.current_stream(DEV).cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0 and int(status.item()) == 1
    perm = ws[:4 * cols].view(torch.int32).cpu().numpy()
    assert np.array_equal(np.sort(perm), np.arange(cols))
    diag = torch.diagonal(H).cpu().numpy()
    assert np.array_equal(perm, np.argsort(-np.where(np.isnan(diag), -np.inf, diag), kind="stable"))
    with pytest.raises(nv.NVFP4Error):
        nv.ldlq(w, H, sc, S, 16)


def test_ldlq_more_row_blocks_than_a_grids_second_dimension():
    """65537 blocks of 64 rows, the last of one row: the launch of every kernel of the pass.  Rows do not
    depend on each other, so the first and the last ones are compared."""
    import paper_2606_07618_amd as nv
    rows, cols = 65536 * 64 + 1, 64
    g = workloads.generator(DEV, 70, 4)
    w = (torch.randn((rows, cols), generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    H = synthetic_hessian(cols, 300, 6)
    _, sc, S = nv.quantize(w, "absmax", 16)
    got = nv.ldlq(w, H, sc, S, 16)
    for sel in (slice(0, 70), slice(rows - 70, rows)):
        ref = oracle.ldlq(workloads.host_array(w[sel]), H.cpu().numpy(), sc[sel].cpu().numpy(), float(S.item()), 16, 0.01)
        part = got[sel].cpu().numpy()
        assert np.array_equal(part, ref), describe_mismatch(part, ref, "nibbles")
