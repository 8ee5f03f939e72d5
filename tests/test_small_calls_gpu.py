"""Small calls on the GPU: what is no real number refused as Python does; the padding of swizzled scales at
the edges of its 128 x 4 tiles, written by the launch that quantizes; and the dynamic global scale on both
sides of the grid size up to which every workgroup folds the reduction's partial maxima itself."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_parity_gpu import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 31, 127, 128, 129, 257])
@pytest.mark.parametrize("k16", [1, 3, 4, 5, 256])
@pytest.mark.parametrize("fused", [False, True])
def test_swizzled_padding(rows, k16, fused):
    import paper_2606_07618_amd as nv
    cols = 16 * k16
    g = workloads.generator(DEV, 71, rows, k16)
    x = torch.randn((rows, cols), generator=g, device=DEV).to(torch.bfloat16)
    nbytes = nv.nvfp4_scales_bytes(rows, cols, 16, 1)
    q = torch.empty((rows, cols // 2), dtype=torch.uint8, device=DEV)
    sc = torch.full((nbytes + 64,), 0xA5, dtype=torch.uint8, device=DEV)     # a guard past the end
    if fused:
        up = torch.randn((rows, cols), generator=g, device=DEV).to(torch.bfloat16)
        h = nv.swiglu(x, up)
        nv.quantize_online_swiglu(x, up, "absmax", 0.004, layout="swizzled", out=(q, sc))
    else:
        h = x
        nv.quantize_online(x, "absmax", 0.004, layout="swizzled", out=(q, sc))
    torch.cuda.synchronize()
    q_ref, sc_ref = oracle.quantize_online("absmax", workloads.host_array(h), 0.004, 16, None, 1, 1, "swizzled")
    assert np.array_equal(q.cpu().numpy(), q_ref)
    got = sc.cpu().numpy()
    assert np.array_equal(got[:nbytes], sc_ref.reshape(-1))
    assert np.all(got[nbytes:] == 0xA5)


# 16 elements a lane, 256 lanes a workgroup: 1, 2, 65, 2047, 2048 and 2049 workgroups; 1 to 256 partials
@pytest.mark.parametrize("rows,cols", [(1, 16), (3, 2048), (65, 4096), (2047, 4096), (2048, 4096), (2049, 4096)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("at", [0, -1])
def test_dynamic_scale_on_both_folds(rows, cols, dtype, at):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 72, rows, cols)
    x = torch.randn((rows, cols), generator=g, device=DEV).to(dtype)
    x.view(-1)[at] = -37.0                            # the maximum, in the first or the last partial
    q, sc, S = nv.quantize(x, "absmax", 16)
    S_ref = float(np.float32(37.0) / np.float32(6.0 * 448.0))
    q2, sc2 = nv.quantize_online(x, "absmax", S_ref)  # the static path
    torch.cuda.synchronize()
    assert S.item() == S_ref
    assert torch.equal(q, q2) and torch.equal(sc, sc2)
    zero_q, zero_sc, zero_S = nv.quantize(torch.zeros_like(x), "scalesweep_mse", 16)
    assert zero_S.item() == 1.0 and int(zero_q.max()) == 0


# 1, 2, 127 and 128 workgroups of 16 elements a lane (4 a lane there), and 129, with ragged last ones
@pytest.mark.parametrize("rows,cols", [(1, 16), (1, 4112), (127, 4096), (128, 4096), (129, 4096), (513, 1008)])
@pytest.mark.parametrize("method", ["absmax", "four_over_six", "scalesweep_mse"])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_four_elements_a_lane(rows, cols, method, dtype):
    import paper_2606_07618_amd as nv
    g = workloads.generator(DEV, 73, rows, cols)
    x = workloads.llm_weight(rows, cols, g, DEV, scale=1.0, outlier_frac=0.02).to(dtype)
    x[0, :16] = 0.0
    x[-1, -16:] = torch.tensor([6.0, 3.0, 1.5, 0.75] * 4, device=DEV).to(dtype)     # equal losses of two codes
    imp = workloads.column_importance(cols, g, DEV, tokens=64) if method == "four_over_six" else None
    q, sc, S = nv.quantize(x, method, 16, weight=imp)
    torch.cuda.synchronize()
    D = 448.0 if method == "absmax" else 256.0
    S_ref, q_ref, sc_ref = oracle.quantize(method, workloads.host_array(x), 16, D, 0.0,
                                           None if imp is None else imp.cpu().numpy())
    assert S.item() == S_ref
    assert np.array_equal(sc.cpu().numpy(), sc_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)


@pytest.mark.parametrize("bad,error", [("0.5", TypeError), (None, TypeError), ([0.5], TypeError), (10 ** 400, OverflowError)])
def test_what_is_no_real_number(bad, error):
    import paper_2606_07618_amd as nv
    x = torch.ones((64, 64), dtype=torch.bfloat16, device=DEV)
    H = torch.eye(64, dtype=torch.float64, device=DEV)
    _, sc, S = nv.quantize(x, "absmax", 16)
    for call in (lambda: nv.quantize(x, "absmax", 16, static_scale=bad),
                 lambda: nv.quantize_window(x, 16, static_scale=bad),
                 lambda: nv.quantize_window(x, 16, fp8_range=bad),
                 lambda: nv.quantize_online(x, "absmax", bad),
                 lambda: nv.quantize_online_swiglu(x, x, "absmax", bad),
                 lambda: nv.ldlq(x, H, sc, S, 16, damp=bad)):
        with pytest.raises(error):
            call()
