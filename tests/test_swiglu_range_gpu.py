"""The SwiGLU producer's two forms on the GPU: waves whose gates (16 a lane) all lie inside (-80, 80) and
waves with one that does not, at the limit and beyond, and every gate inside with several factors; bit for
bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_parity_gpu import DEV

pytestmark = pytest.mark.gpu


def check(nv, gate_bits, up_bits):
    gate = torch.from_numpy(gate_bits.view(np.int16)).to(DEV).view(torch.bfloat16)
    up = torch.from_numpy(up_bits.view(np.int16)).to(DEV).view(torch.bfloat16)
    h = nv.swiglu(gate, up)
    torch.cuda.synchronize()
    ref = oracle.swiglu(workloads.host_array(gate), workloads.host_array(up))
    assert np.array_equal(h.cpu().view(torch.int16).numpy().view(np.uint16), np.asarray(ref).view(np.uint16))


@pytest.mark.parametrize("lane_at", range(16))
@pytest.mark.parametrize("value", [0x429F, 0x42A0, 0xC29F, 0xC2A0, 0xC2B1, 0xC2B2, 0x7F7F, 0xFF7F, 0x8000, 0x0001])
def test_one_gate_at_the_limit(lane_at, value):
    import paper_2606_07618_amd as nv
    rng = np.random.default_rng(lane_at)
    gate = (rng.standard_normal((5, 48)).astype(np.float32) * 3).view(np.uint32) >> 16
    up = (rng.standard_normal((5, 48)).astype(np.float32)).view(np.uint32) >> 16
    gate[1, 16 + lane_at] = value
    check(nv, gate.astype(np.uint16), up.astype(np.uint16))


@pytest.mark.parametrize("seed", range(4))
def test_every_gate_in_range(seed):
    import paper_2606_07618_amd as nv
    bits = np.arange(0x42A0, dtype=np.uint16)                       # 0 .. below 80
    gate = np.concatenate([bits, bits | 0x8000]).reshape(-1, 32)
    up = (np.random.default_rng(seed).standard_normal(gate.shape).astype(np.float32).view(np.uint32) >> 16)
    check(nv, gate, up.astype(np.uint16))


@pytest.mark.parametrize("wave", [0, 1, 4, 6])
@pytest.mark.parametrize("lane_at", [0, 63])
def test_one_wave_out_of_range(wave, lane_at):
    """Seven waves of 1024 gates (the last one short), one of them with a gate at the limit."""
    import paper_2606_07618_amd as nv
    rng = np.random.default_rng([wave, lane_at])
    gate = (rng.standard_normal(6 * 1024 + 1008).astype(np.float32) * 3).view(np.uint32) >> 16
    up = rng.standard_normal(gate.size).astype(np.float32).view(np.uint32) >> 16
    gate[min(wave * 1024 + lane_at * 16 + 5, gate.size - 1)] = 0x42A0
    check(nv, gate.astype(np.uint16).reshape(-1, 48), up.astype(np.uint16).reshape(-1, 48))
