"""The device quantisers against the host routine, bit for bit, where the work split can go wrong: runs of one row,
more rows than runs, several head groups, head counts that do not divide the workgroup, and scales at the ends
of the float32 range (where the encoder divides instead of multiplying by the reciprocal)."""
import numpy as np
import pytest
import torch

from paper_2603_11101_amd import binding as va
from paper_2603_11101_amd import workloads as wl

from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,D,power", [(1, 1, 8, 0), (2, 300, 8, 0), (257, 2, 8, 0), (1031, 7, 16, 0), (4099, 3, 64, 0),
                                         (700, 17, 128, 0), (9000, 1, 256, 0), (333, 4, 64, -110), (333, 4, 64, 126)])
def test_device_quantisers_equal_the_host_routine(T, H, D, power):
    print(f"quantisers T={T} H={H} D={D} power={power}", flush=True)
    r = np.random.default_rng(T + 7 * H + D)
    x = r.standard_normal((T, H, D)).astype(np.float32)
    x /= np.abs(x).max()
    x *= np.exp2(r.integers(-12, 1, size=(T, H, 1))).astype(np.float32)
    x.flat[::11] = -0.0
    x = wl.round_to_bf16(x * np.float32(2.0) ** np.float32(power))
    bits = wl.bf16_bits(x)
    xt = torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).to(DEV)
    codes = torch.full((T, H, D), 0xAA, dtype=torch.uint8, device=DEV)
    descale = torch.full((H,), -1.0, dtype=torch.float32, device=DEV)
    va.va_quantize_e4m3_per_head_device(xt, codes, descale)
    torch.cuda.synchronize()
    want, want_scale = va.va_quantize_e4m3_per_head(bits)
    assert np.array_equal(descale.cpu().numpy().view(np.uint32), want_scale.view(np.uint32))
    assert np.array_equal(codes.cpu().numpy(), want)
    cu = np.array([0, T // 3, T // 3, T], dtype=np.int32)
    codes.fill_(0xAA)
    per_token = torch.full((T, H), -1.0, dtype=torch.float32, device=DEV)
    va.va_quantize_e4m3_blockwise_device(xt, cu, torch.from_numpy(cu).to(DEV), codes, per_token)
    torch.cuda.synchronize()
    want, want_scale = va.va_quantize_e4m3_blockwise(bits, cu)
    assert np.array_equal(per_token.cpu().numpy().view(np.uint32), want_scale.view(np.uint32))
    assert np.array_equal(codes.cpu().numpy(), want)
