"""The adjoint walk in one part and in two (long walks that leave half the CUs free), and two
walks side by side whose groups take several units in turn, against the runtime-sized
kernels (2e-2: both are within it of the oracle), and the same bits twice."""
import numpy as np
import pytest
import torch

from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import ACT_GELU, ACT_SILU, BF16, make_inputs, small_config
from test_gpu_backward import GRADS, check, gpu_backward

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


@pytest.mark.parametrize("B,H,ns,locals_,act", [
    (2, 8, 4, ((4, 128),), ACT_SILU),            # 64 units of 32 chunks: two parts, 128 CUs
    (2, 8, 5, ((4, 128),), ACT_GELU),            # 80 units: one part
    (2, 8, 5, ((4, 128), (2, 128)), ACT_SILU),   # two walks of 80 units in 64 groups each
    (1, 2, 1, ((48, 1536),), ACT_SILU),          # the one-CU walk in two parts
], ids=str)
def test_walk_parts(B, H, ns, locals_, act):
    S = locals_[0][1]
    cfg = small_config(BF16, act, B=B, H=H, L=ns * S, d=64, hid=256, C_G=S, locals_=locals_,
                       name=f"B{B} H{H} x{ns} {locals_}")
    inp = make_inputs(cfg, 504)
    print(f"\n[case] {cfg.name}", flush=True)
    got, again = gpu_backward(cfg, inp), gpu_backward(cfg, inp)
    with tnt.kernel_family(tnt.FAMILY_GENERIC):
        ref = gpu_backward(cfg, inp)
    for n in GRADS:
        assert np.array_equal(got[n], again[n]), n
    check(cfg, got, ref)
