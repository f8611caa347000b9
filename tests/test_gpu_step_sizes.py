"""The step-wise forward at the edges of its launches: the smallest and largest
heads, one and several hidden slices, chunks of one token, more tokens between two
boundaries than one launch takes, no global memory, no local memory.  Against the
oracle (1e-4: fp32 sums in another order) and, cut in two ways, against itself bit
for bit."""
import numpy as np
import pytest
import torch

from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import (ACT_GELU, ACT_SILU, F32, QK_CHUNK, make_inputs, max_rel_err,
                                         small_config)
from test_gpu_step import oracle_o

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


@pytest.mark.parametrize("cfg", [
    small_config(F32, ACT_SILU, B=1, H=1, L=80, d=16, hid=16, C_G=40, locals_=((40, 40),),
                 name="d16 h16, 40 tokens a chunk"),
    small_config(F32, ACT_GELU, B=2, H=1, L=48, d=32, hid=512, C_G=48, locals_=((1, 24), (24, 48)),
                 qk_scope=QK_CHUNK, name="d32 h512, chunks of one token"),
    small_config(F32, ACT_SILU, B=1, H=2, L=64, d=128, hid=32, C_G=32, locals_=(),
                 name="d128 h32, global only"),
    small_config(F32, ACT_SILU, B=1, H=1, L=66, d=128, hid=512, C_G=33, locals_=((33, 66),),
                 has_global=0, name="d128 h512, local only"),
    small_config(F32, ACT_GELU, B=1, H=3, L=60, d=64, hid=64, C_G=20, locals_=((30, 30),),
                 qk_proj=0, name="d64 h64, queries not projected"),
], ids=lambda c: c.name)
def test_step_sizes(cfg):
    print(f"\n[case] {cfg.name}", flush=True)
    inp = make_inputs(cfg, 503)
    x = tnt.device_inputs(inp, cfg)
    whole, s_whole = tnt.step_forward(cfg, x, [cfg.L])
    cut, s_cut = tnt.step_forward(cfg, x, [1, cfg.L // 2, 1, cfg.L - cfg.L // 2 - 2])
    torch.cuda.synchronize()
    nb = cfg.M * cfg.B * cfg.H * (6 * cfg.hid * cfg.d + cfg.d * cfg.d) * 4
    assert torch.equal(whole, cut) and torch.equal(s_whole[:nb], s_cut[:nb])
    e = max_rel_err(whole.cpu().numpy(), oracle_o(cfg, inp))
    print(f"  o vs oracle {e:.3e}", flush=True)
    assert np.isfinite(whole.cpu().numpy()).all() and e <= 1e-4
