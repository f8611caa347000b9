"""The step-wise forward of one token by itself against several together: the same bits,
whichever form a launch takes (a token goes by itself where the weights are wide, or the
workgroups are more than the CUs)."""
import pytest
import torch

from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import ACT_GELU, ACT_SILU, BF16, F32, QK_CHUNK, make_inputs, small_config

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


def state_bytes(cfg):
    return cfg.M * cfg.B * cfg.H * (6 * cfg.hid * cfg.d + cfg.d * cfg.d) * 4


@pytest.mark.parametrize("cfg", [
    small_config(F32, ACT_SILU, B=1, H=1, L=48, d=64, hid=256, C_G=24, locals_=((12, 24),),
                 name="d64 h256"),
    small_config(BF16, ACT_GELU, B=2, H=3, L=48, d=128, hid=512, C_G=48, locals_=((16, 48), (24, 48)),
                 name="d128 h512, two locals"),
    small_config(F32, ACT_GELU, B=1, H=2, L=40, d=128, hid=16, C_G=40, locals_=((20, 40),),
                 qk_proj=0, name="d128 h16, queries not projected"),
    small_config(BF16, ACT_SILU, B=1, H=2, L=40, d=32, hid=512, C_G=40, locals_=((20, 40),),
                 has_global=0, name="d32 h512, local only"),
    small_config(F32, ACT_SILU, B=2, H=2, L=40, d=64, hid=512, C_G=20, locals_=(), name="d64 h512, global only"),
], ids=lambda c: c.name)
def test_one_by_one_and_together(cfg):
    print(f"\n[case] {cfg.name}", flush=True)
    x = tnt.device_inputs(make_inputs(cfg, 521), cfg)
    a, sa = tnt.step_forward(cfg, x, [1] * cfg.L)
    b, sb = tnt.step_forward(cfg, x, [cfg.L])
    torch.cuda.synchronize()
    n = state_bytes(cfg)
    assert torch.isfinite(a.float()).all()
    assert torch.equal(a, b) and torch.equal(sa[:n], sb[:n])


@pytest.mark.parametrize("d,hid,H,B", [(16, 16, 4, 160), (16, 256, 2, 40), (32, 64, 3, 180), (64, 32, 2, 260)])
def test_many_chains(d, hid, H, B):
    """The first chains of a batch of more workgroups than CUs (by itself) against a batch
    of those chains alone (together, at these sizes)."""
    kw = dict(H=H, L=6, d=d, hid=hid, C_G=3, locals_=((2, 6),), qk_scope=QK_CHUNK)
    few = small_config(F32, ACT_SILU, B=1, name=f"d{d} h{hid} few", **kw)
    many = small_config(F32, ACT_SILU, B=B, name=f"d{d} h{hid} many", **kw)
    print(f"\n[case] {many.name}", flush=True)
    x = tnt.device_inputs(make_inputs(many, 522), many)
    y = {k: v[:, :1] if k in ("lr", "mom", "decay") else v[:1] if k in ("q", "k", "v") else v
         for k, v in x.items()}
    a, _ = tnt.step_forward(many, x, [1] * 6)
    b, _ = tnt.step_forward(few, y, [1] * 6)
    torch.cuda.synchronize()
    assert torch.isfinite(a).all() and torch.equal(a[:1], b)
