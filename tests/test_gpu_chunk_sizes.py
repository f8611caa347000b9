"""Chunk sizes at the edges of the fixed-size local kernels' row tiles (one row, a
partial tile, a whole one, one more; 33 to 48 rows run on the 64-row instances),
both activations, forward and every gradient against the oracle, and the two
saving modes against each other.  Bound 2e-2 (bf16 inputs), as in the other
backward tests: every product's operands are rounded to bf16 (2^-9 relative each),
and a gradient passes through about ten such products."""
import numpy as np
import pytest
import torch

from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import ACT_GELU, ACT_SILU, BF16, QK_CHUNK, make_inputs, small_config
from test_gpu_backward import GRADS, check, gpu_backward, oracle_backward

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


def cfg_of(C, act, **kw):
    return small_config(BF16, act, B=1, H=2, L=4 * C, d=64, hid=256, C_G=2 * C,
                        locals_=((C, 2 * C),), name=f"bf16 C_L={C} act={act} {kw}", **kw)


@pytest.mark.parametrize("cfg", [
    cfg_of(3, ACT_GELU), cfg_of(16, ACT_GELU), cfg_of(17, ACT_GELU, qk_scope=QK_CHUNK),
    cfg_of(32, ACT_GELU), cfg_of(33, ACT_SILU), cfg_of(40, ACT_GELU, qk_proj=0),
    cfg_of(48, ACT_GELU, qk_scope=QK_CHUNK), cfg_of(49, ACT_SILU), cfg_of(63, ACT_GELU),
], ids=lambda c: c.name)
def test_chunk_sizes(cfg):
    inp = make_inputs(cfg, 501)
    print(f"\n[case] {cfg.name}", flush=True)
    got = gpu_backward(cfg, inp)
    check(cfg, got, oracle_backward(cfg, inp))
    again = gpu_backward(cfg, inp, use_saved=False)
    for n in GRADS:
        assert np.array_equal(got[n], again[n]), n


def test_forward_modes_agree():
    """The saving, the two-pass and the least-workspace forward of a padded shape."""
    cfg = cfg_of(40, ACT_GELU)
    x = tnt.device_inputs(make_inputs(cfg, 502), cfg)
    ws = torch.empty(tnt.tnt_mem_workspace_size(cfg, tnt.TNT_WS_FWD_MIN), dtype=torch.uint8,
                     device="cuda")
    a, b, c = (tnt.forward(cfg, x, save=True)[0], tnt.forward(cfg, x, save=False)[0],
               tnt.forward(cfg, x, save=False, workspace=ws)[0])
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    # one walk instead of two passes: the same products, some in another order
    assert (c.float() - a.float()).abs().max() <= 1e-2 * a.float().abs().max()


@pytest.mark.parametrize("B,H,locals_", [
    (1, 1, ((16, 32),)),            # one unit: one group of the walk's slices
    (9, 15, ((5, 10),)),            # more units than groups (128), no multiple of them
    (8, 20, ((16, 32), (32, 32))),  # two walks side by side, each with half the groups
], ids=str)
def test_walk_groups(B, H, locals_):
    """The sliced walk of the adjoint over few and many units against the runtime-sized
    kernels (2e-2, the bound of both against the oracle), and twice the same bits: the
    slices add in a fixed order whatever order they run in."""
    S = locals_[0][1]
    cfg = small_config(BF16, ACT_SILU, B=B, H=H, L=2 * S, d=64, hid=256, C_G=2 * S,
                       locals_=locals_, name=f"walk B{B} H{H} {locals_}")
    inp = make_inputs(cfg, 503)
    print(f"\n[case] {cfg.name}", flush=True)
    got, again = gpu_backward(cfg, inp), gpu_backward(cfg, inp)
    with tnt.kernel_family(tnt.FAMILY_GENERIC):
        ref = gpu_backward(cfg, inp)
    for n in GRADS:
        assert np.array_equal(got[n], again[n]), n
    check(cfg, got, ref)
