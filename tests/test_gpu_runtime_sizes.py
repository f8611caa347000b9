"""The runtime-sized local kernels at the edges of their columns of tiles: 1, 2 and 4
tiles per wave (chosen by the chunk rows), contractions that end inside a
request (16 and 48), partial last rows, head sizes and hidden widths that no fixed-size
kernel takes.  Forward and every gradient against the oracle with the bounds of the
backward tests (1e-4 in fp32; 2e-2 in bf16, whose operands are rounded before each
of about ten products)."""
import pytest
import torch

from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import (ACT_GELU, ACT_SILU, BF16, F32, QK_CHUNK, make_inputs,
                                         small_config)
from test_gpu_backward import check, gpu_backward, oracle_backward

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


def cfg_of(dtype, d, hid, C, act=ACT_SILU, **kw):
    name = f"{('f32', 'bf16')[dtype]} d{d} h{hid} C{C} {kw}"
    return small_config(dtype, act, B=1, H=2, L=4 * C, d=d, hid=hid, C_G=2 * C,
                        locals_=((C, 2 * C),), name=name, **kw)


@pytest.mark.parametrize("cfg", [
    cfg_of(F32, 16, 16, 1), cfg_of(F32, 16, 32, 64, ACT_GELU), cfg_of(F32, 32, 64, 33),
    cfg_of(F32, 64, 64, 50), cfg_of(F32, 128, 128, 20, qk_scope=QK_CHUNK, has_global=0),
    cfg_of(F32, 128, 128, 64, ACT_GELU, has_global=0),
    cfg_of(F32, 128, 16, 61, qk_proj=0, has_global=0),
    cfg_of(BF16, 16, 32, 17), cfg_of(BF16, 32, 16, 48, qk_scope=QK_CHUNK),
    cfg_of(BF16, 64, 64, 64, ACT_GELU), cfg_of(BF16, 128, 128, 32), cfg_of(BF16, 128, 128, 55),
], ids=lambda c: c.name)
def test_runtime_sizes(cfg):
    inp = make_inputs(cfg, 601)
    print(f"\n[case] {cfg.name}", flush=True)
    check(cfg, gpu_backward(cfg, inp), oracle_backward(cfg, inp))


@pytest.mark.parametrize("C,d", [(16, 64), (32, 64), (64, 64)])
def test_forced_generic(C, d):
    """The same kernels at a size that has fixed-size ones, against them."""
    cfg = cfg_of(BF16, d, 256, C)
    inp = make_inputs(cfg, 602)
    with tnt.kernel_family(tnt.FAMILY_GENERIC):
        got = gpu_backward(cfg, inp)
    check(cfg, got, gpu_backward(cfg, inp))


@pytest.mark.parametrize("cfg", [cfg_of(F32, 64, 16, 50),
                                 cfg_of(F32, 128, 32, 20, has_global=0),
                                 cfg_of(BF16, 128, 64, 55)], ids=lambda c: c.name)
def test_hid_below_head_size(cfg):
    """hid < d: the packed transpose of the Q-K sum is the largest of a state's matrices
    (only its first hid / 32 rows of tiles used to be written, and dq was wrong)."""
    inp = make_inputs(cfg, 603)
    print(f"\n[case] {cfg.name}", flush=True)
    check(cfg, gpu_backward(cfg, inp), oracle_backward(cfg, inp))
