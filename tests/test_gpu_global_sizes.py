"""Global chunks around the fixed-size kernels' token tiles (64 or 32 rows) and K slabs
(128 tokens), at every head size they are built for: output, final state and every
gradient against the oracle.  Bound 2e-2 (bf16 inputs; every product's operands are
rounded to bf16, 2^-9 relative each, and a gradient passes through about ten such
products); the final state, a sum over two chunks of products of both signs, 4e-2 as
the per-chunk bound of the full-size tests."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import ACT_GELU, ACT_SILU, BF16, make_inputs, max_rel_err, small_config
from test_gpu_backward import check, gpu_backward, oracle_backward

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


def cfg_of(d, hid, C, act, chunks=3, locals_=()):
    return small_config(BF16, act, B=1, H=2, L=chunks * C, d=d, hid=hid, C_G=C, locals_=locals_,
                        name=f"bf16 d{d} h{hid} C_G={C} act={act} {locals_}")


@pytest.mark.parametrize("cfg", [
    cfg_of(64, 256, 1, ACT_SILU, chunks=16), cfg_of(64, 256, 63, ACT_GELU),
    cfg_of(64, 256, 65, ACT_SILU), cfg_of(64, 256, 128, ACT_SILU),
    cfg_of(64, 256, 130, ACT_SILU, locals_=((13, 26),)), cfg_of(64, 128, 100, ACT_GELU),
    cfg_of(32, 128, 129, ACT_SILU), cfg_of(32, 128, 40, ACT_GELU),
    cfg_of(128, 512, 33, ACT_GELU), cfg_of(128, 512, 160, ACT_SILU, chunks=2),
], ids=lambda c: c.name)
def test_global_chunk_sizes(cfg):
    inp = make_inputs(cfg, 511)
    print(f"\n[case] {cfg.name}", flush=True)
    check(cfg, gpu_backward(cfg, inp), oracle_backward(cfg, inp))
    x = tnt.device_inputs(inp, cfg)
    o, _, fin = tnt.forward(cfg, x, save=False, final_state=True)
    o2, _, _ = tnt.forward(cfg, x, save=True)
    torch.cuda.synchronize()
    pairs = O.all_pairs(cfg)
    ref, rfin = O.forward_pairs(inp, cfg, pairs, with_final=True)
    e = max_rel_err(o.float().cpu().numpy(), ref.numpy().reshape(o.shape))
    rf = np.concatenate([f.numpy().reshape(len(pairs), -1) for f in rfin], 1)
    ef = max_rel_err(fin.cpu().numpy().reshape(rf.shape), rf)
    print(f"  o {e:.3e} final state {ef:.3e}", flush=True)
    assert e <= 2e-2 and ef <= 4e-2
    assert torch.equal(o, o2)


@pytest.mark.parametrize("C", [512, 768])
def test_whole_chunks_in_short_splits(C):
    """Few chains: chunks of a multiple of 256 tokens go in splits of 256."""
    cfg = cfg_of(64, 256, C, ACT_GELU, chunks=2)
    inp = make_inputs(cfg, 513)
    check(cfg, gpu_backward(cfg, inp), oracle_backward(cfg, inp))


def test_long_chunk_in_uneven_splits():
    """1100 tokens a chunk: two splits of 640 and 512 padded tokens."""
    cfg = cfg_of(32, 128, 1100, ACT_SILU, chunks=2)
    inp = make_inputs(cfg, 512)
    check(cfg, gpu_backward(cfg, inp), oracle_backward(cfg, inp))
