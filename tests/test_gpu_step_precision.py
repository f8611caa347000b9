"""fp32 precision of the step-wise forward: the products at the entry weights are sums of
matrix instructions, and their error against 64 bits is that of lane sums of vector
products, as a tree's is and one accumulator's is not; the momentum is rounded once."""
import pytest
import torch

import oracle as O
from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import ACT_SILU, F32, make_inputs, small_config

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


def errors(d, hid, T=12):
    """Relative 2-norm errors of o and of the global memory's momentum after T tokens."""
    cfg = small_config(F32, ACT_SILU, B=1, H=4, L=T, d=d, hid=hid, C_G=T, locals_=((T, T),),
                       name=f"step precision d{d} h{hid}")
    inp = make_inputs(cfg, 541)
    x = tnt.device_inputs(inp, cfg)
    o, state = tnt.step_forward(cfg, x, [T])
    torch.cuda.synchronize()
    pairs = O.all_pairs(cfg)
    ref, fin = O.forward_pairs(inp, cfg, pairs, with_final=True)
    hd, n = cfg.hid * cfg.d, len(pairs)
    st = state[: n * (6 * hd + cfg.d ** 2) * 4].view(torch.float32).view(n, -1).double().cpu()
    S = torch.cat([f.reshape(n, -1) for f in fin[2:]], 1).double()
    rel = lambda a, b: float((a - b).norm() / b.norm())
    return rel(o.double().cpu().reshape(-1), ref.double().reshape(-1)), rel(st[:, 4 * hd: 6 * hd], S)


@pytest.mark.parametrize("d,hid", [(16, 32), (32, 128), (64, 128), (64, 256), (128, 128), (128, 512)])
def test_step_fp32_error(d, hid):
    """u = 2^-24.  o: 1.3 to 1.7e-7 as with lane sums, 1.9 to 4.5e-7 with one accumulator a
    product (d 32 and more); momentum: 1.1 to 1.3e-7, 1.4 to 2.2e-7 where its old value is
    rounded once more.  The bounds lie between the two."""
    eo, eS = errors(d, hid)
    print(f"\n[case] d{d} h{hid}: o {eo:.3e} momentum {eS:.3e}", flush=True)
    u = 2.0 ** -24
    assert eo <= 3.0 * u and eS <= 2.2 * u
