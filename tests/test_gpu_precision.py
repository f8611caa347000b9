"""What is held in fp32 stays in fp32 in the fixed-size bf16 kernels.

The runtime-sized kernels keep every intermediate that is no operand of a matrix
product in fp32.  A fixed-size kernel that rounds at the same places differs from
them by the order of its sums alone, and by the operands that such a difference
takes over a rounding boundary.  The initial W1 is scaled up, so that the
activations leave their linear range and an extra rounding of their argument shows.
"""
import pytest
import torch

from paper_2511_07343_amd import tnt
from paper_2511_07343_amd.inputs import ACT_GELU, ACT_SILU, BF16, make_inputs, small_config
from test_gpu_backward import oracle_backward

pytestmark = pytest.mark.gpu
torch.set_num_threads(4)


def both_families(cfg, inp, final_state):
    """Outputs and gradients of the default kernels and of the runtime-sized ones."""
    res = []
    for family in (tnt.FAMILY_DEFAULT, tnt.FAMILY_GENERIC):
        with tnt.kernel_family(family):
            x = tnt.device_inputs(inp, cfg)
            o, saved, fin = tnt.forward(cfg, x, save=True, final_state=final_state)
            g = tnt.backward(cfg, x, x["dO"], saved=saved)
            torch.cuda.synchronize()
        res.append({k: v.double().cpu() for k, v in dict(o=o, final=fin, **g).items()
                    if v is not None})
    return res


@pytest.mark.parametrize("d,hid", [(64, 256), (128, 512), (64, 128), (32, 128)])
@pytest.mark.parametrize("act", [ACT_SILU, ACT_GELU])
def test_global_activation_argument(d, hid, act):
    cfg = small_config(BF16, act, B=1, H=2, L=300, d=d, hid=hid, C_G=100, locals_=(),
                       name=f"global d{d} h{hid} act={act}")
    inp = make_inputs(cfg, 711)
    inp.W1 *= 20.0
    print(f"\n[case] {cfg.name}", flush=True)
    a, b = both_families(cfg, inp, True)
    # o, the final state and dq pass through the same roundings in both families: only
    # flipped ones are left.  dv passes through one operand more that may differ; an
    # operand rounded to bf16 is off by 2^-9 / sqrt(3) of itself in the mean.
    for n, bound in (("o", 1e-4), ("final", 1e-4), ("dq", 1e-4), ("dv", 2.0 ** -9 / 3 ** 0.5)):
        e = float((a[n] - b[n]).norm() / b[n].norm())
        print(f"  {n:7s} {e:.2e}", flush=True)
        assert e <= bound, (n, e)


@pytest.mark.parametrize("act,C", [(ACT_GELU, 16), (ACT_GELU, 32), (ACT_SILU, 33), (ACT_GELU, 48)])
def test_local_roundings(act, C):
    """The error against 64 bits is that of the runtime-sized kernels: operands scaled by a
    gate coefficient are rounded once, after the scaling.  1 %: the two families' errors
    differ by the elements that their sums' order takes over a rounding boundary; one
    operand in ten rounded twice adds 2 to 9 %.  And the adjoint . state products behind the
    gate gradients are taken from fp32 values."""
    cfg = small_config(BF16, act, B=1, H=4, L=32 * C, d=64, hid=256, C_G=32 * C,
                       locals_=((C, 16 * C),), name=f"local C_L={C} act={act}")
    inp = make_inputs(cfg, 712)
    print(f"\n[case] {cfg.name}", flush=True)
    a, b = both_families(cfg, inp, False)
    ref = {k: torch.from_numpy(v) for k, v in oracle_backward(cfg, inp).items()}
    bad = []
    for n in ("dv", "dW1"):
        ea, eb = float((a[n] - ref[n]).norm()), float((b[n] - ref[n]).norm())
        print(f"  {n:7s} {ea / float(ref[n].norm()):.3e} / {eb / float(ref[n].norm()):.3e} = {ea / eb:.3f}",
              flush=True)
        if ea > 1.01 * eb:
            bad.append((n, ea / eb))
    # the gate gradients: half of what one more rounding to bf16 would add (2^-9 / sqrt(3)),
    # of the adjoint or of the state, in the sums of adjoint . state products
    for n in ("dlr", "dmom", "ddecay"):
        e = float((a[n] - b[n]).norm() / b[n].norm())
        print(f"  {n:7s} apart {e:.2e}", flush=True)
        if e > 0.5 * 2.0 ** -9 / 3 ** 0.5:
            bad.append((n, e))
    assert not bad, bad
