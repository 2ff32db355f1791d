"""Grouped products of more groups than a launch has room for (2^32 threads),
and the argument checks of groups without outputs.

Millions of groups of one 1 x 1 block: every output is one product added to
what was there, exact in FP64 to a rounding."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("groups", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1, (1 << 22) + 3])
def test_many_groups(trans, groups):
    import torch
    import paper_1510_07244_amd as pk
    ar = lambda n: torch.arange(n, dtype=torch.int32, device="cuda")
    a_off = torch.arange(groups, dtype=torch.int64, device="cuda")
    A = torch.linspace(1.0, 2.0, groups, dtype=torch.float64, device="cuda")
    x = torch.linspace(-1.0, 3.0, groups, dtype=torch.float64, device="cuda")
    y = torch.ones(groups, dtype=torch.float64, device="cuda")
    ctx = pk.Context(0)
    ctx.gemv_grouped(trans, ar(groups + 1), ar(groups + 1), ar(groups), ar(groups + 1), ar(groups), a_off, A, x, y)
    ctx.check()
    ctx.close()
    assert ((y - (1.0 + A * x)).abs() <= 4e-16 * (1.0 + (A * x).abs())).all()


# one group: no outputs, one block of three inputs
@pytest.mark.parametrize("fault", ["", "input", "offset", "range"])
def test_group_without_outputs_is_checked(fault):
    import torch
    import paper_1510_07244_amd as pk
    i32 = lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda")
    x = torch.ones(8, dtype=torch.float64, device="cuda")
    y = torch.full((4,), 7.0, dtype=torch.float64, device="cuda")
    ctx = pk.Context(0)
    ctx.gemv_grouped(False, i32(0, 1), i32(0, 0), i32(1), i32(0, 5 if fault == "range" else 3),
                     i32(0, 8 if fault == "input" else 1, 2),
                     torch.tensor([9 if fault == "offset" else 0], dtype=torch.int64, device="cuda"), x.clone(), x, y)
    if fault:
        with pytest.raises(pk.BemError):
            ctx.check()
    else:
        ctx.check()
    assert (y == 7.0).all()
    ctx.close()
