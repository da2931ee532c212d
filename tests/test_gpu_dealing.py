"""How the cells of a launch are dealt to its workgroups does not show: every
cell of a grid that takes several rounds of ranges gets the bits that it gets
in a small launch of its own, and nothing beyond the arrays is written."""
import pytest
import torch

from paper_2407_18304_amd import mgrhd, synth

pytestmark = pytest.mark.gpu
KEYS = ("E_g", "F_g", "e_gas", "v")
PAD = 64


def _update(state, tables, kappa, consts):
    n = kappa.numel()
    flat = {k: torch.full((state[k].numel() + PAD,), -7.0, dtype=torch.float64, device="cuda")
            for k in KEYS}
    out = tuple(flat[k][:state[k].numel()].view(state[k].shape) for k in KEYS)
    status = torch.full((n + PAD,), -7, dtype=torch.int32, device="cuda")
    mgrhd.source_update(state["E_g"], state["F_g"], state["rho"], state["e_gas"], state["v"],
                        tables["edges"], tables["chi_lo"], alpha_chi=tables["alpha"],
                        kappa_scale=kappa, polish=1, status=status[:n], out=out, **consts)
    assert all(bool((flat[k][-PAD:] == -7.0).all()) for k in KEYS)
    assert bool((status[-PAD:] == -7).all())
    return dict(zip(KEYS, out)), status[:n]


# 64 groups: 8 cells in flight in a workgroup, up to 1024 workgroups at once,
# so that several rounds begin beyond 4 x 16 x 1024 cells (fewer where fewer
# workgroups fit); sizes at that edge, off any multiple, and a power of two
@pytest.mark.parametrize("n", [49151, 49153, 65535, 65536, 65537, 100003, 131072])
def test_rounds_of_ranges(n):
    dw = synth.device_workload("config2", n=n)
    whole, status = _update(dw.state, dw.tables, dw.kappa, dw.consts())
    step = 8191
    for i in range(0, n, step):
        at = slice(i, min(n, i + step))
        part = {k: dw.state[k][..., at].contiguous() for k in KEYS + ("rho",)}
        got, st = _update(part, dw.tables, dw.kappa[at].contiguous(), dw.consts())
        for k in KEYS:
            assert torch.equal(got[k], whole[k][..., at]), (k, i)
        assert torch.equal(st, status[at])
