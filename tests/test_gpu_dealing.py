"""How the cells of a launch are dealt to its workgroups does not show: every
cell of a grid that takes several rounds of ranges gets the bits that it gets
in a small launch of its own, and nothing beyond the arrays is written."""
import pytest
import torch

from paper_2407_18304_amd import mgrhd, synth
from paper_2407_18304_amd import workloads as W

pytestmark = pytest.mark.gpu
KEYS = ("E_g", "F_g", "e_gas", "v")
PAD = 64


def _update(state, tables, kappa, consts, mode=mgrhd.MEAN_PPL_FIXED):
    n = kappa.numel()
    flat = {k: torch.full((state[k].numel() + PAD,), -7.0, dtype=torch.float64, device="cuda")
            for k in KEYS}
    out = tuple(flat[k][:state[k].numel()].view(state[k].shape) for k in KEYS)
    status = torch.full((n + PAD,), -7, dtype=torch.int32, device="cuda")
    mgrhd.source_update(state["E_g"], state["F_g"], state["rho"], state["e_gas"], state["v"],
                        tables["edges"], tables["chi_lo"], alpha_chi=tables["alpha"],
                        kappa_scale=kappa, polish=1, status=status[:n], out=out,
                        mean_mode=mode, **consts)
    assert all(bool((flat[k][-PAD:] == -7.0).all()) for k in KEYS)
    assert bool((status[-PAD:] == -7).all())
    return dict(zip(KEYS, out)), status[:n]


def _close(got, want, what):
    """The same arithmetic with sums in another order, or contracted otherwise:
    the parity bound of each value, or the rounding of the largest."""
    diff = (got - want).abs()
    err = diff / want.abs().clamp_min(1e-300)
    ok = (err < 1e-10) | (diff < 1e-14 * want.abs().max())
    assert bool(ok.all()), (*what, float(err.max()))


@pytest.fixture
def one_split():
    """The same split of a cell over lanes whatever the launch's size."""
    mgrhd.set_variant(64, 32, 2)
    yield
    mgrhd.set_variant(64, 0, 0)


# 64 groups: 16 cells in flight in a workgroup, up to 512 workgroups at once,
# so that several rounds begin beyond 4 x 32 x 512 cells (fewer where fewer
# workgroups fit); sizes at that edge, off any multiple, and a power of two
@pytest.mark.parametrize("n", [49151, 49153, 65535, 65536, 65537, 100003, 131072])
def test_rounds_of_ranges(n, one_split):
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


# patches whose groups fill their lanes (8, 64, 128), that leave lanes empty
# (1, 7, 65), cut by rounds (256), into single cells' worth of lanes (1) and
# across several items; a cap on the workgroups per CU down to one
@pytest.mark.parametrize("chunk", [1, 9, 256])
@pytest.mark.parametrize("blocks_per_cu", [0, 1, 2, 3])
def test_items_of_a_workgroup(chunk, blocks_per_cu):
    sizes = ((64, 700), (1, 300), (8, 513), (65, 70), (7, 1), (128, 33), (3, 2000))
    layouts, cell0 = [], 0
    for p, (ng, n) in enumerate(sizes):
        edges = W.log_edges(1e-3, 1e3, ng)
        layouts.append(W.PatchLayout(p, n, ng, cell0, edges, edges[:-1] ** -2.0,
                                     torch.full((ng,), -2.0).double().numpy()))
        cell0 += n
    dps = synth.device_patches(layouts)
    patches = []
    for dp in dps:
        out = tuple(torch.full_like(dp.state[k], float("nan")) for k in KEYS)
        patches.append(dict(dp.state, edges=dp.tables["edges"], chi_lo=dp.tables["chi_lo"],
                            alpha_chi=dp.tables["alpha"], kappa_scale=dp.kappa, dt=dp.dt,
                            c_hat=dp.c_hat, out=out,
                            status=torch.full((dp.layout.n,), -7, dtype=torch.int32,
                                              device="cuda")))
    b = mgrhd.Batch(patches, polish=1, c_v=1.5, **W.UNITS["patches"])
    b.set_tuning(2, blocks_per_cu, chunk)
    b.run()
    torch.cuda.synchronize()
    for dp, q in zip(dps, patches):
        want, status = _update(dp.state, dp.tables, dp.kappa,
                               {k: v for k, v in dp.consts().items()})
        assert torch.equal(q["status"], status)
        for k, got in zip(KEYS, q["out"]):
            _close(got, want[k], (dp.layout.ng, k))


# launches around the sizes at which a cell's groups are split over more lanes
# (one and a half, one and three quarters, and two times the lanes that 256
# compute units hold;
# PPL-free three and a half times), and of a few cells, against a split set for
# every size: groups that fill the lanes and that do not
@pytest.mark.parametrize("ng,split,n,mode", [
    (4, (2, 2), 114688, 1), (4, (2, 2), 114689, 1), (16, (8, 2), 24576, 0),
    (16, (8, 2), 24577, 0), (64, (32, 2), 7168, 1), (64, (32, 2), 7169, 1), (3, (2, 2), 7, 1),
    (1, (1, 4), 1, 1), (2, (1, 4), 130, 0), (33, (32, 2), 8192, 1), (33, (32, 2), 8193, 1),
    (64, (32, 2), 14336, 2), (64, (32, 2), 14337, 2), (23, (16, 2), 5000, 2),
    (16, (8, 2), 255, 1), (16, (8, 2), 257, 1), (64, (32, 2), 4097, 0)])
def test_split_of_a_small_launch(ng, split, n, mode):
    edges = W.log_edges(1e-3, 1e3, ng)
    layout = W.PatchLayout(0, n, ng, 0, edges, edges[:-1] ** -2.0,
                           torch.full((ng,), -2.0).double().numpy())
    dp, = synth.device_patches([layout])
    got, st = _update(dp.state, dp.tables, dp.kappa, dp.consts(), mode)
    mgrhd.set_variant(ng, *split)
    try:
        want, want_st = _update(dp.state, dp.tables, dp.kappa, dp.consts(), mode)
    finally:
        mgrhd.set_variant(ng, 0, 0)
    assert torch.equal(st, want_st)
    for k in KEYS:
        _close(got[k], want[k], (ng, n, k))


def _all(state, tables, kappa, consts, mode):
    """Every output of an update of this state."""
    n = kappa.numel()
    out = tuple(torch.empty_like(state[k]) for k in KEYS)
    counts = {k: torch.full((n,), -7, dtype=torch.int32, device="cuda")
              for k in ("iters", "outer", "status")}
    mgrhd.source_update(state["E_g"], state["F_g"], state["rho"], state["e_gas"], state["v"],
                        tables["edges"], tables["chi_lo"], alpha_chi=tables["alpha"],
                        kappa_scale=kappa, polish=1, out=out, mean_mode=mode, **counts, **consts)
    return dict(zip(KEYS, out), **counts)


def _cells(ng, n, td):
    edges = W.log_edges(1e-3, 1e3, ng)
    dp, = synth.device_patches([W.PatchLayout(0, n, ng, 0, edges, edges[:-1] ** -2.0,
                                              torch.full((ng,), -2.0).double().numpy())])
    more = dict(t_exp=-0.5, t_ref=0.8, stim=1) if td else {}
    return dp.state, dp.tables, dp.kappa, dict(dp.consts(), **more)


# groups that fill the lanes of both splits and that do not, every lane count
# of one group per lane (4 to 64)
@pytest.mark.parametrize("td", [False, True])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("ng", [1, 2, 3, 4, 5, 8, 11, 16, 17, 32, 33, 64])
def test_both_splits_give_the_same_bits(ng, mode, td):
    """One group per lane and the split that larger launches take: every
    output of every cell equal bit for bit."""
    args = _cells(ng, 4096, td)
    one = 4
    while one < ng:
        one *= 2
    many = (1, 4) if ng <= 2 else (one // 2, 2)
    got = []
    try:
        for lanes, groups in ((one, 1), many):
            mgrhd.set_variant(ng, lanes, groups)
            got.append(_all(*args, mode))
    finally:
        mgrhd.set_variant(ng, 0, 0)
    for k in got[0]:
        assert torch.equal(got[0][k], got[1][k]), (k, int((got[0][k] != got[1][k]).sum()))


@pytest.mark.parametrize("ng,n,mode,td", [(4, 131072, 1, False), (16, 32768, 0, False),
                                          (64, 16384, 2, False), (11, 40000, 1, False),
                                          (16, 24576, 1, True)])
def test_a_grid_in_pieces_gives_its_bits(ng, n, mode, td):
    """A grid whose launch takes two groups per lane, and the same cells in
    launches small enough for one."""
    state, tables, kappa, consts = _cells(ng, n, td)
    whole = _all(state, tables, kappa, consts, mode)
    step = n // 16 + 3
    for i in range(0, n, step):
        at = slice(i, min(n, i + step))
        part = {k: v[..., at].contiguous() for k, v in state.items()}
        got = _all(part, tables, kappa[at].contiguous(), consts, mode)
        for k in got:
            assert torch.equal(got[k], whole[k][..., at]), (k, i)


@pytest.mark.parametrize("td", [False, True])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_every_variant_against_one_group_per_lane(mode, td):
    """Every compiled split and register budget, at groups that fill its lanes
    and at one fewer, twice: the same bits each time, and the cells of one
    group per lane (which holds the fewest registers)."""
    for lanes, groups, waves in mgrhd.variants():
        for ng in {lanes * groups, max(lanes * groups - 1, 1)}:
            if ng > 64:
                continue
            args = _cells(ng, 1500, td)
            one = 4
            while one < ng:
                one *= 2
            got = []
            try:
                for v in ((lanes, groups, waves), (lanes, groups, waves), (one, 1, 0)):
                    mgrhd.set_variant(ng, *v)
                    got.append(_all(*args, mode))
            finally:
                mgrhd.set_variant(ng, 0, 0)
            what = (lanes, groups, waves, ng)
            for k in got[0]:
                assert torch.equal(got[0][k], got[1][k]), (*what, k)
            assert torch.equal(got[0]["status"], got[2]["status"]), what
            for k in KEYS:
                _close(got[0][k], got[2][k], (*what, k))
