"""Temperature-dependent opacities on the GPU (mgrhd_source_update with
t_exp / t_ref / stim): parity with the oracle in every mean mode and lane
split, the Planck-equilibrium invariant, the full-size pulse-opacity
workload on sampled cells, and the argument checks.  GPU only."""
import math

import numpy as np
import pytest
import torch

from paper_2407_18304_amd import mgrhd
from paper_2407_18304_amd import workloads as W

import gpu_util as U
import oracle

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _check(w, mode, **kw):
    return U.compare(w, U.run_gpu(w, mode, **kw), U.run_oracle(w, mode, **kw),
                     label=f"T-dependent mode {mode}")


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_pulse_opacity_parity(mode):
    """eq. pulsek: nu^-3, (T/T_ref)^-1/2 and the stimulated-emission factor."""
    rng = np.random.default_rng(21)
    w = W.config5(cells=np.sort(rng.choice(128 ** 3, 6000, replace=False)))
    assert w.stim == 1 and w.t_exp == -0.5
    _check(w, mode)


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_temperature_power_parity(mode):
    """(T/T_ref)^(3/2) on the config-1 table (Sec. 4.1.2 simulation (c))."""
    w = W.config1(cells=np.arange(4000))
    w.t_exp, w.t_ref = 1.5, 0.8
    _check(w, mode)


@pytest.mark.parametrize("ng", [1, 5, 33])
def test_ragged_groups_with_temperature_dependence(ng):
    w = W.config1(cells=np.arange(700), ng=ng)
    w.t_exp, w.stim = -0.5, 1
    _check(w, 1)
    _check(w, 2)


def test_lane_splits_agree():
    w = W.config5(cells=np.arange(3000))
    ref = U.run_gpu(w, 1)
    try:
        for lpc, gpl, wps in [(8, 2, 0), (16, 1, 0), (4, 4, 0), (32, 1, 0), (8, 2, 4)]:
            mgrhd.set_variant(w.ng, lpc, gpl, wps)
            U.compare(w, U.run_gpu(w, 1), ref, label=f"variant {lpc}x{gpl}x{wps}")
    finally:
        mgrhd.set_variant(w.ng, 0, 0)


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_planck_equilibrium_is_stationary(mode):
    """v = F = 0 and E_g = a T^4 p_g(T): nothing changes, whatever chi(T)."""
    w = W.config5(cells=np.arange(256))
    T = w.T
    E = np.zeros((w.ng, w.n))
    for i in range(w.n):                # group Planck energies of the oracle
        for g in range(w.ng):
            b, elo, ehi, sg = oracle.group_planck(w.edges[g] / T[i], w.edges[g + 1] / T[i])
            E[g, i] = w.a_rad * T[i] ** 4 * b * math.exp(-sg)
    w.state = {"E_g": E, "F_g": np.zeros((3, w.ng, w.n)), "rho": np.ones(w.n),
               "e_gas": 1.5 * T, "v": np.zeros((3, w.n))}
    g, gi, go, gs = U.run_gpu(w, mode)
    assert (gs == 0).all()
    # the kernels' group integrals agree with the oracle's to ~1e-15, so E_g
    # is an equilibrium to that order: R_g and the temperature change are tiny
    assert np.allclose(g["E_g"], E, rtol=1e-12, atol=1e-300)
    assert np.allclose(g["e_gas"], 1.5 * T, rtol=1e-13)


def test_pulse_full_size_sampled():
    """The whole 128^3 pulse-opacity workload, drawn on the device and solved in
    the launch configuration of the benchmark; 400 cells checked against the
    oracle on the same inputs, which the host generator reproduces."""
    idx, host = U.full_size_sampled("config5", 1, 400, seed=5)
    ref = W.config5(cells=idx)
    for k in U.FIELDS:   # the device and host generators agree to rounding
        assert np.allclose(host.state[k], ref.state[k], rtol=1e-11, atol=0), k


def test_temperature_argument_errors():
    w = W.config0(cells=np.arange(10))
    w.t_exp, w.t_ref = 1.5, 0.0
    with pytest.raises(mgrhd.MgrhdError) as e:
        U.run_gpu(w, 1)
    assert e.value.code == mgrhd.E_TABLE
    w.t_exp, w.t_ref, w.stim = 0.0, 1.0, 2
    with pytest.raises(mgrhd.MgrhdError):
        U.run_gpu(w, 1)
    # stim with a zero lower edge: rejected per cell on the device
    w.stim = 1
    w.edges = np.concatenate([[0.0], w.edges[1:]])
    g, gi, go, gs = U.run_gpu(w, 0)
    assert (gs == mgrhd.ST_BAD_TABLE).all()
    for k in U.FIELDS:
        assert np.array_equal(g[k], w.state[k])


# every split of two groups per lane that the groups fill, the largest of them
# the one that holds the most registers
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("ng,waves", [(4, 0), (8, 0), (16, 0), (16, 4), (32, 0), (64, 0), (64, 4)])
def test_groups_that_fill_two_per_lane(ng, waves, mode):
    """(T/T_ref)^(-1/2) with the stimulated-emission factor: parity with the
    oracle, and the same bits in a second run."""
    w = W.config1(cells=np.arange(1500), ng=ng)
    w.t_exp, w.t_ref, w.stim = -0.5, 0.8, 1
    try:
        mgrhd.set_variant(ng, ng // 2, 2, waves)
        first = U.run_gpu(w, mode)
        again = U.run_gpu(w, mode)
    finally:
        mgrhd.set_variant(ng, 0, 0)
    U.compare(w, first, U.run_oracle(w, mode), label=f"{ng} groups, mode {mode}")
    for k, v in first[0].items():
        assert np.array_equal(v, again[0][k]), k
