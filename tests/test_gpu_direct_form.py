"""The direct kernels where a default plan takes the spectral form, which they stand behind
(values that are not finite, outputs far below their energy block, small workspaces): general
and anti-Hermitian D~, one-shot, persistent and behind the transforms, at tiles, windows and
counts where they can go wrong.  A chunk cap that cuts nothing asks for them.

Bars of the other suites: binary64 1e-12 (relative Frobenius), 1e-7 where the result is stored as
complex64, fp32 products 1e-5, bf16 hi/lo products 1e-3."""
import numpy as np
import pytest

from paper_1912_08810_amd import configs
from tests import gpu_util as gu
from tests.test_gpu_graded import _host, _problem, _worst

pytestmark = pytest.mark.gpu
P = configs.Problem
TOL = {0: 1e-12, 1: 1e-5, 2: 1e-3, 3: 1e-7}

CASES = {
    "small": configs.SMALL,
    "ragged": P(NA=37, NB=5, Norb=10, Nkz=4, Nqz=3, NE=47, Nw=7, shift=(3, 1, -2, 7, 5, 2, 4)),
    "many_chunks": P(NA=6, NB=3, Norb=10, Nkz=2, Nqz=2, NE=40, Nw=9, shift=(0, 8, 16, 24, 32, 39, -8, -16, -39)),
    "taps_128": P(NA=6, NB=2, Norb=4, Nkz=2, Nqz=2, NE=150, Nw=128),
    "neighbours_50": P(NA=51, NB=50, Norb=4, Nkz=2, Nqz=2, NE=12, Nw=3),
    "odd_rows": P(NA=9, NB=3, Norb=5, Nkz=3, Nqz=3, NE=83, Nw=11),
}


def _desc(p, prec, ncomp, ah, direct):
    from paper_1912_08810_amd import sse
    d = sse.make_desc(p.NA, p.NB, p.Norb, p.Nkz, p.Nqz, p.NE, p.Nw, ncomp=ncomp, prec=prec, dt_antiherm=ah)
    return sse.direct_desc(d) if direct else d


def _run(dps, prec, ah, direct, batch):
    """One submission of all problems, or one of each; the forms are checked."""
    import torch
    from paper_1912_08810_amd import sse
    items = [(d.neigh, d.dH, d.G, d.D, d.Sigma) for d in dps]
    descs = [_desc(d.prob, prec, d.ncomp, ah, direct) for d in dps]
    shifts = [d.prob.shifts() for d in dps]
    for d, s in zip(descs, shifts):
        assert sse.sse_plan(d, s).spectral != direct
    stream = torch.cuda.current_stream()
    if batch:
        plan = sse.sse_plan_batch(descs, shifts)
        ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
        sse.sse_wait(sse.sse_submit(plan, items, ws, stream))
        return
    for d, s, it in zip(descs, shifts, items):
        plan = sse.sse_plan(d, s)
        ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
        sse.sse_wait(sse.sse_submit(plan, [it], ws, stream))


def _bits(x):
    import torch
    x = x.view(torch.int64 if x.dtype == torch.float64 else torch.int32)
    return x


@pytest.mark.parametrize("ah", [0, 1], ids=["general", "antiherm"])
@pytest.mark.parametrize("prec", [0, 3])
@pytest.mark.parametrize("name", CASES)
def test_binary64_kernels_match_oracle(name, prec, ah):
    prob = CASES[name]
    dp = gu.DeviceProblem(prob, 610 + len(name), ncomp=2, fp32=prec != 0)
    _run([dp], prec, ah, True, False)
    for c in range(2):
        e = gu.rel_fro(dp.sigma_host(c), gu.oracle_full(dp, c))
        print(f"  {name} prec {prec} ah {ah} comp {c}: rel_fro={e:.3e}", flush=True)
        assert e <= TOL[prec]
    one = dp.Sigma.clone()
    dp.Sigma.fill_(7.0)
    _run([dp], prec, ah, True, True)
    import torch
    assert torch.equal(_bits(one), _bits(dp.Sigma))   # the persistent kernel


@pytest.mark.parametrize("prec", [1, 2])
def test_matrix_core_kernels_above_the_spectral_threshold(prec):
    prob = P(NA=100, NB=4, Norb=10, Nkz=5, Nqz=5, NE=200, Nw=20)
    dp = gu.DeviceProblem(prob, 630, fp32=True, scaled=True)
    _run([dp], prec, 0, True, False)
    blocks = gu.sample_blocks(prob, 3, n_e=8, n_a=4)
    assert gu.rel_fro(dp.device_blocks(0, blocks), gu.oracle_blocks(dp, 0, blocks)) <= TOL[prec]


BEHIND = [P(NA=11, NB=4, Norb=10, Nkz=3, Nqz=3, NE=41, Nw=6), P(NA=9, NB=3, Norb=5, Nkz=3, Nqz=2, NE=83, Nw=11),
          P(NA=70, NB=4, Norb=4, Nkz=3, Nqz=3, NE=64, Nw=4)]


@pytest.mark.parametrize("batch", [False, True], ids=["single", "batch"])
@pytest.mark.parametrize("ah", [0, 1], ids=["general", "antiherm"])
@pytest.mark.parametrize("prec", [0, 3])
def test_not_finite_behind_the_spectral_form(prec, ah, batch):
    """Infinities and NaN: the bits of the direct launch, the anti-Hermitian kernels among them."""
    import torch
    probs = [p for p in BEHIND if p.Norb == 10] if batch else BEHIND
    probs = probs + [P(NA=7, NB=4, Norb=10, Nkz=3, Nqz=3, NE=60, Nw=10)]
    dps = [gu.DeviceProblem(p, 640 + i, ncomp=2, fp32=prec != 0) for i, p in enumerate(probs)]
    for d in dps[:-1]:
        G = d.G.view(-1)
        G[G.numel() // 3], G[G.numel() // 5] = float("inf"), float("nan")
    _run(dps, prec, ah, False, batch)
    got = [d.Sigma.clone() for d in dps]
    _run(dps, prec, ah, True, False)
    for i, (d, g) in enumerate(zip(dps, got)):
        if i < len(dps) - 1:
            assert torch.isnan(d.Sigma).any() and not torch.isnan(d.Sigma).all()
            same = torch.isnan(g) & torch.isnan(d.Sigma) | (_bits(g) == _bits(d.Sigma))
            assert bool(same.all()), i
        else:   # finite: left alone by the others' recovery
            assert gu.rel_fro(d.sigma_host(1), gu.oracle_full(d, 1)) <= TOL[prec]


@pytest.mark.parametrize("batch", [False, True], ids=["single", "batch"])
@pytest.mark.parametrize("prec", [0, 3])
def test_graded_antihermitian_behind_the_spectral_form(prec, batch):
    import oracle
    probs = BEHIND[:1] + [P(NA=7, NB=4, Norb=10, Nkz=3, Nqz=3, NE=60, Nw=10)] if batch else BEHIND
    dps = [_problem(p, "decay_1" if prec == 0 else "step", 660 + i, prec, ncomp=2) for i, p in enumerate(probs)]
    _run(dps, prec, 1, False, batch)
    for d in dps:
        for c in range(2):
            dH, G, D = _host(d, "decay_1" if prec == 0 else "step", c)
            want = oracle.sigma(d.neigh_h, dH, G, D, d.prob.shifts(), d.prob.Nkz, d.prob.NE)
            assert _worst(d.sigma_host(c), want, 3) <= (6e-14 if prec == 0 else 1.2e-7)


@pytest.mark.parametrize("name", ["flat", "step"])
def test_workspace_of_some_atoms_at_a_time_in_the_row_form(name):
    """Three passes of atoms (425 of 900 at most: tests/host_runtime/spectral_limits_check.cpp holds
    the geometry to it), the last one ragged; a step in G has every pass look at its outputs."""
    prob = P(NA=900, NB=4, Norb=16, Nkz=9, Nqz=9, NE=140, Nw=20)
    dp = _problem(prob, name, 680, 0)
    assert gu.run_sse(dp) == 0
    blocks = gu.sample_blocks(prob, 6, n_e=6, n_a=3)
    blocks = np.array([b for b in blocks if b[0] in (0, 4, 8)] + [(3, 69, 424), (3, 70, 425), (5, 71, 849), (5, 139, 850)],
                      dtype=np.int32)
    import oracle
    dH, G, D = _host(dp, name, 0)
    want = oracle.sigma(dp.neigh_h, dH, G, D, prob.shifts(), prob.Nkz, prob.NE, blocks=blocks)
    e = _worst(np.asarray(dp.device_blocks(0, blocks)), np.asarray(want), 1)
    print(f"  {name}: worst block {e:.3e}", flush=True)
    assert e <= 6e-14
