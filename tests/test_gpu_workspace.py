"""Workspaces of the direct kernels' size, through the Python binding: accepted, and the
result is the direct form's, bit for bit; the bytes behind the buffer stay as they were."""
import pytest

from paper_1912_08810_amd import configs
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
P = configs.Problem
PROBS = [P(NA=11, NB=4, Norb=10, Nkz=3, Nqz=3, NE=41, Nw=6), P(NA=7, NB=4, Norb=10, Nkz=3, Nqz=3, NE=60, Nw=10)]


def _desc(p, prec, **kw):
    from paper_1912_08810_amd import sse
    return sse.make_desc(p.NA, p.NB, p.Norb, p.Nkz, p.Nqz, p.NE, p.Nw, prec=prec, **kw)


@pytest.mark.parametrize("prec", [0, 3])
@pytest.mark.parametrize("batch", [False, True], ids=["single", "batch"])
def test_small_workspace_runs_the_direct_form(prec, batch):
    import torch
    from paper_1912_08810_amd import sse
    probs = PROBS if batch else PROBS[:1]
    dps = [gu.DeviceProblem(p, 300 + i, fp32=prec != 0) for i, p in enumerate(probs)]
    items = [(d.neigh, d.dH, d.G, d.D, d.Sigma) for d in dps]
    shifts = [p.shifts() for p in probs]

    def run(nbytes, **kw):
        descs = [_desc(p, prec, **kw) for p in probs]
        plan = sse.sse_plan_batch(descs, shifts) if batch else sse.sse_plan(descs[0], shifts[0])
        assert nbytes is None or nbytes < plan.workspace_bytes
        guard = torch.full(((nbytes or plan.workspace_bytes) + 65536,), 7, dtype=torch.uint8, device="cuda")
        ws = guard[:nbytes or plan.workspace_bytes]
        sse.sse_wait(sse.sse_submit(plan, items, ws, torch.cuda.current_stream()))
        assert bool((guard[ws.numel():] == 7).all())
        return plan, [d.Sigma.clone() for d in dps]

    direct, want = run(None, chunk_taps=128)
    plan, got = run(direct.direct_bytes)
    assert plan.direct_bytes == direct.direct_bytes
    for g, w in zip(got, want):
        assert torch.equal(g.view(torch.int32), w.view(torch.int32))


def test_workspace_behind_a_word_gives_the_same_bits():
    """A workspace that starts four bytes behind an aligned one: Sigma and Pi."""
    import torch
    from paper_1912_08810_amd import sse
    p = PROBS[0]
    dp = gu.DeviceProblem(p, 310, ncomp=2)
    plan = sse.sse_plan(_desc(p, 0, ncomp=2), p.shifts())
    assert plan.workspace_bytes > plan.direct_bytes
    got = []
    for off in (0, 4):
        ws = torch.empty(plan.workspace_bytes + 4, dtype=torch.uint8, device="cuda")[off:off + plan.workspace_bytes]
        Pi = torch.zeros(2, sse.pi_elems(plan.descs[0]) * 2, dtype=torch.float64, device="cuda")
        sse.sse_compute(plan, dp.neigh, dp.dH, dp.G, dp.D, dp.Sigma, ws, torch.cuda.current_stream())
        sse.sse_pi_compute(plan, dp.neigh, dp.dH, dp.G, Pi, ws, torch.cuda.current_stream())
        got.append((dp.Sigma.clone(), Pi))
    for x, y in zip(*got):
        assert torch.equal(x.view(torch.int64), y.view(torch.int64))


def test_served_job_with_room_for_the_direct_workspace_alone():
    """A budget between a job's least and what its plans ask for: admitted, and checked."""
    from paper_1912_08810_amd import serving, sse
    prob = P(NA=100, NB=4, Norb=10, Nkz=5, Nqz=5, NE=200, Nw=20)
    job = serving.make_jobs([prob], rate=1e6, seed=33, iterations=2)[0]
    least = serving.job_bytes(prob)
    assert serving.Server()._need(prob)[0] > 1.01 * least
    srv = serving.Server(slots=1, budget_bytes=1.01 * least)
    res = srv.run([job])
    assert res[0].status == sse.OK and 0 < res[0].max_check_err <= 1e-5


def test_a_miss_of_the_spectral_form_is_recomputed_by_the_direct_kernel():
    """Sigma of the fallback against the same job's direct binary64 result, bit for bit."""
    import torch
    from paper_1912_08810_amd import serving, sse
    prob = P(NA=100, NB=4, Norb=10, Nkz=5, Nqz=5, NE=200, Nw=20)
    assert sse.sse_plan(serving._desc(prob, sse.BF16X3, 2), prob.shifts()).spectral
    job = serving.make_jobs([prob], rate=1e6, seed=35, iterations=1)[0]
    srv = serving.Server(slots=1, tol=1e-12, keep_results=True)   # below the storage's rounding
    res = srv.run([job])
    assert res[0].status == sse.ERR_TOLERANCE and res[0].fallbacks == 1
    dp = gu.DeviceProblem(prob, job.seed, ncomp=2, fp32=True)
    for direct in (True, False):
        desc = serving._desc(prob, sse.FP64C64, 2)
        plan = sse.sse_plan(sse.direct_desc(desc) if direct else desc, prob.shifts())
        ws = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device="cuda")
        sse.sse_compute(plan, dp.neigh, dp.dH, dp.G, dp.D, dp.Sigma, ws, torch.cuda.current_stream())
        assert torch.equal(srv.sigma[job.jid].view(torch.int32), dp.Sigma.cpu().view(torch.int32)) == direct
