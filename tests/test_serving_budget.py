"""What a served job needs at least, and what it gets under a budget (host code only)."""
import math

import pytest

from paper_1912_08810_amd import configs, serving, sse

P = configs.Problem
PROBS = [P(NA=400, NB=4, Norb=10, Nkz=5, Nqz=5, NE=400, Nw=25), P(NA=512, NB=4, Norb=10, Nkz=5, Nqz=5, NE=500, Nw=25),
         P(NA=30, NB=4, Norb=10, Nkz=3, Nqz=3, NE=41, Nw=9), P(NA=64, NB=4, Norb=25, Nkz=3, Nqz=3, NE=41, Nw=9)]
ZERO_PAGE = 256


@pytest.mark.parametrize("prob", PROBS)
def test_least_bytes_are_the_tensors_and_the_direct_kernels_workspace(prob):
    """Two G-shaped tensors per component, D~, dH, the tables; 2048 bytes of fragments per (atom,
    neighbour, q, eight frequencies) behind a page of zeros (sse_mfma.h: kZeroPage); one component's
    G again in bf16 halves; 512 for status words and alignment each."""
    g, d = prob.g_elems() * 16, prob.d_elems() * 16
    most = 2 * g + d + prob.NA * prob.NB * (3 * prob.NN * 8 + 4) + 1024 + ZERO_PAGE + sse.check_workspace_bytes(64, 2) + \
        prob.NA * prob.NB * prob.Nqz * math.ceil(prob.Nw / 8) * 2048 + prob.g_elems() * 8
    assert 2 * g + d < serving.job_bytes(prob) <= most


@pytest.mark.parametrize("prec", [sse.FP32, sse.BF16X3, sse.FP64C64])
def test_a_budget_below_the_spectral_workspace_gets_the_direct_one(prec):
    prob = PROBS[0]
    least = serving.job_bytes(prob)
    need, ws = serving.Server(prec=prec)._need(prob)
    assert need > least and ws >= sse.sse_plan(serving._desc(prob, prec, 2), prob.shifts()).workspace_bytes
    need, ws = serving.Server(prec=prec, budget_bytes=1.01 * least)._need(prob)
    assert need == least and ws >= sse.sse_plan(serving._desc(prob, prec, 2), prob.shifts()).direct_bytes
    assert ws < sse.sse_plan(serving._desc(prob, sse.FP64C64, 2), prob.shifts()).workspace_bytes


def test_fallback_is_another_kernel_than_the_form_that_missed():
    large, small = PROBS[0], PROBS[2]
    for prec in (sse.FP32, sse.BF16X3, sse.FP64C64):
        plan = sse.sse_plan(serving._desc(large, prec, 2), large.shifts())
        assert plan.spectral
        fb = serving._fallback_desc(large, plan, plan.workspace_bytes)
        assert fb.prec == sse.FP64C64 and not sse.sse_plan(fb, large.shifts()).spectral
        # in the direct form's workspace the fast plan runs that form, and the fallback is free
        assert serving._fallback_desc(large, plan, plan.direct_bytes).chunk_taps == 0
    plan = sse.sse_plan(serving._desc(small, sse.BF16X3, 2), small.shifts())
    assert not plan.spectral and serving._fallback_desc(small, plan, plan.workspace_bytes).chunk_taps == 0
