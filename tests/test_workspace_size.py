"""The size that the binding declares for a caller's workspace is the buffer's own, never the
plan's: a binary64 plan asks for gigabytes and takes 256 bytes.  The library's calls are
replaced by a recorder; nothing here touches a GPU."""
import numpy as np
import pytest
import torch

from paper_1912_08810_amd import sse


class Recorder:
    """Stands for the loaded library: plans are the real ones, submissions are noted."""

    def __init__(self, lib):
        self._lib, self.declared = lib, []

    def __getattr__(self, name):
        if name in ("sse_compute", "sse_pi_compute"):
            return lambda *a: self.declared.append(a[-2]) or 0
        if name in ("sse_submit", "sse_pi_submit"):
            return lambda *a: self.declared.append(a[-3]) or 0
        return getattr(self._lib, name)


CALLS = {
    "compute": lambda p, ws: sse.sse_compute(p, 1, 1, 1, 1, 1, ws),
    "submit": lambda p, ws: sse.sse_submit(p, [(1, 1, 1, 1, 1)], ws),
    "pi_compute": lambda p, ws: sse.sse_pi_compute(p, 1, 1, 1, 1, ws),
    "pi_submit": lambda p, ws: sse.sse_pi_submit(p, 1, 1, 1, 1, ws),
}


def _desc(prec=sse.FP64):
    return sse.make_desc(64, 4, 10, 3, 3, 100, 6, ncomp=2, prec=prec)


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("ws", [torch.empty(256, dtype=torch.uint8), torch.empty(33, dtype=torch.float64), 4096],
                         ids=["256_bytes", "264_bytes", "pointer"])
def test_declared_size_is_the_buffers(monkeypatch, call, ws):
    plan = sse.sse_plan(_desc(), np.arange(1, 7))
    assert plan.workspace_bytes > 1 << 20 and plan.direct_bytes == 256
    rec = Recorder(sse.lib)
    monkeypatch.setattr(sse, "lib", rec)
    CALLS[call](plan, ws)
    # a bare pointer is one to the least that the call documents
    assert rec.declared == [256 if isinstance(ws, int) else ws.numel() * ws.element_size()]


def test_direct_bytes_are_the_direct_plans(monkeypatch):
    shift = np.arange(1, 7)
    for prec in (sse.FP64, sse.FP32, sse.BF16X3, sse.FP64C64):
        one = sse.sse_plan(_desc(prec), shift)
        batch = sse.sse_plan_batch([_desc(prec)] * 3, [shift] * 3)
        assert 256 <= one.direct_bytes <= one.workspace_bytes
        assert 512 <= batch.direct_bytes <= batch.workspace_bytes
        rec = Recorder(sse.lib)
        monkeypatch.setattr(sse, "lib", rec)
        sse.sse_submit(batch, [(1, 1, 1, 1, 1)] * 3, 4096)
        assert rec.declared == [batch.direct_bytes]
        monkeypatch.undo()
