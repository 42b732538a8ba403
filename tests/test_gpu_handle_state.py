"""What a handle keeps between calls: the stream its lazily allocated buffers
belong to, the form of its convolutions and the bits of repeated calls."""
import numpy as np
import pytest

from tests.test_gpu_two_pass import mvd, problem  # noqa: F401

pytestmark = pytest.mark.gpu


def test_lazy_buffers_belong_to_the_handles_stream(mvd):
    """Buffers allocated by a later call come from the pool of the handle's
    stream, not of the stream that is current then (whose pending work may
    still use what its pool hands out)."""
    import torch
    v, p, _ = problem((48, 45, 16), 2, 800, False)
    with mvd.Deconvolver(v, p) as d:
        before, other = set(d._bufs), torch.cuda.Stream()
        with torch.cuda.stream(other):
            d.iterate(2, "eff")
        new = set(d._bufs) - before
        assert new
        segs = [(s["address"], s["total_size"], s["stream"]) for s in torch.cuda.memory_snapshot()]
        for a in new:
            assert [st for lo, n, st in segs if lo <= a < lo + n] == [d.stream.cuda_stream]
