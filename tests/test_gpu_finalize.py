"""Segment scales at every number of lanes per segment that the finalize
kernel is launched with (one lane, 8, 16, a wave, a workgroup): the worker's
and the chunk owners' scales against the root mean square, in 64 bits, of the
compensated values that the same call stored."""
import numpy as np
import pytest
import torch

from parity_util import check_scales, host

pytestmark = pytest.mark.gpu


def _rms(z, plan):
    s = np.zeros(plan.S, np.float32)
    for q, (b, e) in enumerate(zip(plan.seg_begin, plan.seg_end)):
        if e > b:
            s[q] = np.sqrt(np.mean(z[b:e].astype(np.float64) ** 2))
    return s


def _lanes(plan, segments):
    """Lanes per segment of a finalize launch over that many (row, segment)
    pairs, the launch rule's line."""
    tiles = [-(-int(e) // 1024) - int(b) // 1024 if e > b else 0
             for b, e in zip(plan.seg_begin, plan.seg_end)]
    longest = max(tiles)
    if longest > 256:
        return 256
    if longest > 4 and segments <= 4096:
        return 64
    return 16 if longest > 64 else 8 if longest > 4 else 1


# lanes: of the workers' call, of all owners' call, of one owner's
@pytest.mark.parametrize("big,small,n,lanes", [
    (3000, 50, 2, (1, 1, 1)),            # at most 3 tiles
    (40_000, 3, 2, (64, 64, 64)),        # 21 tiles, few segments
    (40_000, 2200, 2, (8, 8, 64)),       # 21 tiles, 8,808, 4,404 and 2,202 segments
    (150_000, 2200, 2, (16, 16, 64)),    # 74 tiles
    (600_000, 3, 2, (256, 256, 256)),    # 294 tiles
    (5000, 70, 33, (1, 1, 1)),           # n > 32
])
def test_scales_of_every_lane_count(dev, big, small, n, lanes):
    """Through the separate calls, which always finalize (the fused step forms
    the scales of small plans in its passes)."""
    import paper_2102_02888_amd as ob
    plan = ob.Plan([100] * (small // 2) + [big, 0] + [300] * (small - small // 2), n)
    assert lanes == tuple(_lanes(plan, k) for k in (plan.S * n, plan.S, plan.K))
    st = ob.State(plan, dev)
    g = torch.Generator(device=dev)
    g.manual_seed(big + n)
    for t in (st.grads, st.m, st.x):
        t.normal_(generator=g)
    for t in (st.worker_scales, st.server_scales):
        t.fill_(3.0)   # a scale that is not written would show
    ob.onebit_worker_compress(plan, st.m, st.grads, st.worker_err, st.worker_bits,
                              st.worker_scales, 0.9, st.workspace)
    ob.onebit_server_reduce_compress(plan, 0, n, st.worker_bits, st.worker_scales, st.server_err,
                                     st.server_bits, st.server_scales, st.workspace)
    torch.cuda.synchronize()
    for i in range(n):
        check_scales("worker %d" % i, host(st.worker_scales[i]), _rms(host(st.worker_err[i]), plan))
    check_scales("server", host(st.server_scales), _rms(host(st.server_err), plan))
    # one owner's segments only (the others' scales stay as they are)
    before = st.server_scales.clone()
    ob.onebit_server_reduce_compress(plan, 1, 2, st.worker_bits, st.worker_scales, st.server_err,
                                     st.server_bits, st.server_scales, st.workspace)
    torch.cuda.synchronize()
    own = np.arange(plan.S) % n == 1
    want = np.where(own, _rms(host(st.server_err), plan), host(before))
    check_scales("owner 1", host(st.server_scales), want)
    plan.close()


@pytest.mark.parametrize("numel,n", [
    ([1 << 20], 4),                                   # 256 tiles a segment: both formed
    ([1 << 20], 3),                                   # 342 tiles: neither
    ([0, 0, 100, 0, 5000, 64, 0], 32),                # empty segments before, between, after
    ([300] * 40 + [0] + [4000] * 30, 7),              # mixed blocks, both formed
    ([2000 * 1024 + 5], 16),                          # 125 tiles: owners' alone
    ([4_000_000], 16),                                # 245 tiles, over 3,000: neither
    ([65_000] * 50, 8),                               # over 3,000, few tiles a segment: both
    ([1_000_000, 70_000], 8),                         # 123 tiles: both
    ([1_000_000] * 4, 4),                             # 245 tiles, over 3,000: workers' alone
    ([129 * 64], 33),                                 # n > 32: owners' alone
    ([1], 1),
])
def test_fused_step_equals_the_three_calls(dev, numel, n):
    """The fused step, which forms the scales inside its passes on small
    plans, against the separate calls, which finalize them: every output bit
    for bit, as both add a segment's partial sums in one order."""
    import paper_2102_02888_amd as ob
    plan = ob.Plan(numel, n)
    a, b = ob.State(plan, dev), ob.State(plan, dev)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    a.x.normal_(generator=g)
    a.m.normal_(generator=g)
    a.v.uniform_(0.5, 1.0, generator=g)
    for k in ("x", "m", "v"):
        getattr(b, k).copy_(getattr(a, k))
    for t in (a.worker_scales, a.server_scales):
        t.fill_(3.0)   # a scale that is not written would show, in an error too
    b.worker_scales.fill_(3.0)
    b.server_scales.fill_(3.0)
    for step in range(3):
        a.grads.normal_(generator=g)
        b.grads.copy_(a.grads)
        m = b.m if step == 0 else None
        a.step(1e-3, 0.9, 1e-8)
        ob.onebit_worker_compress(plan, m, b.grads, b.worker_err, b.worker_bits, b.worker_scales,
                                  0.9, b.workspace, m_bits=b.server_bits, m_scales=b.server_scales)
        ob.onebit_server_reduce_compress(plan, 0, n, b.worker_bits, b.worker_scales, b.server_err,
                                         b.server_bits, b.server_scales, b.workspace)
        ob.onebit_decompress_update(plan, b.server_bits, b.server_scales, b.x, m, b.v, 1e-3, 1e-8)
        torch.cuda.synchronize()
        for k in ("worker_bits", "server_bits"):
            assert torch.equal(getattr(a, k), getattr(b, k)), (k, step)
        for k in ("worker_scales", "server_scales", "worker_err", "server_err", "x"):
            assert torch.equal(getattr(a, k).view(torch.int32), getattr(b, k).view(torch.int32)), \
                (k, step)
    plan.close()
