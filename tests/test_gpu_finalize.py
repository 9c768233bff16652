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


@pytest.mark.parametrize("big,small,n", [
    (3000, 50, 2),        # at most 4 tiles: one lane
    (40_000, 3, 2),       # 20 tiles, few segments: a wave
    (40_000, 1100, 2),    # 20 tiles, over 4,096 pairs: 8 lanes
    (150_000, 1100, 2),   # 74 tiles: 16 lanes
    (600_000, 3, 2),      # 293 tiles: a workgroup
    (5000, 70, 33),       # n > 32
])
def test_scales_of_every_lane_count(dev, big, small, n):
    import paper_2102_02888_amd as ob
    plan = ob.Plan([100] * (small // 2) + [big, 0] + [300] * (small - small // 2), n)
    st = ob.State(plan, dev)
    g = torch.Generator(device=dev)
    g.manual_seed(big + n)
    for t in (st.grads, st.m, st.x):
        t.normal_(generator=g)
    st.v.fill_(1.0)
    for _ in range(2):
        st.step(1e-3, 0.9, 1e-8)
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
