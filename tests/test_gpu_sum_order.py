"""One order of every 64-bit sum per plan: the same values give the same scale
bit for bit whichever call, momentum form, gradient type or lookup-table mode
computes it.  The values are chosen so that the last bits of a sum of squares
decide its scale (parity_util.knife_edge); without gradients, momentum and
earlier scales the compensated values are the error state's own."""
import numpy as np
import pytest
import torch

from parity_util import knife_edge_rows

pytestmark = pytest.mark.gpu


def _state(plan, dev, worker=None, server=None, **more):
    """A state whose next step's compensated values are the given rows."""
    import paper_2102_02888_amd as ob
    st = ob.State(plan, dev, **more)
    st.v.fill_(1.0)
    if worker is not None:
        st.worker_err.copy_(worker)
    if server is not None:
        st.server_err.copy_(server)
    return st


def _knife(plan, dev, seed, rows=1):
    return torch.from_numpy(knife_edge_rows(np.random.default_rng(seed), plan, rows)).to(dev)


def _compress(st, m=None, rows=None):
    import paper_2102_02888_amd as ob
    ob.onebit_worker_compress(st.plan, m, st.grads, st.worker_err, st.worker_bits,
                              st.worker_scales, 0.9, st.workspace, n_local=rows,
                              m_bits=st.server_bits, m_scales=st.server_scales)


def _reduce(st, begin, end):
    import paper_2102_02888_amd as ob
    ob.onebit_server_reduce_compress(st.plan, begin, end, st.worker_bits, st.worker_scales,
                                     st.server_err, st.server_bits, st.server_scales,
                                     st.workspace)


def _same(a, b, what):
    bad = int((a.view(torch.int32) != b.view(torch.int32)).sum())
    assert bad == 0, "%s: %d of %d scales differ" % (what, bad, a.numel())


# The segments of one row (or owner) and of all of them lie on both sides of
# the number below which the finalize kernel gives each segment a wave.
@pytest.mark.parametrize("each,count,n", [
    (160_000, 300, 8),       # 20 tiles a segment
    (560_000, 90, 8),        # 69
    (4_000_000, 20, 16),     # 245
    (6000, 1200, 2),         # 3
])
def test_worker_scale_does_not_depend_on_the_rows_of_the_call(dev, each, count, n):
    import paper_2102_02888_amd as ob
    plan = ob.Plan([each] * count, n)
    row = _knife(plan, dev, each)
    got = []
    for r in (1, n):
        st = _state(plan, dev, row.expand(r, -1), n_local=r, grad_dtype=torch.bfloat16)
        _compress(st)
        torch.cuda.synchronize()
        for i in range(r):
            got.append(st.worker_scales[i].clone())
        del st
    assert plan.S <= 4096 < plan.S * n
    for i, s in enumerate(got[1:]):
        _same(got[0], s, "row %d" % i)
    plan.close()


@pytest.mark.parametrize("each,count,n", [(160_000, 600, 8), (1_000_000, 75, 4), (700_000, 9, 3)])
def test_server_scale_does_not_depend_on_the_owned_range(dev, each, count, n):
    import paper_2102_02888_amd as ob
    plan = ob.Plan([each] * count, n)
    z = _knife(plan, dev, each)[0]
    a, b = (_state(plan, dev, server=z, n_local=n, grad_dtype=torch.bfloat16) for _ in range(2))
    _reduce(a, 0, n)
    for j in range(n):
        _reduce(b, j, j + 1)
    torch.cuda.synchronize()
    _same(a.server_scales, b.server_scales, "server scales")
    plan.close()


# Small plans, whose fused step forms both scales, the workers' or the owners'
# alone in its passes (the separate calls finalize them): segments of up to 16
# words, of several tiles, of more than 64 and of more than 128.
@pytest.mark.parametrize("numel,n", [
    ([1000] * 300 + [0] + [64 * 5] * 100, 2),
    ([9000] * 110, 7),
    ([65_000] * 60, 8),
    ([250_000] * 30, 4),
    ([1 << 20], 4),
    ([500_000] * 4, 3),
    ([150_000] * 6, 16),
    ([30_000] * 30, 32),
    ([3000] * 60, 33),
    ([200_000], 1),
])
def test_fused_step_rounds_its_scales_as_the_three_calls(dev, numel, n):
    import paper_2102_02888_amd as ob
    plan = ob.Plan(numel, n)
    for seed, what in ((1, "worker"), (2, "server"), (3, "worker"), (4, "server")):
        z = _knife(plan, dev, seed, n if what == "worker" else 1)
        z = {"worker": z} if what == "worker" else {"server": z[0]}
        a, b = _state(plan, dev, **z), _state(plan, dev, **z)
        a.compression_steps = 1
        a.step(1e-3, 0.9, 1e-8)
        _compress(b)
        _reduce(b, 0, n)
        torch.cuda.synchronize()
        _same(a.worker_scales, b.worker_scales, "worker scales")
        _same(a.server_scales, b.server_scales, "server scales")
    plan.close()


@pytest.mark.parametrize("numel,n", [
    ([5000] * 800, 4),                 # 3,950 blocks, whole and mixed: the row walk
    ([1024] * 2040, 4),                # 2,040: the row walk
    ([5000] * 800, 2),                 # two rows: the packed pass's grid
    ([1024] * 2500, 5),                # 2,500: the packed pass's grid
    ([300] * 400 + [2000] * 100, 5),   # few: the packed pass's grid
])
def test_worker_scale_does_not_depend_on_the_momentum_form_or_gradient_type(dev, numel, n):
    import paper_2102_02888_amd as ob
    plan = ob.Plan(numel, n)
    z = _knife(plan, dev, len(numel), n)
    first = None
    for dtype in (torch.float32, torch.bfloat16, torch.float16):
        for fp32_m in (False, True):
            st = _state(plan, dev, worker=z, grad_dtype=dtype)
            _compress(st, m=st.m if fp32_m else None)
            torch.cuda.synchronize()
            if first is None:
                first = st
            what = "%s, %s momentum" % (dtype, "fp32" if fp32_m else "packed")
            _same(first.worker_scales, st.worker_scales, what)
            assert torch.equal(first.worker_bits, st.worker_bits), what
            assert torch.equal(first.worker_err, st.worker_err), what
    plan.close()


def _mixed(rng, n, tiles):
    """Tensor sizes whose chunks are one word to a few blocks long."""
    out = []
    while sum(-(-d // (64 * n)) > 0 for d in out) * n < tiles:
        words = [0.5, 1, 1, 2, 2, 3, 4, 5, 7, 12, 20] if n <= 128 else [0.5, 1, 2, 2, 3, 5, 8]
        out.append(int(64 * n * rng.choice(words)) + int(rng.integers(0, 60)))
    return out


@pytest.mark.parametrize("n", [2, 7, 8, 32, 33, 64, 130])
def test_server_scale_does_not_depend_on_the_table_mode_or_owned_range(dev, n):
    """Plans of many short tiles, which the automatic mode gives the owners'
    pass over blocks when every chunk is owned."""
    import paper_2102_02888_amd as ob
    plan = ob.Plan(_mixed(np.random.default_rng(n), n, 9500 if n <= 128 else 12_500), n)
    assert plan.T > 8192 and plan.T >= (3 if n <= 128 else 4) * ((plan.D + 1023) // 1024)
    z = _knife(plan, dev, n)[0]
    got = {}
    for mode in (ob.SERVER_TABLES_AUTO, ob.SERVER_TABLES_ON, ob.SERVER_TABLES_OFF, "one by one"):
        plan.set_server_tables(ob.SERVER_TABLES_AUTO if mode == "one by one" else mode)
        st = _state(plan, dev, server=z, grad_dtype=torch.bfloat16)
        for j in range(n) if mode == "one by one" else (None,):
            _reduce(st, *((0, n) if j is None else (j, j + 1)))
        torch.cuda.synchronize()
        got[mode] = st.server_scales
    for mode, s in got.items():
        _same(got[ob.SERVER_TABLES_ON], s, str(mode))
    plan.close()
