"""Layouts whose 1024-element blocks hold several short tiles: ragged and
one-word tensors, chunks of one word, a last block that ends early, against
the CPU oracle in a free run of every pass.  Padding elements hold values that
would show in any sum or store that took them in (gradients: NaN)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity_util import check_bits, check_fp, check_scales, host

pytestmark = pytest.mark.gpu

PAD = 7.5


def _sizes(seed, count, lo, hi):
    rng = np.random.default_rng(seed)
    return [int(a) for a in rng.integers(lo, hi, size=count)]


CASES = [
    ("one-word tensors", [64] * 16 + [1] * 20 + [63, 65, 127], 1),     # 16 tiles in a block
    ("up to 200", _sizes(1, 90, 1, 200), 2),
    ("up to 2500", _sizes(2, 40, 1, 2500), 3),
    ("one-word chunks", [5000, 0, 1024, 3000, 64, 1], 40),             # n > 32
    ("full blocks at the end of short ones", [64, 960, 1024, 4096, 1000, 24], 1),
    ("one full block", [1024], 1),
    ("short chunks, 32 workers", _sizes(3, 12, 500, 9000), 32),
]


@pytest.mark.parametrize("grad_dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("name,numel,n", CASES)
def test_short_tiles_free_running(dev, name, numel, n, packed, grad_dtype):
    import paper_2102_02888_amd as ob
    wl = synth.Workload(name=name, numel=numel, n=n, warmup_steps=2, steps=3)
    L = oracle.Layout(numel, n)
    plan = ob.Plan(numel, n)
    mask = L.real_mask()
    pad = torch.from_numpy(~mask).to(dev)
    st = ob.State(plan, dev, grad_dtype=grad_dtype, packed_momentum=packed)
    x = synth.host_params(wl, L.D)
    x[~mask] = 0
    st.x.copy_(torch.from_numpy(x))
    padded = (st.x, st.m, st.v, st.worker_err, st.server_err)
    for t in padded:
        t[..., pad] = PAD

    def grads(t):
        gt = torch.from_numpy(synth.host_grads(wl, L.D, L.tensor_off, t)).to(grad_dtype)
        st.grads.copy_(gt.to(dev))
        st.grads[:, pad] = float("nan")
        return gt.float().numpy()

    m, v = np.zeros(L.D, np.float32), np.zeros(L.D, np.float32)
    for t in (1, 2):
        g = grads(t)
        oracle.warmup_step(L, x, m, v, g, n, wl.lr, wl.beta1, wl.beta2, wl.eps, 0, t)
        st.warmup(wl.lr, wl.beta1, wl.beta2, wl.eps, t)
    norm = st.variance_l1_norm()
    assert abs(norm - oracle.l1_norm(L, host(st.v))) <= 1e-12 * norm
    ref = oracle.State(L, x, m, v)
    for t in (3, 4, 5):
        g = grads(t)
        ref.step(g, wl.lr, wl.beta1, wl.eps)
        st.step(wl.lr, wl.beta1, wl.eps)
        torch.cuda.synchronize()
        check_bits("worker bits", host(st.worker_bits), ref.wbits)
        check_bits("server bits", host(st.server_bits), ref.sbits)
        check_scales("worker scales", host(st.worker_scales), ref.wscales)
        check_scales("server scales", host(st.server_scales), ref.sscales)
    for what, a, b in (("x", st.x, ref.x), ("m", st.momentum(), ref.m),
                       ("worker delta", st.worker_delta(), ref.delta),
                       ("server delta", st.server_delta(), ref.delta_bar)):
        check_fp(what, host(a), b, mask=mask)
    # explicit values leave the padding of a caller's buffer alone unless asked
    for got, fill in ((torch.full_like(st.x, PAD), False), (torch.full_like(st.x, PAD), True)):
        ob.onebit_decode(plan, st.server_bits, st.server_scales, got, zero_padding=fill)
        err = got.clone() if fill else torch.full_like(got, PAD)
        ob.onebit_error_materialize(plan, st.server_err, st.server_scales, err, rows=1,
                                    zero_padding=fill)
        check_fp("decoded", host(got), ref.m, mask=mask)
        check_fp("server delta", host(err), ref.delta_bar, mask=mask)
        for t in (got, err):
            assert bool((t[pad] == (0.0 if fill else PAD)).all())
    for t in (st.momentum() if packed else torch.zeros(1, device=dev), st.worker_delta(),
              st.server_delta()):
        if t.shape[-1] == plan.D:
            assert bool((t[..., pad] == 0).all())
    # the comparison steps on the same layout
    m, v, x = host(st.momentum()).copy(), host(st.v).copy(), host(st.x).copy()
    st.m.copy_(torch.from_numpy(m))
    g = grads(6)
    oracle.step_uncompressed(L, x, m, v, g, wl.lr, wl.beta1, wl.eps)
    st.step_uncompressed(wl.lr, wl.beta1, wl.eps)
    dec = oracle.decode_message(L, host(st.server_bits), host(st.server_scales))
    oracle.warmup_step(L, x, m, v, dec[None, :].copy(), 1, wl.lr, wl.beta1, wl.beta2, wl.eps, 0, 7)
    ob.onebit_adam_message_step(plan, st.x, st.m, st.v, st.server_bits, st.server_scales, wl.lr,
                                wl.beta1, wl.beta2, wl.eps, 0, 7)
    torch.cuda.synchronize()
    check_fp("x", host(st.x), x, mask=mask)
    check_fp("m", host(st.m), m, mask=mask)
    check_fp("v", host(st.v), v, mask=mask)
    for t in (st.x, st.v, st.worker_err, st.server_err):
        assert bool((t[..., pad] == PAD).all()), "a padding element was written"
    plan.close()


# Row-summing shapes: small plans take four rows at a time, larger ones one
# sub-block per wave for few rows and a whole block (fp32) or two sub-blocks
# (16-bit) for many; the sizes lie on both sides of each line and end inside a
# block (odd sizes) or on its edge.
@pytest.mark.parametrize("variant", ["warmup", "uncompressed"])
@pytest.mark.parametrize("grad_dtype,numel,n", [
    (torch.float32, [1], 1), (torch.float32, [2048 * 1024 - 64, 63], 5),
    (torch.float32, [2048 * 1024 + 1], 3), (torch.float32, [8192 * 1024], 13),
    (torch.float32, [8192 * 1024 + 77], 12), (torch.float32, [8000 * 1024, 300_007], 13),
    (torch.bfloat16, [4096 * 1024], 7), (torch.bfloat16, [4096 * 1024 + 1], 4),
    (torch.float16, [4096 * 1024, 1000], 5),
])
def test_row_sum_shapes(dev, variant, grad_dtype, numel, n):
    """Against the same formula in torch: the fp64 sum of the rows in row
    order, one rounding, then fp32 operations rounded one by one."""
    import paper_2102_02888_amd as ob
    lr, b1, b2, eps = 1e-3, 0.9, 0.999, 1e-8
    plan = ob.Plan(numel, n)
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    f = dict(device=dev, dtype=torch.float32)
    x, m = (torch.empty(plan.D, **f).normal_(generator=gen) for _ in range(2))
    v = torch.empty(plan.D, **f).uniform_(0.1, 1.0, generator=gen)
    g = torch.empty((n, plan.D), dtype=grad_dtype, device=dev).normal_(generator=gen)
    real = torch.from_numpy(oracle.Layout(numel, n).real_mask()).to(dev)
    one = np.float32(1)
    o1, o2 = float(one - np.float32(b1)), float(one - np.float32(b2))
    total = torch.zeros(plan.D, dtype=torch.float64, device=dev)
    if variant == "warmup":
        for i in range(n):
            total += g[i].double()
        gbar = (total / n).float()
        m1 = b1 * m + o1 * gbar
        v1 = b2 * v + o2 * (gbar * gbar)
        x1 = x - lr * (m1 / (v1.sqrt() + eps))
    else:
        for i in range(n):
            total += (b1 * m + o1 * g[i].float()).double()
        m1, v1 = (total / n).float(), v
        x1 = x - lr * (m1 / (v + eps).sqrt())
    want = [torch.where(real, a, b) for a, b in ((x1, x), (m1, m), (v1, v))]
    if variant == "warmup":
        ob.onebit_warmup_adam_step(plan, x, m, v, g, lr, b1, b2, eps, 0, 1)
    else:
        ob.onebit_uncompressed_step(plan, x, m, v, g, lr, b1, eps)
    torch.cuda.synchronize()
    # torch's fp32 division and square root round as the kernels do, but for
    # an ulp here and there: 2 ulp of the value, as x is near 1
    for name, a, b in zip("xmv", (x, m, v), want):
        worst = float(((a - b).abs() / b.abs().clamp(min=1e-3)).max())
        assert worst <= 2 ** -22, (name, worst)
    plan.close()


@pytest.mark.parametrize("n,narrow", [(2, True), (5, True), (8, False), (9, True), (32, True),
                                      (33, False), (70, True)])
def test_one_by_one_owners_equal_the_lookup_tables(dev, n, narrow):
    """Plans of many short tiles take the owners' pass that adds the workers
    one by one; with the tables forced on, the same call takes the lookup
    tables: equal bit for bit, for scales whose sums are exact in any order
    (narrow) and for scales of 40 binades and zeros, which are not."""
    import paper_2102_02888_amd as ob
    rng = np.random.default_rng(n)
    numel = [int(a) for a in rng.integers(1, 64 * 2 * n, size=14000 // n + 300)] + [1 << 15, 0, 1024]
    plan = ob.Plan(numel, n)
    assert plan.T > 8192 and plan.T >= 3 * ((plan.D + 1023) // 1024)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    bits = torch.randint(-(1 << 62), 1 << 62, (n, plan.W), dtype=torch.int64, device=dev,
                         generator=g)
    scales = torch.empty((n, plan.S), device=dev).log_normal_(-7, 0.3 if narrow else 7.0,
                                                              generator=g)
    if not narrow:
        scales[:, ::5] = 0
    err = torch.empty(plan.D, device=dev).normal_(0, 1e-3, generator=g)
    old = torch.empty(plan.S, device=dev).log_normal_(-7, 0.3, generator=g)
    out = []
    for mode in (ob.SERVER_TABLES_AUTO, ob.SERVER_TABLES_ON):
        plan.set_server_tables(mode)
        e, sb, ss = err.clone(), torch.zeros(plan.W, dtype=torch.int64, device=dev), old.clone()
        ob.onebit_server_reduce_compress(plan, 0, n, bits, scales, e, sb, ss, plan.workspace(dev))
        torch.cuda.synchronize()
        out.append((e, sb, ss))
    assert torch.equal(out[0][0].view(torch.int32), out[1][0].view(torch.int32))
    assert torch.equal(out[0][1], out[1][1])
    assert torch.equal(out[0][2].view(torch.int32), out[1][2].view(torch.int32))
    plan.close()
