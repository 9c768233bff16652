"""Timed cases of the 1-bit Adam path: what a program that uses this package
has it do, from one small model to the BERT-Large shape.

A case is one call sequence of a training program on one GPU:

  step          State.step(): a steady compression step of n simulated workers
                (packed False: the momentum is kept in fp32, as it is in the
                first compression step of every run)
  warmup        State.warmup(), with norm True also State.variance_l1_norm():
                a warm-up step, and the indicator that ends the warm-up
  share         one GPU's part of an n-worker step: its own worker's
                compression, the owner of one chunk reducing the n received
                messages, and the update with the gathered message
  naive         State.step_naive(), the "Adam(1-bit Naive)" comparison run
  uncompressed  State.step_uncompressed(), the "1-bit Adam (32-bits)" run
  explicit      State.momentum(), worker_delta() and server_delta(): the state
                in explicit form, for a checkpoint or an inspection

over one flat buffer ("layout": "flat", d elements) or a list of tensors that
are compressed one by one ("layout": "tensors", log-uniform sizes).
"""
import math

import numpy as np
import torch

import paper_2102_02888_amd as ob

LR, BETA1, BETA2, EPS = 1e-4, 0.9, 0.999, 1e-8
GRAD_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
GRAD_BYTES = {"f32": 4, "bf16": 2, "f16": 2}
BERT_BASE = 108_888_576
BERT_LARGE = 334_088_192


def _flat(kind, d, n, dtype="f32", **more):
    return dict(kind=kind, layout="flat", d=d, n=n, dtype=dtype, **more)


def _tensors(kind, count, lo, hi, n, dtype="f32", layout_seed=2, **more):
    return dict(kind=kind, layout="tensors", count=count, lo=lo, hi=hi,
                layout_seed=layout_seed, n=n, dtype=dtype, **more)


def listed():
    return [
        # a handful of small tensors: launches and host time are all there is
        dict(_tensors("step", 16, 64, 1 << 14, 4, packed=True), name="step-small"),
        # one flat buffer of 2^20 elements, the smallest benchmark workload
        dict(_flat("step", 1 << 20, 4, packed=True), name="step-2^20"),
        # a small network compressed per tensor, 16-bit gradients (ragged sizes)
        dict(_tensors("step", 80, 64, 1 << 20, 8, "bf16", packed=True), name="step-80-tensors-bf16"),
        # the BERT-Base shape as one flat buffer
        dict(_flat("step", BERT_BASE, 16, packed=True), name="step-bert-base"),
        # the BERT-Large shape with bf16 gradients, as mixed-precision training gives them
        dict(_flat("step", BERT_LARGE, 16, "bf16", packed=True), name="step-bert-large-bf16"),
        # 5,000 tensors compressed one by one: 40,000 segments, many of them short
        dict(_tensors("step", 5000, 64, 1 << 20, 8, packed=True), name="step-5000-tensors"),
        # the first compression step (fp32 momentum), BERT-Base shape
        dict(_flat("step", BERT_BASE, 16, packed=False), name="step-fp32-momentum"),
        # a warm-up step with the indicator that decides when to freeze the variance
        dict(_flat("warmup", BERT_LARGE, 8, norm=True), name="warmup-bert-large-norm"),
        # one GPU of a 256-GPU run, BERT-Large shape
        dict(_flat("share", BERT_LARGE, 256, chunk=0), name="share-of-256"),
        # one GPU of an 8-GPU run, a network compressed per tensor, bf16 gradients
        dict(_tensors("share", 400, 64, 1 << 20, 8, "bf16", chunk=3), name="share-of-8-tensors"),
        # the naive comparison run with fp16 gradients, ragged tensors
        dict(_tensors("naive", 200, 64, 1 << 20, 8, "f16"), name="naive-200-tensors-f16"),
        # the whole state in explicit form, an odd length
        dict(_flat("explicit", 29_999_957, 8), name="explicit-30M"),
    ]


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["warmup", "warmup", "share", "share", "naive",
                                      "uncompressed", "explicit"])
    n = rng.choice([2, 3, 4, 5, 8, 8, 16, 16, 24, 32])
    if kind == "share":
        n = rng.choice([4, 8, 16, 32, 64, 100, 128, 256])
    rows = 1 if kind == "share" else n
    dtype = "f32" if kind == "explicit" else rng.choice(["f32", "f32", "bf16", "f16"])
    more = {}
    if kind == "step":
        more["packed"] = rng.random() < 0.8
    elif kind == "warmup":
        more["norm"] = rng.random() < 0.5
    elif kind == "share":
        more["chunk"] = rng.randrange(n)
    most = min(200_000_000, 1_500_000_000 // rows)  # elements: below the largest listed case
    if rng.random() < 0.5:
        d = int(math.exp(rng.uniform(math.log(3000), math.log(most))))
        return _flat(kind, d, n, dtype, **more)
    hi = rng.choice([1 << 13, 1 << 16, 1 << 20])
    if kind == "share":
        most = min(most, 800_000_000 // n)  # n whole rows of sign words are held
    mean = (hi - 64) / math.log(hi / 64)
    count = int(math.exp(rng.uniform(math.log(2), math.log(max(3, min(4000, most / (1.2 * mean)))))))
    return _tensors(kind, count, 64, hi, n, dtype, layout_seed=rng.randrange(1 << 20), **more)


# ---------------------------------------------------------------------------
# Inputs: every array is a seeded draw of its own
# ---------------------------------------------------------------------------

def _numel(case):
    if case["layout"] == "flat":
        return [case["d"]]
    rng = np.random.Generator(np.random.Philox(key=[case["layout_seed"], 0x5157]))
    u = rng.uniform(math.log(case["lo"]), math.log(case["hi"]), size=case["count"])
    return [int(min(case["hi"], max(case["lo"], round(math.exp(a))))) for a in u]


X, M, V, GRADS, WORKER_ERR, WORKER_SCALES, SERVER_ERR, SERVER_BITS, SERVER_SCALES, IN_BITS, \
    IN_SCALES = range(11)


def _gen(seed, what, row=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(((int(seed) * 16 + what) * 4099 + row) & ((1 << 62) - 1))
    return g


def _floats(size, seed, what, row=0, dtype=torch.float32):
    """Parameters N(0, 0.02); gradients N(0, 1e-3); the moments and the
    compensated values of the magnitudes that such gradients lead to; scales
    spread a little around the root mean square of what they scale."""
    out = torch.empty(size, dtype=dtype, device="cuda")
    g = _gen(seed, what, row)
    if what in (WORKER_SCALES, SERVER_SCALES, IN_SCALES):
        mid = {WORKER_SCALES: 1.2e-3, SERVER_SCALES: 4e-4, IN_SCALES: 9e-4}[what]
        return out.log_normal_(math.log(mid), 0.3 if what == IN_SCALES else 0.05, generator=g)
    if what == V:
        return out.log_normal_(math.log(1e-6), 0.5, generator=g)
    std = {X: 0.02, M: 4e-4, GRADS: 1e-3, WORKER_ERR: 1.2e-3, SERVER_ERR: 4e-4}[what]
    return out.normal_(0.0, std, generator=g)


def _words(size, seed, what, row=0):
    half = torch.randint(-(1 << 31), 1 << 31, (2 * size,), dtype=torch.int32, device="cuda",
                         generator=_gen(seed, what, row))
    return half.view(torch.int64)


def _rows(case):
    return 1 if case["kind"] == "share" else case["n"]


def prepare(case, seed):
    kind, n, rows = case["kind"], case["n"], _rows(case)
    dev = torch.device("cuda", torch.cuda.current_device())
    plan = ob.Plan(_numel(case), n)
    D, W, S = plan.D, plan.W, plan.S
    more = {}
    if kind == "explicit":  # reads no gradients
        more["grads"] = torch.zeros((1, D), dtype=torch.float32, device=dev)
    st = ob.State(plan, dev, n_local=rows, grad_dtype=GRAD_DTYPES[case["dtype"]],
                  packed_momentum=case.get("packed", True), **more)
    s = {"case": case, "plan": plan, "st": st, "t": 1}
    st.x.copy_(_floats(D, seed, X))
    st.m.copy_(_floats(D, seed, M))
    st.v.copy_(_floats(D, seed, V))
    if kind != "explicit":
        for i in range(rows):
            st.grads[i].copy_(_floats(D, seed, GRADS, i, st.grads.dtype))
    if kind in ("warmup", "uncompressed"):
        return s
    st.compression_steps = 2  # a run that is past its first compression steps
    for i in range(rows):
        st.worker_err[i].copy_(_floats(D, seed, WORKER_ERR, i))
        st.worker_scales[i].copy_(_floats(S, seed, WORKER_SCALES, i))
    st.server_err.copy_(_floats(D, seed, SERVER_ERR))
    st.server_bits.copy_(_words(W, seed, SERVER_BITS))
    st.server_scales.copy_(_floats(S, seed, SERVER_SCALES))
    if kind == "share":
        j = case["chunk"]
        if plan.K == 1:  # the chunk's words and scale of every worker, as received
            q = j
            base, cols = int(plan.seg_begin[q]) // 64, int(plan.seg_end[q] - plan.seg_begin[q] + 63) // 64
            cols = max(cols, 1)
            s["in_bits"] = torch.stack([_words(cols, seed, IN_BITS, i) for i in range(n)])
            s["in_scales"] = _floats(n, seed, IN_SCALES).view(n, 1)
            s["in_at"] = dict(bits_word_base=base, scales_seg_base=j, bits_ld=cols, scales_ld=1)
        else:  # one slice per tensor, kept at its place in plan-wide rows
            s["in_bits"] = torch.stack([_words(W, seed, IN_BITS, i) for i in range(n)])
            s["in_scales"] = torch.stack([_floats(S, seed, IN_SCALES, i) for i in range(n)])
            s["in_at"] = {}
    return s


def run(s):
    st, plan, kind = s["st"], s["plan"], s["case"]["kind"]
    s["t"] += 1
    if kind == "warmup":
        st.warmup(LR, BETA1, BETA2, EPS, s["t"])
        out = {"x": st.x, "m": st.m, "v": st.v}
        if s["case"]["norm"]:
            out["norm"] = st.variance_l1_norm()
        return out
    if kind == "uncompressed":
        st.step_uncompressed(LR, BETA1, EPS)
        return {"x": st.x, "m": st.m}
    if kind == "explicit":
        return {"m": st.momentum(), "worker": st.worker_delta(), "server": st.server_delta()}
    out = {"x": st.x, "worker_err": st.worker_err, "worker_bits": st.worker_bits,
           "worker_scales": st.worker_scales, "server_err": st.server_err,
           "server_bits": st.server_bits, "server_scales": st.server_scales}
    if kind == "step":
        st.step(LR, BETA1, EPS)
        if not s["case"]["packed"]:
            out["m"] = st.m
    elif kind == "naive":
        st.step_naive(LR, BETA1, BETA2, EPS, s["t"])
        out.update(m=st.m, v=st.v)
    else:
        j = s["case"]["chunk"]
        ob.onebit_worker_compress(plan, None, st.grads, st.worker_err, st.worker_bits,
                                  st.worker_scales, BETA1, st.workspace, n_local=1,
                                  m_bits=st.server_bits, m_scales=st.server_scales)
        ob.onebit_server_reduce_compress(plan, j, j + 1, s["in_bits"], s["in_scales"],
                                         st.server_err, st.server_bits, st.server_scales,
                                         st.workspace, **s["in_at"])
        ob.onebit_decompress_update(plan, st.server_bits, st.server_scales, st.x, None, st.v,
                                    LR, EPS)
    return out


def work(case):
    """Each input read once, each output written once (sign words 1/8 byte an element)."""
    kind, n, rows = case["kind"], case["n"], _rows(case)
    d = sum(_numel(case))
    g = GRAD_BYTES[case["dtype"]]
    own = d
    if kind == "share":
        own = sum(e - b for k, j, b, e in _segments(case) if j == case["chunk"])
    worker = rows * (g + 4 + 4 + 1 / 8)
    server = n / 8 + 4 + 4 + 1 / 8
    if kind == "warmup":
        per, flops = g * n + 24 + (4 if case["norm"] else 0), n + 14 + (1 if case["norm"] else 0)
        return {"bytes": d * per, "flops": d * flops}
    if kind == "uncompressed":
        return {"bytes": d * (g * n + 20), "flops": d * (3 * n + 6)}
    if kind == "explicit":
        return {"bytes": d * (4 + 1 / 8 + (rows + 1) * 8), "flops": d * (rows + 1)}
    if kind == "naive":
        return {"bytes": d * (worker + server + 1 / 8 + 24), "flops": d * (8 * n + 20)}
    m = 1 / 8 if case.get("packed", True) else 8
    return {"bytes": d * (m + worker + 1 / 8 + 12) + own * server,
            "flops": d * (6 * rows + 5) + own * (n + 5)}


def tolerance(case):
    """Every fp32 value is a few roundings of its inputs (measured 2e-8 to
    5e-8 off the 64-bit value, 3e-7 at most for a single element); sums run in
    64 bits.  A scale that another order of its sum rounds to the next fp32
    value may turn the sign of a server value within an ulp of zero (measured
    on the BERT-Large shape: one such element in 10^8 takes x to 3.1e-7 off
    as a whole and that element 0.4% of the root mean square; in a later pass
    its momentum is another), which is one word in 10^5 at most."""
    if case["kind"] in ("warmup", "uncompressed", "explicit"):
        return {"rel": 2e-7, "max": 2e-6}
    return {"rel": 1.5e-6, "max": 0.1, "differ": 2e-5}


# ---------------------------------------------------------------------------
# The same pass in 64 bits, plain torch
# ---------------------------------------------------------------------------

def _segments(case):
    """(tensor, chunk, begin, end) of every segment: tensors start on
    multiples of 64 elements, chunks are 64 ceil(d / 64 n) elements."""
    off, out = 0, []
    for k, d in enumerate(_numel(case)):
        c = -(-d // (64 * case["n"])) * 64
        for j in range(case["n"]):
            out.append((k, j, off + min(j * c, d), off + min((j + 1) * c, d)))
        off += -(-d // 64) * 64
    return out


class _Layout:
    def __init__(self, case):
        segs = _segments(case)
        numel = _numel(case)
        self.D = sum(-(-d // 64) * 64 for d in numel)
        self.S = len(segs)
        b = torch.tensor([s[2] for s in segs])
        e = torch.tensor([s[3] for s in segs])
        self.len = (e - b).cuda()
        self.b, self.e = b.cuda(), e.cuda()
        self.seg = torch.zeros(self.D, dtype=torch.int32, device="cuda")
        self.real = torch.zeros(self.D, dtype=torch.bool, device="cuda")
        if self.S <= 4096:
            for q, s in enumerate(segs):
                self.seg[s[2]:s[3]] = q
                self.real[s[2]:s[3]] = True
        else:
            at = [q for q in range(self.S) if segs[q][3] > segs[q][2]]
            begin = torch.tensor([segs[q][2] for q in at])
            end = torch.tensor([segs[q][3] for q in at])
            nxt = torch.cat([begin[1:], torch.tensor([self.D])])
            self.seg = torch.repeat_interleave(torch.tensor(at, dtype=torch.int32).cuda(),
                                               (nxt - begin).cuda())
            self.real = torch.zeros(self.D + 1, dtype=torch.int32, device="cuda")
            self.real.index_add_(0, begin.cuda(), torch.ones(len(at), dtype=torch.int32, device="cuda"))
            self.real.index_add_(0, end.cuda(), -torch.ones(len(at), dtype=torch.int32, device="cuda"))
            self.real = self.real.cumsum(0)[:self.D] > 0

    def spread(self, scales):
        return scales[self.seg]

    def scales(self, z):
        """root mean square of each segment; 0 for an empty one"""
        total = torch.zeros(self.D + 1, dtype=torch.float64, device="cuda")
        torch.cumsum(torch.where(self.real, z * z, 0.0), 0, out=total[1:])
        mean = (total[self.e] - total[self.b]) / self.len.clamp(min=1)
        return mean.clamp(min=0.0).sqrt() * (self.len > 0)


def _error(z, s):
    return torch.where(z >= 0, z - s, z + s)


def _signs(words, D):
    """+1 or -1 of each element (bit 1 is +1)"""
    shift = torch.arange(64, device="cuda")
    out = torch.empty(D // 64, 64, dtype=torch.float32, device="cuda")
    step = 1 << 20
    for a in range(0, D // 64, step):
        bits = (words[a:a + step, None] >> shift) & 1
        out[a:a + step] = bits * 2 - 1
    return out.view(-1)


def exact(case, seed):
    """What run() returns, in 64 bits.  Signs are decided on the fp32 value,
    computed by the same single roundings: near zero the sign of a rounded sum
    is a matter of its rounding, and the signs are inputs of what follows."""
    kind, n, rows = case["kind"], case["n"], _rows(case)
    L = _Layout(case)
    D = L.D
    f = np.float32
    lr, b1, b2, eps = (float(f(a)) for a in (LR, BETA1, BETA2, EPS))
    o1, o2 = float(f(1) - f(BETA1)), float(f(1) - f(BETA2))
    x, v = _floats(D, seed, X).double(), _floats(D, seed, V).double()

    def grad(i):
        return _floats(D, seed, GRADS, i, GRAD_DTYPES[case["dtype"]])

    if kind in ("warmup", "uncompressed"):
        m = _floats(D, seed, M).double()
        g = torch.zeros(D, dtype=torch.float64, device="cuda")
        for i in range(n):
            g += grad(i).double()
        g /= n
        m1 = b1 * m + o1 * g
        if kind == "uncompressed":
            x1 = x - lr * m1 / (v + eps).sqrt()
            return {"x": torch.where(L.real, x1, x), "m": torch.where(L.real, m1, m)}
        v1 = b2 * v + o2 * g * g
        x1 = x - lr * m1 / (v1.sqrt() + eps)
        out = {"x": torch.where(L.real, x1, x), "m": torch.where(L.real, m1, m),
               "v": torch.where(L.real, v1, v)}
        if case["norm"]:
            out["norm"] = float(torch.where(L.real, v1, 0.0).abs().sum())
        return out

    sserr, sscales = _floats(D, seed, SERVER_ERR), _floats(L.S, seed, SERVER_SCALES)
    swords = _words(D // 64, seed, SERVER_BITS)
    msign = _signs(swords, D)
    if kind == "explicit":
        worker = torch.empty(rows, D, dtype=torch.float64, device="cuda")
        for i in range(rows):
            z = _floats(D, seed, WORKER_ERR, i).double()
            worker[i] = _error(z, L.spread(_floats(L.S, seed, WORKER_SCALES, i).double()))
            worker[i].mul_(L.real)
        server = _error(sserr.double(), L.spread(sscales.double())) * L.real
        return {"m": msign.double() * L.spread(sscales.double()) * L.real, "worker": worker,
                "server": server}

    # the workers
    if kind == "naive":
        m32, c1, d1 = torch.zeros(D, device="cuda"), 0.0, 1.0
    elif kind == "step" and not case["packed"]:
        m32, c1, d1 = _floats(D, seed, M), b1, o1
    else:
        m32, c1, d1 = msign * L.spread(sscales), b1, o1
    werr = torch.empty(rows, D, dtype=torch.float64, device="cuda")
    wscales = torch.empty(rows, L.S, dtype=torch.float64, device="cuda")
    total = torch.zeros(D, dtype=torch.float64, device="cuda")
    total32 = torch.zeros(D, dtype=torch.float64, device="cuda")
    for i in range(rows):
        e, s, g = _floats(D, seed, WORKER_ERR, i), _floats(L.S, seed, WORKER_SCALES, i), grad(i)
        z32 = (c1 * m32 + d1 * g.float()) + _error(e, L.spread(s))
        z = c1 * m32.double() + d1 * g.double() + _error(e.double(), L.spread(s.double()))
        werr[i] = torch.where(L.real, z, e.double())
        wscales[i] = L.scales(z)
        if kind != "share":
            sign = torch.where(z32 >= 0, 1.0, -1.0).double()
            total += sign * L.spread(wscales[i])
            total32 += sign * L.spread(wscales[i].float().double())
    out = {"worker_err": werr, "worker_bits": None, "worker_scales": wscales, "server_bits": None}

    # the chunk owners
    own = L.real
    if kind == "share":
        j = case["chunk"]
        segs = _segments(case)
        mine = [q for q in range(L.S) if segs[q][1] == j]
        owns = torch.zeros(L.S, dtype=torch.bool, device="cuda")
        owns[torch.tensor(mine, device="cuda")] = True
        own = own & owns[L.seg]
        if len(_numel(case)) == 1:
            b, e = segs[j][2], segs[j][3]
            cols = max((e - b + 63) // 64, 1)
            ins = _floats(n, seed, IN_SCALES)
            for i in range(n):
                sign = _signs(_words(cols, seed, IN_BITS, i), cols * 64)[:e - b]
                total[b:e] += sign.double() * float(ins[i])
        else:
            for i in range(n):
                sign = _signs(_words(D // 64, seed, IN_BITS, i), D)
                total += sign.double() * L.spread(_floats(L.S, seed, IN_SCALES, i).double())
        total32 = total
    zs = total / n + _error(sserr.double(), L.spread(sscales.double()))
    zs32 = (total32 / n).float() + _error(sserr, L.spread(sscales))
    new = L.scales(zs)
    if kind == "share":
        new = torch.where(owns, new, sscales.double())
    sign = torch.where(own, torch.where(zs32 >= 0, 1.0, -1.0), msign).double()
    out["server_err"] = torch.where(own, zs, sserr.double())
    out["server_scales"] = new
    mbar = sign * L.spread(new)
    if kind == "naive":
        m = _floats(D, seed, M).double()
        m1 = b1 * m + o1 * mbar
        v1 = b2 * v + o2 * mbar * mbar
        x1 = x - lr * m1 / (v1.sqrt() + eps)
        out["m"], out["v"] = torch.where(L.real, m1, m), torch.where(L.real, v1, v)
    else:
        x1 = x - lr * mbar / (v + eps).sqrt()
        if kind == "step" and not case["packed"]:
            out["m"] = torch.where(L.real, mbar, _floats(D, seed, M).double())
    out["x"] = torch.where(L.real, x1, x)
    return out
