"""Host-side logic of the Python binding (no GPU, but for the last test): the per-chunk word ranges
that size a chunk owners' call, against brute force, and their per-call cost
on the 5,000-tensor stress layout; the paired gradient and error rows that
State allocates."""
import time

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2102_02888_amd.onebit import chunk_extent, chunk_word_ranges


def _brute_extent(L, sb, se):
    """Every owned non-empty segment visited one by one."""
    wlo, whi = -1, -1
    for k in range(L.K):
        for j in range(sb, se):
            q = k * L.n + j
            b, e = int(L.seg_begin[q]), int(L.seg_end[q])
            if e > b:
                wlo = b // 64 if wlo < 0 else min(wlo, b // 64)
                whi = max(whi, (e - 1) // 64)
    return wlo, whi, (L.K - 1) * L.n + se - 1


@pytest.mark.parametrize("numel,n", [
    ([1], 1), ([64], 3), ([5000, 70_001, 64, 0, 300], 4), ([0, 0, 10], 5),
    ([200, 1, 129, 64 * 33 + 1, 7], 33), ([10 ** 6], 32), ([0], 2),
])
def test_chunk_extent_matches_brute_force(numel, n):
    L = oracle.Layout(numel, n)
    lo, hi = chunk_word_ranges(L.seg_begin, L.seg_end, L.K, L.n)
    for sb in range(n):
        for se in range(sb + 1, n + 1):
            assert chunk_extent(lo, hi, L.K, L.n, sb, se) == _brute_extent(L, sb, se), (sb, se)


def test_chunk_extent_cost_on_stress_layout():
    """40,000 segments: the ranges are built once per plan and each chunk
    owners' call costs O(n) host work, far below one kernel's time."""
    wl = synth.get("stress")
    L = oracle.Layout(wl.numel, wl.n)
    t0 = time.perf_counter()
    lo, hi = chunk_word_ranges(L.seg_begin, L.seg_end, L.K, L.n)
    build_s = time.perf_counter() - t0
    assert build_s < 0.5, build_s
    calls = 2000
    t0 = time.perf_counter()
    for _ in range(calls):
        ext = chunk_extent(lo, hi, L.K, L.n, 0, L.n)
    per_call_ms = (time.perf_counter() - t0) * 1e3 / calls
    assert per_call_ms < 0.1, per_call_ms
    assert ext == _brute_extent(L, 0, L.n)
    for j in (0, 3, L.n - 1):
        assert chunk_extent(lo, hi, L.K, L.n, j, j + 1) == _brute_extent(L, j, j + 1)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_paired_rows_layout(dtype):
    """State's gradient and error rows share one allocation: row i holds D
    gradients and then D fp32 errors.  The views have the shapes and leading
    dimensions the ABI is given, every row starts 16-byte aligned, and a
    worker's two rows do not overlap each other or the next worker's."""
    from paper_2102_02888_amd.onebit import paired_rows
    n, D = 5, 192
    g, e = paired_rows(n, D, dtype, "cpu")
    gs = g.element_size()
    assert g.dtype == dtype and e.dtype == torch.float32
    assert g.shape == (n, D) and e.shape == (n, D)
    row_bytes = (gs + 4) * D
    assert g.stride() == (row_bytes // gs, 1) and e.stride() == (row_bytes // 4, 1)
    base = g.data_ptr()
    for i in range(n):
        g0, e0 = g[i].data_ptr() - base, e[i].data_ptr() - base
        assert g0 == i * row_bytes and e0 == i * row_bytes + gs * D
        assert g0 % 16 == 0 and e0 % 16 == 0
    g.fill_(1)
    assert float(e.abs().sum()) == 0.0
    e.fill_(2)
    assert bool((g == 1).all())
    with pytest.raises(ValueError):
        paired_rows(n, 100, dtype, "cpu")
    with pytest.raises(ValueError):
        paired_rows(n, 0, dtype, "cpu")


@pytest.mark.parametrize("make", [
    lambda: torch.zeros(10), lambda: torch.zeros(0), lambda: torch.zeros(()),
    lambda: torch.zeros(4, 64), lambda: torch.zeros(0, 64), lambda: torch.zeros(3, 130)[:, 64:128],
    lambda: torch.zeros(64, 4).t(), lambda: torch.zeros(20)[::2], lambda: torch.zeros(2, 2, 64),
    lambda: torch.zeros(4, 64, dtype=torch.float64), lambda: torch.zeros(128)[3:],
    lambda: torch.zeros(1, 64).expand(4, 64), lambda: torch.nn.Parameter(torch.zeros(64)),
    lambda: torch.zeros(4, 64, device="meta"), lambda: None, lambda: 5, lambda: np.zeros(64),
])
@pytest.mark.parametrize("cols,rows", [(None, 1), (64, 1), (64, 4), (65, 1), (10, 2), (0, 1)])
def test_native_argument_checks_accept_what_the_binding_does(make, cols, rows):
    """pointer() gives the data pointer exactly where the one-by-one checks
    accept a tensor (their device check left out here), else -1."""
    from paper_2102_02888_amd._native import args_module
    pointer = args_module().pointer
    t = make()
    want = -1
    if isinstance(t, torch.Tensor) and t.dtype == torch.float32 and t.dim() <= 2 \
            and (t.dim() == 0 or t.stride(-1) == 1):
        have = tuple(t.shape) if t.dim() == 2 else (1, t.numel())
        if cols is None or (have[0] >= rows and have[1] >= cols):
            want = t.data_ptr()
    args = (t, torch.float32, -1 if cols is None else cols, rows)
    assert pointer(*args, False) == want
    assert pointer(*args, True) == -1  # no GPU tensor


def test_a_failed_check_is_named():
    from paper_2102_02888_amd.onebit import _ptr
    f = torch.float32
    assert _ptr(None, f, "m") is None
    with pytest.raises(TypeError, match="m must be a torch.Tensor"):
        _ptr(np.zeros(4), f, "m")
    with pytest.raises(TypeError, match="m must be torch.float32, got torch.float64"):
        _ptr(torch.zeros(4, dtype=torch.float64), f, "m")
    with pytest.raises(ValueError, match="m must be a GPU tensor"):
        _ptr(torch.zeros(4), f, "m", 4)


def test_argument_checks_are_named_after_the_torch_and_python_they_are_built_for(monkeypatch):
    import sysconfig

    from paper_2102_02888_amd import _native, build
    name = build.args_path()
    assert torch.__version__ in name and name.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(torch, "__version__", "0.0.0+other")
    assert build.args_path() != name
    with pytest.raises(ImportError, match="not built for this torch and Python"):
        _native.args_module()


def test_current_stream_without_torchs_private_function(monkeypatch):
    from paper_2102_02888_amd import onebit

    class Stream:
        cuda_stream = 1234
    monkeypatch.setattr(onebit, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    assert onebit._stream(None) == 1234
    assert onebit._stream(Stream()) == 1234


@pytest.mark.gpu
def test_current_stream_is_torchs():
    from paper_2102_02888_amd import onebit
    for s in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            assert onebit._stream(None) == onebit._stream(s) == torch.cuda.current_stream().cuda_stream
