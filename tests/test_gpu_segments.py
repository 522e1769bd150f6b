"""GPU parity of sfda_chunk_fwd_segmented (each head's sequence scanned as G parallel
segments, joined by the affine law of a segment, Thm 4.4, composed along the segments,
Lemma A.2) against the complex128 oracle recurrence, and against sfda_chunk_fwd.

Bars as for sfda_chunk_fwd: max-norm relative error <= 1e-4 for float32 inputs, <= 2e-2
for bfloat16 inputs, on o and on S_T.  The long-context workload runs at full size with
the segments the benchmark uses and is checked on sampled heads over prefix windows.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import I, ensure_built, rel_err, run_oracle, to_complex, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return ensure_built()


def say(*a):
    print("[case]", *a, flush=True)


def run(x, C, G, in_place=False):
    import torch
    from paper_2607_11897_amd import sfda
    d = upload(x)
    S0 = d["S0"]
    S_T = S0 if (in_place and S0 is not None) else None
    o, S = sfda.chunk_fwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], S0, C=C,
                          segments=G, S_T=S_T)
    torch.cuda.synchronize()
    return to_complex(o), to_complex(S)


def run_plain(x, C):
    import torch
    from paper_2607_11897_amd import sfda
    d = upload(x)
    o, S = sfda.chunk_fwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"], C=C,
                          segments=None)
    torch.cuda.synchronize()
    return to_complex(o), to_complex(S)


def make(B, H, T, m, n, C, dtype="f32", zero_state=False, seed=21):
    w = I.Workload("seg", B, H, T, m, n, C, dtype, I.LAWS_MAIN, seed, 1e-4)
    x = I.make_chunk_inputs(w)
    if zero_state:
        x = x.__class__(x.q, x.k, x.v, x.alpha, x.theta, x.beta, None, x.dtype)
    return x


@pytest.mark.parametrize("B,H,T,m,n,C,G", [
    (1, 2, 128, 64, 64, 16, 4),
    (2, 1, 96, 33, 24, 16, 3),
    (1, 3, 256, 64, 80, 32, 2),
    (1, 1, 64, 16, 8, 16, 1),
    (1, 2, 512, 64, 64, 64, 8),
    (3, 1, 192, 5, 3, 64, 3),
])
def test_segmented_f32(B, H, T, m, n, C, G):
    x = make(B, H, T, m, n, C)
    say("f32", (B, H, T, m, n), "C", C, "G", G)
    o, S = run(x, C, G)
    o_ref, S_ref = run_oracle(x)
    eo, es = rel_err(o, o_ref), rel_err(S, S_ref)
    op, Sp = run_plain(x, C)
    say("err(o)", eo, "err(S_T)", es, "vs plain", rel_err(o, op), rel_err(S, Sp))
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(S))
    assert eo <= 1e-4 and es <= 1e-4


@pytest.mark.parametrize("m,n,G", [(64, 40, 4), (21, 64, 2)])
def test_segmented_f32_in_bf16_out(m, n, G):
    """float32 inputs, bfloat16 output: o within the bf16 bar, S_T (float32) within 1e-4."""
    import torch
    from paper_2607_11897_amd import sfda
    x = make(2, 1, 256, m, n, 16, seed=17)
    say("f32 -> bf16", (2, 1, 256, m, n), "G", G)
    d = upload(x)
    o, S = sfda.chunk_fwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"], C=16,
                          segments=G, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    o, S = to_complex(o), to_complex(S)
    o_ref, S_ref = run_oracle(x)
    eo, es = rel_err(o, o_ref), rel_err(S, S_ref)
    say("err(o)", eo, "err(S_T)", es)
    assert eo <= 2e-2 and es <= 1e-4


@pytest.mark.parametrize("dtype,G", [("f32", 4), ("bf16", 8)])
def test_segmented_strong_decay(dtype, G):
    """alpha ~ U(0.02, 0.1): a segment's transfer decays to far below the float range (its
    product P_g and the readouts X_t underflow to zero after a few chunks) and each 16-token
    block stays inside it; o and S_T within the bars (float32: the segment forward and the
    join; bfloat16: three passes)."""
    import math
    laws = I.Laws(alpha=("uniform", 0.02, 0.1), theta=("uniform", -math.pi, math.pi),
                  beta=("uniform", 0.0, 1.0), s0_scale=0.1)
    w = I.Workload("seg_strong", 1, 2, 512, 64, 48, 16, dtype, laws, 23, 1e-4)
    x = I.make_chunk_inputs(w)
    say(dtype, "strong decay, G", G)
    o, S = run(x, 16, G)
    o_ref, S_ref = run_oracle(x)
    eo, es = rel_err(o, o_ref), rel_err(S, S_ref)
    say("err(o)", eo, "err(S_T)", es)
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert np.all(np.isfinite(o)) and np.all(np.isfinite(S))
    assert eo <= tol and es <= tol


def test_segmented_zero_state_and_in_place():
    x = make(1, 2, 128, 64, 64, 16, zero_state=True)
    o, S = run(x, 16, 4)
    o_ref, S_ref = run_oracle(x)
    assert rel_err(o, o_ref) <= 1e-4 and rel_err(S, S_ref) <= 1e-4
    x = make(1, 2, 128, 64, 64, 16, seed=5)
    o, S = run(x, 16, 4, in_place=True)          # S_T written over S0
    o_ref, S_ref = run_oracle(x)
    say("in place: err(o)", rel_err(o, o_ref), "err(S_T)", rel_err(S, S_ref))
    assert rel_err(o, o_ref) <= 1e-4 and rel_err(S, S_ref) <= 1e-4


@pytest.mark.parametrize("C,G", [(64, 4), (32, 8), (16, 2)])
def test_segmented_bf16(C, G):
    x = make(1, 2, 512, 64, 64, C, dtype="bf16")
    say("bf16 C", C, "G", G)
    o, S = run(x, C, G)
    o_ref, S_ref = run_oracle(x)
    eo, es = rel_err(o, o_ref), rel_err(S, S_ref)
    say("err(o)", eo, "err(S_T)", es)
    assert eo <= 2e-2 and es <= 2e-2


def test_segmented_shape_error_launches_nothing():
    import torch
    from paper_2607_11897_amd import sfda
    x = make(1, 1, 96, 16, 8, 16)
    d = upload(x)
    with pytest.raises(sfda.SfdaError):
        sfda.chunk_fwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"], C=16,
                       segments=4)          # 96 is not a multiple of 4 * 16
    torch.cuda.synchronize()


def test_long_f32_h16_t64k_segmented_sampled_heads():
    """The long-context workload with 16 segments per head (the benchmarked setting): error
    of o over prefix windows and of S_T for two heads."""
    w = I.WORKLOADS["long_f32_h16_t64k"]
    say(w.name, "generating")
    x = I.make_chunk_inputs(w)
    say(w.name, "running, 16 segments")
    o, S = run(x, w.C, 16)
    for h in (0, 9):
        o_ref, S_ref = run_oracle(x.head(0, h))
        errs = {2 ** lg: rel_err(o[0, h, :2 ** lg], o_ref[0, 0, :2 ** lg]) for lg in range(10, 17)}
        es = rel_err(S[0, h], S_ref[0, 0])
        say(w.name, "head", h, "err(o) by prefix", errs, "err(S_T)", es)
        assert max(errs.values()) <= w.tol and es <= w.tol


def _policy(B, H, T, m, n, C, cus, dtype):
    """The segment count rule of sfda_chunk_fwd_auto_segments, restated."""
    per = B * H * ((n + 63) // 64)
    G = 1
    while G < 1024 and per * 2 * G <= cus and T % (2 * G * C) == 0 and T // (2 * G) >= 256:
        G *= 2
    return G if G >= (4 if dtype == "f32" else 8) else 1


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,T,m,n,C", [
    (4, 8, 2048, 64, 64, 64),       # the float32 workload: 32 heads
    (8, 16, 4096, 64, 64, 64),      # the benchmarked bf16 workload: enough heads, no segments
    (1, 16, 65536, 64, 64, 64),     # long context
    (4, 16, 4096, 64, 64, 64),      # 64 heads: G = 4, segments for float32 only
    (1, 2, 4096, 64, 64, 64),
    (1, 2, 4000, 64, 64, 64),       # T not a multiple of 8 C: no segments
    (1, 1, 1024, 64, 130, 16),
])
def test_auto_segments_policy(B, H, T, m, n, C, dtype):
    import torch
    from paper_2607_11897_amd import sfda
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    G = sfda.auto_segments(B, H, T, m, n, C, dtype)
    say("auto segments", (B, H, T, m, n, C), dtype, "CUs", cus, "G", G)
    assert G == _policy(B, H, T, m, n, C, cus, dtype)
    if cus >= 256 and (B, H, T) == (4, 8, 2048):
        assert G == 8
    if (B, H, T) == (8, 16, 4096):
        assert G == 1


@pytest.mark.parametrize("dtype,H,T", [("f32", 2, 16384), ("bf16", 12, 4096)])
def test_default_picks_segments_for_few_heads(dtype, H, T):
    """chunk_fwd's default on a few heads over a long sequence runs the segmented scan the policy
    picks: the same bits as asking for that G, and the oracle's result within the bar."""
    import torch
    from paper_2607_11897_amd import sfda
    x = make(1, H, T, 64, 64, 64, dtype=dtype)
    G = sfda.auto_segments(1, H, T, 64, 64, dtype=dtype)
    say("default segments", dtype, G)
    assert G > 1 and sfda.load_library().sfda_chunk_fwd_auto_factored(1, H, T, 64, 64, 64, int(dtype == "bf16"), 0) == 0
    d = upload(x)
    o1, S1 = sfda.chunk_fwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"], C=64)
    o2, S2 = sfda.chunk_fwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"], C=64,
                            segments=G)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(S1, S2)
    o_ref, S_ref = run_oracle(x.head(0, H - 1))
    eo, es = rel_err(to_complex(o1)[:, H - 1:], o_ref), rel_err(to_complex(S1)[:, H - 1:], S_ref)
    say("default segments err(o)", eo, "err(S_T)", es)
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert eo <= tol and es <= tol


def _segments_and_factored(x, C, G, out_dtype=None, in_place=False):
    """chunk_fwd over G segments, and the factored forward's result (C entry)."""
    import ctypes
    import torch
    from paper_2607_11897_amd import sfda
    lib = sfda.load_library()
    d = upload(x)
    args = (d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"])
    B, H, T, m, n = x.shape
    od = torch.bfloat16 if out_dtype == "bf16" else torch.float32
    need = lib.sfda_chunk_fwd_factored_workspace_bytes(B, H, T, m, n, 0, 0)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    of = torch.full((B, H, T, n, 2), float("nan"), device="cuda", dtype=od)
    Sf = torch.full((B, H, m, n, 2), float("nan"), device="cuda")
    p = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())
    assert lib.sfda_chunk_fwd_factored(*map(p, args), p(d["S0"]), p(of), p(Sf), B, H, T, m, n, C, 0, int(od == torch.bfloat16),
                                       p(ws), need, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    o = torch.full_like(of, float("nan"))
    o, S = sfda.chunk_fwd(*args, d["S0"], C=C, segments=G, o=o, out_dtype=od, S_T=d["S0"] if in_place else None)
    torch.cuda.synchronize()
    return o, S, of, Sf


STRONG = I.Laws(alpha=("uniform", 0.02, 0.1), theta=("uniform", -3.14159, 3.14159), beta=("uniform", 0.0, 1.0),
                s0_scale=0.1)


@pytest.mark.parametrize("B,H,T,m,n,C,G,out,laws", [
    (1, 1, 4096, 16, 16, 64, 16, "f32", I.LAWS_MAIN),
    (1, 2, 1024, 5, 3, 16, 8, "f32", I.LAWS_MAIN),          # ragged channels and columns
    (2, 1, 8192, 33, 33, 64, 32, "f32", I.LAWS_MAIN),
    (1, 1, 8192, 64, 64, 64, 32, "f32", I.LAWS_LONG),
    (1, 1, 8192, 17, 72, 64, 32, "f32", I.LAWS_MAIN),       # past 64 columns: two passes
    (1, 1, 4096, 12, 24, 16, 16, "f32", STRONG),            # transfers below the float range
    (1, 2, 8192, 20, 9, 64, 32, "bf16", I.LAWS_MAIN),       # bfloat16 o: a third pass, rounded once
    (1, 1, 8192, 8, 80, 64, 32, "bf16", I.LAWS_MAIN),
])
def test_few_heads_long_sequences_run_segments(B, H, T, m, n, C, G, out, laws):
    """float32 where G segments are faster than one scan on prepared operands: other bits than the
    factored forward's, both within the bar of the oracle, and of each other (float32: each within
    2e-6 relative 2-norm at these lengths; bfloat16 o: one rounding each, 2^-8 of the value)."""
    import torch
    x = I.make_chunk_inputs(I.Workload("seg_long", B, H, T, m, n, C, "f32", laws, 31, 1e-4))
    say((B, H, T, m, n), "C", C, "G", G, out)
    o, S, of, Sf = _segments_and_factored(x, C, G, out, in_place=True)
    assert not torch.equal(S, Sf)                           # (the factored forward would give these bits)
    rel = lambda a, b: float((a.double() - b.double()).norm() / b.double().norm())
    say("o", rel(o, of), "S", rel(S, Sf))
    assert rel(o, of) <= (4e-6 if out == "f32" else 2 ** -8) and rel(S, Sf) <= 4e-6
    o_ref, S_ref = run_oracle(x)
    assert rel_err(to_complex(o), o_ref) <= (1e-4 if out == "f32" else 2 ** -8) and rel_err(to_complex(S), S_ref) <= 1e-4


def test_default_float32_long_few_heads():
    """The default takes segments where they are faster, and the prepared operands elsewhere."""
    import torch
    from paper_2607_11897_amd import sfda
    lib = sfda.load_library()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus == 256:
        for heads, T, m, n, want in ((1, 65536, 64, 64, 0), (1, 16384, 64, 64, 0), (1, 4096, 64, 64, 1), (16, 65536, 64, 64, 1),
                                     (4, 4096, 16, 16, 0), (4, 2048, 16, 16, 1), (16, 65536, 16, 16, 0), (32, 16384, 64, 64, 1)):
            assert lib.sfda_chunk_fwd_auto_factored(1, heads, T, m, n, 64, 0, 0) == want, (heads, T, m, n)
    x = I.make_chunk_inputs(I.Workload("seg_default", 1, 1, 16384, 8, 8, 64, "f32", I.LAWS_LONG, 33, 1e-4))
    d = upload(x)
    args = (d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"])
    G = sfda.auto_segments(1, 1, 16384, 8, 8)
    say("default, segments", G)
    assert G > 1
    o1, S1 = sfda.chunk_fwd(*args)
    o2, S2 = sfda.chunk_fwd(*args, segments=G)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(S1, S2)
    o_ref, S_ref = run_oracle(x)
    assert rel_err(to_complex(o1), o_ref) <= 1e-4 and rel_err(to_complex(S1), S_ref) <= 1e-4
