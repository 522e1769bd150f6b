"""The factored forwards (sfda_chunk_fwd_factored, sfda_chunk_fwd_decoupled_factored) at the edges
of their tiles and steps, against the complex128 oracle: tokens around the 16-token block and the
64-token step, key channels around the 16-channel block, value columns around the scans' 8 and
32 columns; in several pieces, and with a piece's scan beside the next one's preparation
(few heads, many steps), bitwise the same as in one piece.

Bars as for sfda_chunk_fwd: max |x - ref| / max |ref| <= 1e-4 (float32 inputs), <= 2e-2 (bfloat16)."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

from gpu_util import I, ensure_built, rel_err, run_oracle, to_complex, to_device, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return ensure_built()


def say(*a):
    print("[case]", *a, flush=True)


def factored(lib, x):
    """sfda_chunk_fwd_factored through the C entry (every dtype), its workspace poisoned."""
    import torch
    from paper_2607_11897_amd import sfda
    d = upload(x)
    B, H, T, m, n = x.shape
    code = sfda.SFDA_F32 if x.dtype == "f32" else sfda.SFDA_BF16
    need = lib.sfda_chunk_fwd_factored_workspace_bytes(B, H, T, m, n, code, 0)
    assert need > 0
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")     # NaN, whatever the type
    o = torch.full((B, H, T, n, 2), float("nan"), device="cuda", dtype=d["q"].dtype)
    S = torch.full((B, H, m, n, 2), float("nan"), device="cuda")
    p = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())
    st = lib.sfda_chunk_fwd_factored(p(d["q"]), p(d["k"]), p(d["v"]), p(d["alpha"]), p(d["theta"]), p(d["beta"]),
                                     p(d["S0"]), p(o), p(S), B, H, T, m, n, 64, code, code, p(ws), need,
                                     ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    torch.cuda.synchronize()
    return to_complex(o), to_complex(S)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,T,m,n", [
    (1, 1, 1, 64, 64), (1, 2, 16, 16, 8), (2, 5, 17, 17, 9), (1, 3, 63, 33, 33), (1, 8, 64, 48, 32),
    (3, 3, 65, 64, 65), (1, 9, 129, 5, 7), (1, 2, 200, 47, 1), (1, 1, 130, 3, 40), (2, 1, 96, 62, 96),
])
def test_factored_edges(lib, B, H, T, m, n, dtype):
    x = I.make_chunk_inputs(I.Workload("edge", B, H, T, m, n, 64, dtype, I.LAWS_MAIN, 900 + T + m, 1e-4))
    say("factored", (B, H, T, m, n), dtype)
    o, S = factored(lib, x)
    o_ref, S_ref = run_oracle(x)
    tol = 1e-4 if dtype == "f32" else 2e-2
    eo, es = rel_err(o, o_ref), rel_err(S, S_ref)
    say("err(o)", eo, "err(S_T)", es)
    assert eo <= tol and es <= tol


@pytest.mark.parametrize("B,H,T,m,n,G", [
    (1, 3, 768, 40, 24, 1),       # 2 * 3 * 3 workgroups at most: pieces with the next one prepared beside
    (1, 64, 640, 64, 64, 1),      # 512 workgroups: pieces one after the other
])
def test_factored_pieces_bitwise(lib, B, H, T, m, n, G):
    """sfda_chunk_fwd_segmented's workspace holds the records of a part of the sequence only: the
    result is bitwise that of the workspace that holds them all."""
    import torch
    from paper_2607_11897_amd import sfda
    x = I.make_chunk_inputs(I.Workload("pieces", B, H, T, m, n, 64, "f32", I.LAWS_LONG, 950, 1e-4))
    d = upload(x)
    args = (d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"])
    small = sfda.segmented_workspace_bytes(B, H, T, m, n, G)
    assert small < lib.sfda_chunk_fwd_factored_workspace_bytes(B, H, T, m, n, 0, 0)
    say("pieces", (B, H, T, m, n))
    o1, S1 = sfda.chunk_fwd(*args, C=64)
    o2, S2 = sfda.chunk_fwd(*args, C=64, segments=G)
    o3, _ = sfda.chunk_fwd(*args, C=64, segments=G, want_state=False)     # the state carried in the workspace
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and torch.equal(S1, S2) and torch.equal(o1, o3)
    x0 = x.head(0, H - 1)
    o_ref, S_ref = run_oracle(x0)
    assert rel_err(to_complex(o1)[:1, H - 1:], o_ref) <= 1e-4 and rel_err(to_complex(S1)[:1, H - 1:], S_ref) <= 1e-4


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,m,n", [(1, 16, 8), (33, 17, 33), (64, 64, 64), (131, 50, 7)])
def test_decoupled_edges(T, m, n, dtype):
    from test_gpu_decoupled import oracle_dec, run_dec
    x = I.make_decoupled_inputs(1, 9, T, m, n, dtype, seed=970 + T)
    say("decoupled", (T, m, n), dtype)
    o, S = run_dec(x, 16)
    o_ref, S_ref = oracle_dec(x)
    tol = 1e-4 if dtype == "f32" else 2e-2
    assert rel_err(o, o_ref) <= tol and rel_err(S, S_ref) <= tol


@pytest.mark.parametrize("field,bad", [("theta", float("nan")), ("theta", float("inf")), ("alpha", 1e-39)])
def test_bad_gate_gives_nan_from_its_block_on(lib, field, bad):
    """A phase that is not finite, or a decay below the block range: NaN from that 16-token block
    on and in S_T, the blocks before it untouched."""
    x = I.make_chunk_inputs(I.Workload("bad", 1, 2, 100, 20, 12, 64, "f32", I.LAWS_MAIN, 990, 1e-4))
    o_ref, _ = run_oracle(x)
    a = getattr(x, field).copy()
    a[0, 1, 53, 7] = bad                                  # block 3 of head 1
    import dataclasses
    o, S = factored(lib, dataclasses.replace(x, **{field: a}))
    say("bad", field, bad)
    assert np.all(np.isnan(o[0, 1, 48:])) and np.all(np.isnan(S[0, 1]))
    assert rel_err(o[0, 1, :48], o_ref[0, 1, :48]) <= 1e-4 and rel_err(o[0, 0], o_ref[0, 0]) <= 1e-4
    assert np.all(np.isfinite(S[0, 0]))


@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("f32", "bf16"), ("bf16", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("B,H,T,m,n", [
    (2, 4, 1, 64, 64), (1, 2, 49, 16, 8), (2, 5, 48, 17, 9), (1, 3, 63, 33, 33), (1, 8, 64, 48, 32),
    (3, 3, 65, 64, 65), (1, 9, 129, 5, 7), (1, 2, 200, 47, 1), (1, 1, 130, 3, 40), (2, 1, 96, 62, 96),
])
def test_backward_edges(lib, B, H, T, m, n, dtype, out):
    """sfda_chunk_bwd with the workspace of its scans on prepared operands and with the smaller
    one (scans in place), each poisoned: both against the oracle, at the bars of the backward's tests
    (1e-4 float32, 2e-2 bfloat16 inputs or dL/do).  Those are relative to a gradient's largest
    entry, so no case has one token alone: its one dbeta is a sum of n products of either sign, each
    in error by up to 2^-8 of its size, and nothing bounds the sum from below."""
    import torch
    from oracle import backward as BW
    from paper_2607_11897_amd import sfda
    x = I.make_chunk_inputs(I.Workload("edge", B, H, T, m, n, 64, dtype, I.LAWS_MAIN, 970 + T + m, 1e-4))
    dO, dS = I.make_cotangents(B, H, T, m, n, out, seed=980 + T)
    d = upload(x)
    dO_t, dS_t = to_device(I.to_storage(dO, out), out), to_device(I.to_storage(dS, "f32"), "f32")
    ref = BW.recurrence_backward(x.q, x.k, x.v, x.alpha, x.theta, x.beta, x.S0, dO, dS)
    code = sfda.SFDA_F32 if dtype == "f32" else sfda.SFDA_BF16
    full = lib.sfda_chunk_bwd_auto_workspace_bytes(B, H, T, m, n, 64, code)
    least = sfda.bwd_workspace_bytes(B, H, T, m, n, 64)
    assert full >= least > 0                           # (equal: in place alone, or alone on prepared operands)
    tol = 2e-2 if "bf16" in (dtype, out) else 1e-4
    for size in {full, least}:
        say("backward", (B, H, T, m, n), dtype, out, size)
        g = sfda.chunk_bwd(d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"], dO_t, dS_t,
                           workspace=torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        errs = {}
        for name, t in g.items():
            got = to_complex(t) if t.shape[-1] == 2 and name in ("dq", "dk", "dv", "dS0") else t.double().cpu().numpy()
            assert np.all(np.isfinite(got)), name
            errs[name] = rel_err(got, ref[name])
        say({k: f"{e:.2e}" for k, e in errs.items()})
        assert max(errs.values()) <= tol, errs


class _Handle:
    """A stream of some other library: only its handle."""
    def __init__(self, h):
        self.cuda_stream = h


@pytest.mark.parametrize("wrap", [lambda s: s, lambda s: _Handle(s.cuda_stream)])
def test_streams_given_as_objects(lib, wrap):
    """Whatever has a cuda_stream is taken as the stream, also where the call allocates a workspace
    on it; the workspace then belongs to that stream."""
    import torch
    from paper_2607_11897_amd import sfda
    x = I.make_chunk_inputs(I.Workload("stream", 1, 2, 130, 16, 8, 64, "f32", I.LAWS_MAIN, 960, 1e-4))
    d = upload(x)
    args = [d[k] for k in ("q", "k", "v", "alpha", "theta", "beta", "S0")]
    o, S = sfda.chunk_fwd(*args)
    g = sfda.chunk_bwd(*args, o, S)
    dec = sfda.chunk_fwd_decoupled(args[0], args[1], args[1], *args[2:5], args[5], args[5], args[6])
    torch.cuda.synchronize()
    say("streams")
    side = torch.cuda.Stream()
    st = wrap(side)
    o2, S2 = sfda.chunk_fwd(*args, stream=st)
    g2 = sfda.chunk_bwd(*args, o, S, stream=st)
    dec2 = sfda.chunk_fwd_decoupled(args[0], args[1], args[1], *args[2:5], args[5], args[5], args[6], stream=st)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(S, S2) and all(torch.equal(g[k], g2[k]) for k in g)
    assert all(torch.equal(a, b) for a, b in zip(dec, dec2))


def test_backward_rows_keep_32_bits(lib):
    """bfloat16 inputs: G_F is recorded in 32 bits.  One key channel, alpha 1, theta 0, beta 0 and
    no state: G_F of a token is dS_T plus the last token's dL/do, here 1 + 2^-10 and 1 in two columns
    whose v are 1 and -1, every product exact; dbeta = 2^-10 in the last block, 0 from rows rounded
    to bfloat16."""
    import torch
    from paper_2607_11897_amd import sfda
    T, m, n = 64, 16, 16
    bf = dict(dtype=torch.bfloat16, device="cuda")
    q = torch.zeros(1, 1, T, m, 2, **bf)
    q[..., 0, 0] = 1
    v, dO = torch.zeros(1, 1, T, n, 2, **bf), torch.zeros(1, 1, T, n, 2, **bf)
    v[..., 0, 0], v[..., 1, 0], dO[0, 0, -1, 0, 0] = 1, -1, 2.0 ** -10
    dS = torch.zeros(1, 1, m, n, 2, device="cuda")
    dS[0, 0, 0, :2, 0] = 1
    least = sfda.bwd_workspace_bytes(1, 1, T, m, n, 64)
    assert sfda.bwd_auto_workspace_bytes(1, 1, T, m, n, 64, "bf16") > least
    say("rows in 32 bits")
    g = sfda.chunk_bwd(q, q.clone(), v, torch.ones(1, 1, T, m, **bf), torch.zeros(1, 1, T, m, **bf),
                       torch.zeros(1, 1, T, **bf), None, dO, dS)
    torch.cuda.synchronize()
    assert torch.equal(g["dbeta"][0, 0, -16:].float().cpu(), torch.full((16,), 2.0 ** -10))


@pytest.mark.parametrize("dtype,B,H,T,m,n,decoupled,want", [
    ("f32", 1, 4, 48, 64, 64, 0, 0), ("f32", 1, 4, 49, 64, 64, 0, 1), ("f32", 1, 4, 33, 64, 64, 1, 1),
    ("f32", 1, 96, 96, 64, 64, 0, 0), ("f32", 1, 96, 97, 64, 64, 0, 1), ("f32", 4, 64, 512, 64, 64, 0, 0),
    ("f32", 4, 64, 512, 16, 64, 0, 1), ("bf16", 1, 32, 255, 64, 64, 0, 0), ("bf16", 1, 32, 256, 64, 64, 0, 1),
    ("bf16", 1, 48, 639, 64, 64, 0, 0), ("bf16", 1, 64, 1537, 64, 64, 0, 0), ("bf16", 1, 64, 1537, 64, 32, 0, 1), ("bf16", 1, 64, 1537, 48, 64, 0, 0), ("bf16", 1, 65, 1024, 64, 64, 0, 0),
    ("bf16", 1, 12, 4096, 64, 64, 0, 0), ("bf16", 1, 12, 4095, 64, 64, 0, 1), ("bf16", 1, 48, 1024, 64, 97, 0, 0),
    ("bf16", 8, 16, 48, 64, 64, 1, 0), ("bf16", 8, 16, 49, 64, 64, 1, 1),
])
def test_rule_and_both_paths(lib, dtype, B, H, T, m, n, decoupled, want):
    """The rule at its edges; where it takes a bfloat16 or float32 forward to prepared operands, the
    default's result is the factored entry's, bit for bit, and the in-place one's to rounding (twice
    the bar against the oracle: each within it)."""
    import torch
    from paper_2607_11897_amd import sfda
    code = sfda.SFDA_F32 if dtype == "f32" else sfda.SFDA_BF16
    assert lib.sfda_chunk_fwd_auto_factored(B, H, T, m, n, 64, code, decoupled) == want
    if decoupled or not want or B * H * T > 32 * 1024:
        return
    x = I.make_chunk_inputs(I.Workload("rule", B, H, T, m, n, 64, dtype, I.LAWS_MAIN, 990 + T, 1e-4))
    say("rule", (B, H, T, m, n), dtype)
    d = upload(x)
    args = (d["q"], d["k"], d["v"], d["alpha"], d["theta"], d["beta"], d["S0"])
    o, S = sfda.chunk_fwd(*args)
    o1, S1 = sfda.chunk_fwd(*args, segments=None)
    of, Sf = factored(lib, x)
    torch.cuda.synchronize()
    assert np.array_equal(to_complex(o), of) and np.array_equal(to_complex(S), Sf)
    tol = 2 * (1e-4 if dtype == "f32" else 2e-2)
    assert rel_err(of, to_complex(o1)) <= tol and rel_err(Sf, to_complex(S1)) <= tol
