"""C ABI checks that need no GPU: the library loads, exports every symbol the
header declares, sizes its workspace, and rejects bad arguments before any
launch (fake, never dereferenced, aligned pointers are used)."""
import ctypes
import os
import re

import pytest

from paper_2606_08804_amd import qdelta

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "qdelta.h")


def header_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(qdelta_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = qdelta.lib()
    names = header_functions()
    assert len(names) == 23
    for n in names:
        assert hasattr(L, n), n
    assert sorted(names) == sorted(qdelta.EXPORTS)


def test_status_strings_and_version():
    L = qdelta.lib()
    for s in range(5):
        assert L.qdelta_status_string(s)
    assert L.qdelta_status_string(99) == b"unknown status"
    assert L.qdelta_version() >= 10000


def test_saved_state_slots():
    assert qdelta.saved_state_slots(4, 4096) == 4 * 64
    assert qdelta.saved_state_slots(2, 65) == 4
    assert qdelta.saved_state_slots(1, 0) == 0
    assert qdelta.saved_state_slots(1, 32768, 20) == 512 + 20
    assert qdelta.lib().qdelta_saved_state_slots(1, 64, 32, 0) == 0   # chunk 32 unsupported


def test_saved_context_bytes():
    # per (slot, head): Dv x Dk state, C x Dv new values D, fp32 gate block
    # (b, beta, lambda: 3 x C), P and M (the ten 16 x 16 blocks on and below
    # the diagonal of C x C), all but the gates in the activation dtype; plus
    # one 1 KB zero block
    def per_unit(Dk, Dv, e):
        return Dk * Dv * e + 64 * Dv * e + 3 * 64 * 4 + 2 * 10 * 256 * e
    assert qdelta.saved_bytes(4, 4096, 16, 128, 128, 1) == 256 * 16 * per_unit(128, 128, 2) + 1024
    assert qdelta.saved_bytes(1, 100, 2, 64, 64, 0) == 2 * 2 * per_unit(64, 64, 4) + 1024
    assert qdelta.saved_bytes(4, 4096, 16, 96, 128, 1) == 0


def test_workspace_sizes_monotone_and_zero_for_unsupported():
    ws = qdelta.workspace_bytes
    a = ws(4, 4096, 16, 128, 128, 1)
    b = ws(4, 4096, 16, 128, 128, 1, is_bwd=True)
    assert 0 < a < b
    assert ws(4, 8192, 16, 128, 128, 1) > a
    assert ws(4, 4096, 32, 128, 128, 1) > a
    # the forward's chunk factors are C x C per unit: independent of Dv
    assert ws(4, 4096, 16, 128, 256, 1) == a
    assert ws(4, 4096, 16, 128, 256, 1, is_bwd=True) > b
    assert ws(4, 4096, 16, 96, 128, 1) == 0      # Dk 96 unsupported
    assert ws(4, 4096, 16, 128, 128, 0) == 0     # fp32 needs Dk 64
    assert ws(1, 100, 2, 64, 64, 0) > 0
    assert ws(-1, 100, 2, 64, 64, 0) == 0


FAKE = 1 << 20          # aligned, never dereferenced: every call below fails validation


def _fwd(B=1, T=64, H=1, Dk=64, Dv=64, chunk=64, dtype=1, ptrs=None, ws=FAKE, ws_bytes=1 << 40):
    p = dict(q=FAKE, k=FAKE, v=FAKE, beta=FAKE, lam=FAKE, la=None, s0=None, o=FAKE, sf=None, sv=None)
    if ptrs:
        p.update(ptrs)
    return qdelta.lib().qdelta_chunk_fwd(B, T, H, Dk, Dv, chunk, dtype, p["q"], p["k"], p["v"],
                                         p["beta"], p["lam"], 0.0, p["la"], p["s0"], p["o"], p["sf"],
                                         p["sv"], ws, ws_bytes, None)


def test_fwd_rejects_bad_arguments_before_launch():
    E = qdelta
    assert _fwd(Dk=96) == E.QDELTA_EUNSUPPORTED
    assert _fwd(Dv=32) == E.QDELTA_EUNSUPPORTED
    assert _fwd(chunk=32) == E.QDELTA_EUNSUPPORTED
    assert _fwd(dtype=0, Dk=128) == E.QDELTA_EUNSUPPORTED
    assert _fwd(dtype=7) == E.QDELTA_EINVAL
    assert _fwd(H=0) == E.QDELTA_EINVAL
    assert _fwd(T=-1) == E.QDELTA_EINVAL
    assert _fwd(ptrs=dict(q=None)) == E.QDELTA_EINVAL
    assert _fwd(ptrs=dict(v=FAKE + 4)) == E.QDELTA_EINVAL          # misaligned
    assert _fwd(ptrs=dict(sf=FAKE + 8)) == E.QDELTA_EINVAL
    assert _fwd(ws_bytes=16) == E.QDELTA_ENOWORKSPACE
    assert _fwd(ws=None) == E.QDELTA_EINVAL
    # nothing to do: zero sequences
    assert _fwd(B=0, ws=None, ws_bytes=0) == E.QDELTA_OK


def test_noalloc_forward_validates_before_any_device_call():
    """The allocation-free forward rejects bad arguments, and sizes whose
    workspace exceeds its scratch array, before touching the device."""
    L = qdelta.lib()
    E = qdelta
    f = FAKE

    def call(B=1, T=64, H=1, Dk=64, Dv=64, dtype=1, q=f, o=f):
        return L.qdelta_chunk_fwd_noalloc(B, T, H, Dk, Dv, 64, dtype, q, f, f, f, f, 0.0, None, None, o, None,
                                          None)

    assert call(Dk=96) == E.QDELTA_EUNSUPPORTED
    assert call(dtype=0, Dk=128) == E.QDELTA_EUNSUPPORTED
    assert call(T=-1) == E.QDELTA_EINVAL
    assert call(q=None) == E.QDELTA_EINVAL
    assert call(o=f + 4) == E.QDELTA_EINVAL
    assert call(B=0) == E.QDELTA_OK
    # bf16 forward workspace: 11008 B per chunk-head unit (packed T and P, the
    # gate block) and a 1 KB zero block, against 64 MiB
    cap = qdelta.NOALLOC_SCRATCH_BYTES
    assert qdelta.workspace_bytes(4, 4096, 16, 128, 128, 1) <= cap
    assert qdelta.workspace_bytes(8, 4096, 16, 128, 128, 1) > cap
    assert call(B=8, T=4096, H=16, Dk=128, Dv=128) == E.QDELTA_ENOWORKSPACE
    assert call(B=1, T=65536, H=16, Dk=128, Dv=128) == E.QDELTA_ENOWORKSPACE


def test_segmented_forward_sizes_and_validation():
    """Workspace of the segment-parallel forward: the forward's own plus each
    segment's map (Dv + Dk rows of Dk, fp32) and entry state (Dv x Dk fp32);
    bad arguments are rejected before any launch; the suggested segment
    count is 1 where the single pass fills the chip."""
    L = qdelta.lib()
    E = qdelta
    f = FAKE
    base = qdelta.workspace_bytes(1, 65536, 16, 128, 128, 1)
    # 1024 chunks in 4 segments of 256
    extra = 16 * 4 * (256 * 128 * 4 + 128 * 128 * 4)
    assert qdelta.segmented_workspace_bytes(1, 65536, 16, 128, 128, 1, 4) == base + extra
    # 10 chunks asked for 4 segments: 3 chunks each, so 4 non-empty segments
    b10 = qdelta.workspace_bytes(2, 640, 2, 64, 64, 0)
    assert qdelta.segmented_workspace_bytes(2, 640, 2, 64, 64, 0, 4) == b10 + 4 * 4 * (128 * 64 * 4 + 64 * 64 * 4)
    assert qdelta.segmented_workspace_bytes(1, 640, 2, 64, 64, 0, 0) == 0

    def call(n_segments=4, ws_bytes=1 << 40, Dk=64, q=f):
        return L.qdelta_chunk_fwd_segmented(1, 640, 2, Dk, 64, 64, 1, q, f, f, f, f, 0.0, None, None, f, None,
                                            None, n_segments, f, ws_bytes, None)

    assert call(n_segments=0) == E.QDELTA_EINVAL
    assert call(Dk=96) == E.QDELTA_EUNSUPPORTED
    assert call(q=None) == E.QDELTA_EINVAL
    assert call(ws_bytes=qdelta.workspace_bytes(1, 640, 2, 64, 64, 1)) == E.QDELTA_ENOWORKSPACE
    assert qdelta.suggest_segments(4, 4096, 16, 128, 128) == 1
    assert qdelta.suggest_segments(1, 65536, 2, 128, 128) > 1


@pytest.mark.parametrize("dtype", [0, 1])
def test_suggested_segments_range(dtype):
    """The suggestion stays within 1 and 32 segments of at least 6 chunks, is
    the single pass for sequences of under 12 chunks or more (sequence,
    head) pairs than CUs, and holds at the largest sizes."""
    for T in (1, 64, 704, 769, 4000, 8191, 65536, 2**31 - 1):
        for H in (1, 2, 5, 16, 24, 33, 257):
            G = qdelta.suggest_segments(1, T, H, 64, 128, dtype)
            assert 1 <= G <= 32
            assert G == 1 or -(-T // 64) // G >= 6, (T, H, G)
    assert qdelta.suggest_segments(1, 704, 1, 64, 64, dtype) == 1
    assert qdelta.suggest_segments(2**31 - 1, 2**31 - 1, 2**31 - 1, 128, 128, 1) == 1


def test_recurrent_bwd_sizes_and_validation():
    L = qdelta.lib()
    E = qdelta
    f = FAKE
    # per token-head 3 Dv + Dk + 1 fp32, per (sequence, head) Dv fp32 (each region 256-byte aligned)
    r = lambda b: (b + 255) // 256 * 256
    tok, H, Dk, Dv = 64 * 16, 16, 128, 128
    assert qdelta.recurrent_workspace_bytes(64, 16, H, Dk, Dv) == \
        3 * r(tok * H * Dv * 4) + r(tok * H * Dk * 4) + r(64 * H * Dv * 4) + r(tok * H * 4)
    assert qdelta.recurrent_workspace_bytes(1, 8, 1, 64, 96) == 0

    def call(Dk=64, Dv=64, dtype=1, lam=f, dlam=f, la=None, dla=None, ws_bytes=1 << 40, dq=f):
        return L.qdelta_recurrent_bwd(1, 8, 1, Dk, Dv, dtype, f, f, f, f, lam, 0.5, la, None, f, None, dq, f, f, f,
                                      dlam, dla, None, f, ws_bytes, None)

    assert call(Dv=96) == E.QDELTA_EUNSUPPORTED
    assert call(dtype=5) == E.QDELTA_EINVAL
    assert call(dq=None) == E.QDELTA_EINVAL
    assert call(la=f) == E.QDELTA_EINVAL                  # log alpha without its gradient
    assert call(dlam=None) == E.QDELTA_EINVAL             # per-token lambda without its gradient
    assert call(lam=None, dlam=f + 2) == E.QDELTA_EINVAL  # constant lambda's gradient: one aligned float
    assert call(ws_bytes=16) == E.QDELTA_ENOWORKSPACE
    assert L.qdelta_recurrent_bwd_varlen(8, 1, None, 1, 64, 64, 1, f, f, f, f, f, 0.0, None, None, f, None, f, f, f,
                                         f, f, None, None, f, 1 << 40, None) == E.QDELTA_EINVAL


def test_bwd_and_varlen_reject_bad_arguments():
    L = qdelta.lib()
    E = qdelta
    f = FAKE
    # log_alpha given but dlog_alpha missing
    rc = L.qdelta_chunk_bwd(1, 64, 1, 64, 64, 64, 1, f, f, f, f, f, 0.0, f, None, None, f, None, f, f, f, f,
                            f, None, None, f, 1 << 40, None)
    assert rc == E.QDELTA_EINVAL
    # too small workspace
    rc = L.qdelta_chunk_bwd(1, 64, 1, 64, 64, 64, 1, f, f, f, f, f, 0.0, None, None, None, f, None, f, f, f, f,
                            f, None, None, f, 1024, None)
    assert rc == E.QDELTA_ENOWORKSPACE
    # varlen needs cu_seqlens
    rc = L.qdelta_chunk_fwd_varlen(64, 1, None, 1, 64, 64, 64, 1, f, f, f, f, f, 0.0, None, None, f, None,
                                   None, f, 1 << 40, None)
    assert rc == E.QDELTA_EINVAL
    rc = L.qdelta_chunk_bwd_varlen(64, -1, f, 1, 64, 64, 64, 1, f, f, f, f, f, 0.0, None, None, None, f, None,
                                   f, f, f, f, f, None, None, f, 1 << 40, None)
    assert rc == E.QDELTA_EINVAL


def test_bwd_lambda_gradient_rules():
    """A per-token lambda needs its per-token gradient; a constant lambda
    (lam NULL) takes either no gradient or one float (4-byte aligned)."""
    L = qdelta.lib()
    E = qdelta
    f = FAKE

    def bwd(lam, dlam, ws_bytes=1):
        # the workspace check comes after the argument checks: 1 byte means
        # "arguments valid" shows as QDELTA_ENOWORKSPACE, with no launch
        return L.qdelta_chunk_bwd(1, 64, 1, 64, 64, 64, 1, f, f, f, f, lam, 0.5, None, None, None, f, None,
                                  f, f, f, f, dlam, None, None, f, ws_bytes, None)

    assert bwd(f, None) == E.QDELTA_EINVAL            # per-token lambda without its gradient
    assert bwd(f, f + 4) == E.QDELTA_EINVAL           # misaligned per-token gradient
    assert bwd(None, f + 4) == E.QDELTA_ENOWORKSPACE  # one float: 4-byte alignment suffices
    assert bwd(None, f + 2) == E.QDELTA_EINVAL
    assert bwd(None, None) == E.QDELTA_ENOWORKSPACE
    assert bwd(f, f) == E.QDELTA_ENOWORKSPACE


def test_recurrent_step_rejects_bad_arguments():
    L = qdelta.lib()
    E = qdelta
    f = FAKE
    assert L.qdelta_recurrent_step(1, 1, 96, 64, 1, f, f, f, f, f, 0.0, None, f, f, None) == E.QDELTA_EUNSUPPORTED
    assert L.qdelta_recurrent_step(1, 1, 64, 12, 1, f, f, f, f, f, 0.0, None, f, f, None) == E.QDELTA_EUNSUPPORTED
    assert L.qdelta_recurrent_step(1, 1, 64, 64, 1, f, f, f, f, f, 0.0, None, f + 4, f, None) == E.QDELTA_EINVAL
    assert L.qdelta_recurrent_step(1, 0, 64, 64, 1, f, f, f, f, f, 0.0, None, f, f, None) == E.QDELTA_EINVAL
    assert L.qdelta_recurrent_step(0, 1, 64, 64, 1, None, None, None, None, None, 0.0, None, None, None,
                                   None) == E.QDELTA_OK


def test_recurrent_fwd_rejects_bad_arguments():
    """Validation of the recurrent forward happens before any launch; calls
    with nothing to do return OK without touching the device."""
    L = qdelta.lib()
    E = qdelta
    f = FAKE
    args = (f, f, f, f, None, 0.0, None, None, f, None, None)
    assert L.qdelta_recurrent_fwd(1, 8, 1, 96, 64, 1, *args) == E.QDELTA_EUNSUPPORTED
    assert L.qdelta_recurrent_fwd(1, 8, 1, 64, 300, 1, *args) == E.QDELTA_EUNSUPPORTED
    assert L.qdelta_recurrent_fwd(1, 8, 1, 64, 64, 7, *args) == E.QDELTA_EINVAL
    assert L.qdelta_recurrent_fwd(1, -1, 1, 64, 64, 1, *args) == E.QDELTA_EINVAL
    assert L.qdelta_recurrent_fwd(1, 8, 1, 64, 64, 1, f + 4, f, f, f, None, 0.0, None, None, f, None,
                                  None) == E.QDELTA_EINVAL
    assert L.qdelta_recurrent_fwd(1, 8, 1, 64, 64, 1, None, f, f, f, None, 0.0, None, None, f, None,
                                  None) == E.QDELTA_EINVAL
    assert L.qdelta_recurrent_fwd(1, 8, 1, 64, 64, 1, f, f, f, f, f + 8, 0.0, None, None, f, None,
                                  None) == E.QDELTA_EINVAL
    # no sequences: nothing to do
    none10 = [None] * 5 + [0.0] + [None] * 5
    assert L.qdelta_recurrent_fwd(0, 8, 1, 64, 64, 1, *none10) == E.QDELTA_OK
    assert L.qdelta_recurrent_fwd_varlen(0, 0, f, 1, 64, 64, 1, *none10) == E.QDELTA_OK
    assert L.qdelta_recurrent_fwd_varlen(8, 1, None, 1, 64, 64, 1, *args) == E.QDELTA_EINVAL


def test_layer_entries_reject_bad_arguments():
    """The entry points of the layer's own path validate before any launch; everything valid shows as
    QDELTA_ENOWORKSPACE with one byte of workspace."""
    L = qdelta.lib()
    E = qdelta
    f = FAKE

    def fwd(B=2, T=8, N=2, cu=None, H=1, Dk=64, Dv=64, dtype=1, qkv=f, beta=f, lam=f, la=None, S0=None, q=f, k=f, rq=f,
            rk=f, o=f, Sf=None, saved=None, ws=f, ws_bytes=1):
        return L.qdelta_layer_fwd(B, T, N, cu, H, Dk, Dv, dtype, qkv, beta, lam, 0.5, la, S0, q, k, rq, rk, o, Sf,
                                  saved, ws, ws_bytes, None)

    def bwd(B=2, T=8, N=2, cu=None, H=1, Dk=64, Dv=64, dtype=1, qkv=f, q=f, k=f, rq=f, rk=f, beta=f, lam=f, la=None,
            S0=None, saved=f, dO=f, dSf=None, dqkv=f, dbeta=f, dlam=f, dla=None, dS0=None, ws=f, ws_bytes=1):
        return L.qdelta_layer_bwd(B, T, N, cu, H, Dk, Dv, dtype, qkv, q, k, rq, rk, beta, lam, 0.5, la, S0, saved, dO,
                                  dSf, dqkv, dbeta, dlam, dla, dS0, ws, ws_bytes, None)

    for call in (fwd, bwd):
        assert call() == call(B=0, T=8, N=1, cu=f) == call(lam=None, **({"dlam": None} if call is bwd else {})) \
            == E.QDELTA_ENOWORKSPACE
        for name in ("qkv", "q", "k", "rq", "rk", "beta"):
            assert call(**{name: None}) == E.QDELTA_EINVAL, (call.__name__, name)
            assert call(**{name: f + 4}) == E.QDELTA_EINVAL, (call.__name__, name)
        for name in ("lam", "la", "S0"):
            assert call(**{name: f + 8}) == E.QDELTA_EINVAL, (call.__name__, name)
        assert call(H=0) == call(T=-1) == call(B=-1) == call(dtype=3) == call(ws=None) == E.QDELTA_EINVAL
        assert call(N=-1, cu=f) == E.QDELTA_EINVAL
        assert call(Dk=96) == call(Dv=32) == call(Dk=128, dtype=0) == E.QDELTA_EUNSUPPORTED
    assert fwd(o=None) == fwd(Sf=f + 4) == fwd(saved=f + 4) == E.QDELTA_EINVAL
    for name in ("saved", "dO", "dqkv", "dbeta", "dlam"):
        assert bwd(**{name: None}) == bwd(**{name: f + 4}) == E.QDELTA_EINVAL, name
    assert bwd(la=f) == bwd(dla=f) == E.QDELTA_EINVAL        # log alpha without its gradient, and the other way round
    assert bwd(dSf=f + 4) == bwd(dS0=f + 4) == E.QDELTA_EINVAL


def test_layer_gate_entries_reject_bad_arguments():
    L = qdelta.lib()
    E = qdelta
    f = FAKE

    def fwd(tokens=8, H=2, dtype=1, bias_dtype=1, x=f, bias=f, beta=f, lam=f, la=f):
        return L.qdelta_layer_gates_fwd(tokens, H, dtype, bias_dtype, x, bias, beta, lam, la, None)

    def bwd(tokens=8, H=2, dtype=1, bias_dtype=1, beta=f, lam=f, la=f, dx=f, parts=f, dbias=f):
        return L.qdelta_layer_gates_bwd(tokens, H, dtype, bias_dtype, beta, lam, la, f, f, f, dx, parts, dbias, None)

    for call in (fwd, bwd):
        assert call(tokens=0) == call(tokens=-1) == call(H=0) == call(tokens=1 << 30, H=2) == E.QDELTA_EINVAL
        assert call(dtype=2) == call(bias_dtype=-1) == call(beta=None) == E.QDELTA_EINVAL
    assert fwd(x=None) == fwd(bias=None) == E.QDELTA_EINVAL
    assert bwd(dx=None) == bwd(parts=None) == bwd(dbias=None) == E.QDELTA_EINVAL
    assert L.qdelta_layer_gate_parts(0, 2) == L.qdelta_layer_gate_parts(8, 0) == 0
    assert L.qdelta_layer_gate_parts(300, 2) == 3             # one float per 256 (token, head) pairs, at most 1024


def test_l2norm_rejects_bad_arguments():
    L = qdelta.lib()
    E = qdelta
    f = FAKE
    assert L.qdelta_l2norm_fwd(4, 96, 96, 1, f, f, f, None) == E.QDELTA_EUNSUPPORTED
    assert L.qdelta_l2norm_fwd(4, 128, 100, 1, f, f, f, None) == E.QDELTA_EINVAL    # ld below D
    assert L.qdelta_l2norm_fwd(4, 128, 132, 1, f, f, f, None) == E.QDELTA_EINVAL    # 264-byte rows
    assert L.qdelta_l2norm_fwd(4, 128, 128, 1, f + 2, f, f, None) == E.QDELTA_EINVAL
    assert L.qdelta_l2norm_fwd(-1, 128, 128, 1, f, f, f, None) == E.QDELTA_EINVAL
    assert L.qdelta_l2norm_fwd(0, 128, 128, 1, None, None, None, None) == E.QDELTA_OK
    assert L.qdelta_l2norm_bwd(4, 128, 1, f, f, None, f, None) == E.QDELTA_EINVAL
    assert L.qdelta_l2norm_bwd(0, 128, 1, None, None, None, None, None) == E.QDELTA_OK


def test_binding_validates_before_calling_library():
    import torch
    q = torch.zeros(1, 64, 1, 64)
    with pytest.raises(ValueError):
        qdelta.chunk_fwd(q, q, q, torch.zeros(1, 64, 1), torch.zeros(1, 64, 1))   # CPU tensors
