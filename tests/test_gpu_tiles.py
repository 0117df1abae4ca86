"""GPU parity where the launch rules change the tile width: unit counts on both sides of each line, ragged lengths,
forward and backward against the fp64 oracle (sampled heads; normwise tolerances as everywhere)."""
import numpy as np
import pytest
import torch

from paper_2606_08804_amd import qdelta, synth
from tests.gpu_helpers import TOL, bwd_errors, dev, fwd_errors, gpu_bwd, gpu_fwd, select_heads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Dv", [(16, 256), (17, 256), (32, 128), (33, 128), (64, 64), (65, 64)])
def test_fp32_scan_tile_widths(H, Dv):
    """fp32 scans: 16-row tiles while all of them fit one to a CU (H * Dv / 16 <= 256 at B = 1), 32-row tiles beyond."""
    d = synth.make(1, 150, H, 64, Dv, "f32", "G3", seed=701 + H, s0=True, with_do=True)
    o, Sf, saved = gpu_fwd(d, save_states=True)
    g = gpu_bwd(d, saved)
    heads = [0, H // 2, H - 1]
    ds = select_heads(d, heads)
    o, Sf = o[:, :, heads], Sf[:, heads]
    g = {k: v[:, heads] if k == "d_initial_state" else v[:, :, heads] for k, v in g.items()}
    errs = {**fwd_errors(ds, o, Sf), **bwd_errors(ds, g)}
    assert all(v <= TOL["f32"] for v in errs.values()), errs


def _rec(d):
    return qdelta.recurrent_fwd(dev(d["q"]), dev(d["k"]), dev(d["v"]), dev(d["beta"]), dev(d["lam"]),
                                dev(d["log_alpha"]), dev(d["initial_state"]), cu_seqlens=dev(d["cu_seqlens"]))


# fp32 state arithmetic: bf16 inputs add only the rounding of o (2^-9 of a value)
REC_TOL = {"f32": 5e-6, "bf16": 4e-3}


@pytest.mark.parametrize("dt,Dk,Dv", [("bf16", 128, 72), ("bf16", 64, 8), ("f32", 128, 40), ("f32", 64, 256)])
@pytest.mark.parametrize("T", [1, 2, 4, 5, 6, 7, 15, 16, 17, 49])
def test_recurrent_fwd_lengths(T, dt, Dk, Dv):
    """Both sides of the step / block rule, block edges, and value rows that no tile divides."""
    d = synth.make(2, T, 3, Dk, Dv, dt, "G3", seed=720 + T, s0=True)
    errs = fwd_errors(d, *_rec(d))
    assert all(v <= REC_TOL[dt] for v in errs.values()), errs


@pytest.mark.parametrize("dt,Dk,B,H,T", [("bf16", 128, 64, 16, 18), ("bf16", 128, 33, 16, 33), ("bf16", 64, 64, 16, 18),
                                         ("f32", 128, 16, 16, 18), ("f32", 64, 15, 17, 18)])
def test_recurrent_fwd_wide_tiles(dt, Dk, B, H, T):
    """Unit counts at and beside the wide-tile rule."""
    d = synth.make(B, T, H, Dk, 128, dt, "G3", seed=741, s0=True)
    o, Sf = _rec(d)
    heads = [0, H - 1]
    errs = fwd_errors(select_heads(d, heads), o[:, :, heads], Sf[:, heads])
    assert all(v <= REC_TOL[dt] for v in errs.values()), errs


@pytest.mark.parametrize("lengths", [[1, 1, 1], [2, 0, 3, 1], [0, 40, 0, 16, 17, 1]])
def test_recurrent_fwd_packed_routes(lengths):
    """Packed batches on both sides of the mean-length rule, empty sequences among them."""
    d = synth.make(1, 0, 2, 128, 64, "f32", "G2", seed=751, lengths=lengths, s0=True)
    errs = fwd_errors(d, *_rec(d))
    assert all(v <= REC_TOL["f32"] for v in errs.values()), errs


@pytest.mark.parametrize("dt,Dk,Dv", [("bf16", 64, 64), ("bf16", 128, 24), ("f32", 64, 72)])
def test_recurrent_fwd_packed_skewed(dt, Dk, Dv):
    """One long sequence among single tokens, still within the mean of the step route: every token's operands are
    loaded while the one before is computed, the last one's with none after it."""
    d = synth.make(1, 0, 3, Dk, Dv, dt, "G3", seed=757, lengths=[1] * 9 + [17, 0, 2] + [1] * 9, s0=True)
    errs = fwd_errors(d, *_rec(d))
    assert all(v <= REC_TOL[dt] for v in errs.values()), errs


@pytest.mark.parametrize("T", [4, 12, 40])
def test_recurrent_fwd_is_causal_and_takes_alpha_zero(T):
    """alpha = 0 (log alpha = -inf) forgets the state exactly; a NaN in one token leaves every earlier output as it was."""
    d = synth.make(1, T, 2, 64, 64, "f32", "G2", seed=761, s0=True)
    d["log_alpha"][0, T // 2] = -np.inf
    o, Sf = _rec(d)
    errs = fwd_errors(d, o, Sf)
    assert all(v <= REC_TOL["f32"] for v in errs.values()), errs
    d2 = {k: v.clone() if isinstance(v, torch.Tensor) else v for k, v in d.items()}
    at = T // 2 + 1
    for key in ("q", "k", "v", "beta"):
        d2[key][0, at] = float("nan")
    o2, _ = _rec(d2)
    assert torch.equal(o2[:, :at], o[:, :at]) and not torch.isfinite(o2[:, at]).any()


def _rec_bwd(d, dsf, need=True):
    return qdelta.recurrent_bwd(dev(d["q"]), dev(d["k"]), dev(d["v"]), dev(d["beta"]), dev(d["lam"]),
                                dev(d["log_alpha"]), dev(d["initial_state"]), dev(d["d_o"]), d_final_state=dev(dsf),
                                cu_seqlens=dev(d["cu_seqlens"]), need_d_initial_state=need)


def _dsf(d, N):
    H, Dv, Dk = d["v"].shape[2], d["v"].shape[3], d["q"].shape[3]
    return torch.from_numpy(np.random.default_rng(5).standard_normal((N, H, Dv, Dk)).astype(np.float32))


@pytest.mark.parametrize("dt,Dk,Dv", [("bf16", 128, 128), ("f32", 128, 256), ("f32", 64, 32), ("bf16", 64, 64)])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 15, 16, 17, 32, 33, 49, 97])
def test_recurrent_bwd_lengths(T, dt, Dk, Dv):
    """One block and several, on and beside the block edges and the spacing of the stored states (2, 3, 1 and 1 blocks
    at these sizes), with a final-state gradient; alpha = 0 in one token.  fp32 sums: 1e-5 of the largest value."""
    d = synth.make(2, T, 3, Dk, Dv, dt, "G3", seed=770 + T, s0=True, with_do=True)
    d["log_alpha"][1, T // 2] = -np.inf
    dsf = _dsf(d, 2)
    errs = bwd_errors(d, _rec_bwd(d, dsf), dsf)
    tol = 1e-5 if dt == "f32" else REC_TOL[dt]
    assert all(v <= tol for v in errs.values()), errs


@pytest.mark.parametrize("Dk,Dv", [(64, 64), (128, 128), (128, 256)])
@pytest.mark.parametrize("lengths", [[16, 0, 17, 1, 33, 50, 15], [40, 31, 32, 33, 1, 64],
                                     [5, 81, 97, 50, 0, 113, 65, 49], [47, 49, 98, 33, 96, 1, 130]])
def test_recurrent_bwd_packed_stored_states(lengths, Dk, Dv):
    """The stored states of packed sequences that start anywhere within a block, or within a group of the 1, 2 or 3
    blocks between stored states, do not overlap, and the blocks between are walked again from the right one."""
    d = synth.make(1, 0, 2, Dk, Dv, "f32", "G2", seed=781, lengths=lengths, s0=True, with_do=True)
    dsf = _dsf(d, len(lengths))
    errs = bwd_errors(d, _rec_bwd(d, dsf), dsf)
    assert all(v <= 1e-5 for v in errs.values()), errs


@pytest.mark.parametrize("dt,Dk,Dv", [("bf16", 128, 128), ("f32", 64, 256), ("bf16", 64, 256), ("f32", 128, 32)])
@pytest.mark.parametrize("lengths", [[1, 2, 0, 3] * 6, [1] * 23 + [17], [2, 0] * 12])
def test_recurrent_bwd_packed_few(lengths, dt, Dk, Dv):
    """Packed batches of more (sequence, head) pairs than CUs whose mean is within the few-token limit (2, 4 at d_k 64,
    d_v 256): each sequence is one of two launches', by its length."""
    H = 12
    assert len(lengths) * H > 256 and sum(lengths) <= 2 * len(lengths)
    d = synth.make(1, 0, H, Dk, Dv, dt, "G3", seed=787, lengths=lengths, s0=True, with_do=True)
    d["log_alpha"][0, 1] = -np.inf
    dsf = _dsf(d, len(lengths))
    g = _rec_bwd(d, dsf)
    heads = [0, H - 1]
    g = {k: None if v is None else v[:, heads] if k == "d_initial_state" else v[:, :, heads] for k, v in g.items()}
    errs = bwd_errors(select_heads(d, heads), g, dsf[:, heads])
    tol = 1e-5 if dt == "f32" else REC_TOL[dt]
    assert all(v <= tol for v in errs.values()), errs


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("B,H,T", [(22, 12, 3), (22, 12, 4), (16, 16, 4)])
def test_recurrent_bwd_few_tokens_wide_values(B, H, T, dt):
    """Three and four tokens at d_k 64, d_v 256, with more units than CUs and with as many."""
    d = synth.make(B, T, H, 64, 256, dt, "G3", seed=789, s0=True, with_do=True)
    dsf = _dsf(d, B)
    g = _rec_bwd(d, dsf)
    heads = [0, H - 1]
    g = {k: None if v is None else v[:, heads] if k == "d_initial_state" else v[:, :, heads] for k, v in g.items()}
    errs = bwd_errors(select_heads(d, heads), g, dsf[:, heads])
    tol = 1e-5 if dt == "f32" else REC_TOL[dt]
    assert all(v <= tol for v in errs.values()), errs


@pytest.mark.parametrize("T", [2, 5, 40])
def test_recurrent_bwd_without_state_gradients(T):
    """No initial state, no final-state gradient, no initial-state gradient wanted: the same token gradients."""
    d = synth.make(2, T, 2, 128, 64, "f32", "G1", seed=791, with_do=True)
    full = _rec_bwd(d, None)
    part = _rec_bwd(d, None, need=False)
    assert part["d_initial_state"] is None
    for key in ("dq", "dk", "dv", "dbeta", "dlam"):
        assert torch.equal(full[key], part[key]), key
    errs = bwd_errors(d, part, skip=("d_initial_state",))
    assert all(v <= 1e-5 for v in errs.values()), errs


@pytest.mark.parametrize("dt,T", [("f32", 4), ("f32", 12), ("bf16", 16), ("f32", 40)])
@pytest.mark.parametrize("key,bad,later,same", [
    ("v", float("inf"), False, ("dq", "dk", "dbeta", "dlam")), ("v", float("nan"), False, ("dq", "dk", "dbeta", "dlam")),
    ("d_o", float("-inf"), True, ("dq", "dk", "dv", "dbeta", "dlam", "dlog_alpha")),
    ("k", float("nan"), True, ("dv",)), ("q", float("nan"), True, ("dv",))])
def test_recurrent_bwd_keeps_tokens_apart(dt, T, key, bad, later, same):
    """A value that is not finite, in one token, leaves the gradients it does not enter as they were: those of the
    earlier tokens where it is in v (dv does not depend on v at all), of the later ones where it is in d_o, and the
    later dv where it is in k or q.  Up to the order of the sums in the block that holds it (fp32; bf16 gradients to
    one rounding, 2^-8)."""
    d = synth.make(2, T, 2, 64, 64, dt, "G3", seed=797, s0=True, with_do=True)
    at = T // 2
    ref = _rec_bwd(d, _dsf(d, 2))
    d2 = dict(d, **{key: d[key].clone()})
    d2[key][0, at, 1, 5] = bad
    got = _rec_bwd(d2, _dsf(d, 2))
    rows = slice(at + 1, None) if later else slice(None, at)
    tol = 1e-5 if dt == "f32" else 2.0 ** -8
    for name in same:
        a, b = got[name][0, rows, 1], ref[name][0, rows, 1]
        assert torch.isfinite(a).all(), name
        assert float((a.float() - b.float()).abs().max()) <= tol * float(b.float().abs().max()), name
    if key == "v":
        assert torch.equal(got["dv"], ref["dv"])
    assert not torch.isfinite(got["dk"][0, at, 1]).all()
    for name in ("dq", "dk", "dv", "dbeta", "dlam"):        # the other heads and sequences
        assert torch.equal(got[name][1], ref[name][1]) and torch.equal(got[name][0, :, 0], ref[name][0, :, 0]), name
