"""The fully recurrent backward (qdelta_recurrent_bwd[_varlen]) against the
fp64 oracle's BPTT gradient: fp32 within 1e-4 and bf16 within 2e-2 (normwise
per gradient), at T = 1, 16 and 150, every gate mode, every supported head
size, packed sequences, a non-zero final-state gradient and a constant
lambda; plus run-to-run determinism and agreement with the chunk backward."""
import numpy as np
import pytest
import torch

from paper_2606_08804_amd import qdelta, synth
from tests.gpu_helpers import TOL, bwd_errors, dev, f64, gpu_bwd, gpu_fwd, normwise, oracle_bwd

pytestmark = pytest.mark.gpu


def rec_bwd(d, d_final_state=None, lam="tensor"):
    lam_arg = dev(d["lam"]) if lam == "tensor" else lam
    g = qdelta.recurrent_bwd(dev(d["q"]), dev(d["k"]), dev(d["v"]), dev(d["beta"]), lam_arg, dev(d["log_alpha"]),
                             dev(d["initial_state"]), dev(d["d_o"]), d_final_state=dev(d_final_state),
                             cu_seqlens=dev(d["cu_seqlens"]))
    torch.cuda.synchronize()
    return g


def _dsf(d, seed):
    N = d["initial_state"].shape[0]
    H, Dv, Dk = d["v"].shape[2], d["v"].shape[3], d["q"].shape[3]
    return torch.from_numpy(np.random.default_rng(seed).standard_normal((N, H, Dv, Dk)).astype(np.float32))


def _check(e, tol, what):
    bad = {k: v for k, v in e.items() if not (v <= tol)}
    assert not bad, f"{what}: {e}"


@pytest.mark.parametrize("gate", ["G1", "G2", "G3"])
@pytest.mark.parametrize("T", [1, 16, 150])
def test_recurrent_bwd_fp32(gate, T):
    d = synth.make(2, T, 2, 64, 64, "f32", gate, seed=180 + T, s0=True, with_do=True)
    dSf = _dsf(d, 181)
    g = rec_bwd(d, dSf)
    _check(bwd_errors(d, g, dSf), TOL["f32"], f"rec bwd fp32 {gate} T={T}")


@pytest.mark.parametrize("gate", ["G1", "G2", "G3"])
@pytest.mark.parametrize("T", [1, 16, 150])
def test_recurrent_bwd_bf16(gate, T):
    d = synth.make(2, T, 2, 128, 128, "bf16", gate, seed=182 + T, s0=True, with_do=True)
    g = rec_bwd(d)
    _check(bwd_errors(d, g), TOL["bf16"], f"rec bwd bf16 {gate} T={T}")


@pytest.mark.parametrize("dt,Dk,Dv", [("bf16", 64, 32), ("bf16", 64, 256), ("bf16", 128, 64), ("bf16", 128, 256),
                                      ("f32", 128, 128), ("f32", 64, 256), ("f32", 128, 256)])
def test_recurrent_bwd_head_sizes(dt, Dk, Dv):
    d = synth.make(1, 40, 2, Dk, Dv, dt, "G3", seed=184, s0=True, with_do=True)
    dSf = _dsf(d, 185)
    g = rec_bwd(d, dSf)
    _check(bwd_errors(d, g, dSf), TOL[dt], f"rec bwd {dt} Dk={Dk} Dv={Dv}")


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_recurrent_bwd_varlen(dt):
    D = 64 if dt == "f32" else 128
    d = synth.make(1, 0, 2, D, D, dt, "G2", seed=186, s0=True, with_do=True, lengths=[5, 17, 0, 1, 40])
    g = rec_bwd(d)
    _check(bwd_errors(d, g), TOL[dt], f"rec bwd varlen {dt}")


@pytest.mark.parametrize("c", [0.2, 1.0])
def test_recurrent_bwd_constant_lambda(c):
    d = synth.make(2, 30, 2, 128, 128, "bf16", "G2", seed=187, s0=True, with_do=True)
    dc = dict(d, lam=torch.full_like(d["beta"], c))
    g = rec_bwd(d, lam=c)
    assert g["dlam"].shape == ()
    _check(bwd_errors(dc, g, skip=("dlam",)), TOL["bf16"], f"rec bwd lambda={c}")
    ref = oracle_bwd(dc)["dlam"]
    assert abs(float(g["dlam"].cpu()) - ref.sum()) <= TOL["bf16"] * np.abs(ref).sum()


def test_recurrent_bwd_deterministic_and_matches_chunk_backward():
    d = synth.make(4, 64, 4, 128, 128, "bf16", "G2", seed=188, s0=True, with_do=True)
    g1 = rec_bwd(d)
    g2 = rec_bwd(d)
    for key in g1:
        if g1[key] is not None:
            assert torch.equal(g1[key], g2[key]), key
    _, _, saved = gpu_fwd(d, save_states=True)
    gc = gpu_bwd(d, saved)
    for key in g1:
        if g1[key] is not None:
            assert normwise(f64(g1[key].cpu()), f64(gc[key].cpu())) <= TOL["bf16"], key


def test_recurrent_bwd_training_shape_sampled_heads():
    """64 continuing sequences of 16 tokens, H=16, d=128 (the shape the
    recurrent form serves): sampled heads against the oracle."""
    from tests.gpu_helpers import select_heads
    d = synth.make(64, 16, 16, 128, 128, "bf16", "G2", seed=189, s0=True, with_do=True)
    g = rec_bwd(d)
    heads = [0, 11]
    ds = select_heads(d, heads)
    gs = {k: (None if v is None else (v[:, heads] if k == "d_initial_state" else v[:, :, heads]).contiguous())
          for k, v in g.items()}
    _check(bwd_errors(ds, gs), TOL["bf16"], "rec bwd B64 T16 H16")


@pytest.mark.parametrize("dt,D,gate,T", [("f32", 64, "G3", 2048), ("f32", 64, "G1", 2048), ("bf16", 128, "G2", 4096)])
def test_recurrent_bwd_long_sequences(dt, D, gate, T):
    """The reverse walk starts every block from a stored or recomputed state
    and carries the state's gradient through all of them: long sequences (slow
    decay, no decay) stay within the tolerance, dlog alpha included."""
    d = synth.make(1, T, 2, D, D, dt, gate, seed=190, s0=True, with_do=True)
    g = rec_bwd(d)
    _check(bwd_errors(d, g), TOL[dt], f"rec bwd {dt} {gate} T={T}")


def test_recurrent_bwd_empty_sequences():
    """T = 0: no token gradients; the initial-state gradient is the
    final-state gradient passed straight through."""
    d = synth.make(2, 0, 2, 128, 128, "bf16", "G2", seed=191, s0=True, with_do=True)
    dSf = _dsf(d, 192)
    g = rec_bwd(d, dSf)
    assert g["dq"].numel() == 0
    assert torch.equal(g["d_initial_state"].cpu(), dSf)
