"""GPU parity where the launch rules change the tile width: unit counts on both sides of each line, ragged lengths,
forward and backward against the fp64 oracle (sampled heads; normwise tolerances as everywhere)."""
import pytest
import torch

from paper_2606_08804_amd import synth
from tests.gpu_helpers import TOL, bwd_errors, fwd_errors, gpu_bwd, gpu_fwd, select_heads

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
