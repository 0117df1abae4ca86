"""bf16 results bit for bit: digests of outputs and gradients on exact dyadic inputs (the same on every machine).

Without decay a bf16 state keeps every rounding of the chunk factors, so sums taken in another order show in later
outputs though no result is further from the exact one.  These digests hold the order.  A change that rounds
differently on purpose records new ones, together with its error against 64 bits beside the former one's."""
import hashlib

import pytest
import torch

from paper_2606_08804_amd import qdelta

pytestmark = pytest.mark.gpu

# (B, T, H, Dk, Dv, decay, constant lambda, lengths) -> sha256 of o, final state and gradients, first 16 digits
CASES = {
    (2, 515, 3, 128, 128, True, None, None): "bbee336d0970b770",
    (2, 515, 3, 64, 64, False, None, None): "63e3e89bafa8c898",
    (1, 900, 2, 64, 128, False, 0.5, (333, 1, 470, 96)): "cbb139c52f88bc11",
    (1, 700, 2, 128, 256, False, None, (64, 500, 136)): "225600b55fd1b4f7",
}


def digest(B, T, H, Dk, Dv, decay, lam_c, lengths):
    g = torch.Generator().manual_seed(T + Dk + Dv)

    def dyadic(lo, hi, scale, *shape):
        return (torch.randint(lo, hi + 1, shape, generator=g) / scale).cuda()

    q, k = (dyadic(-8, 8, 64, B, T, H, Dk).bfloat16() for _ in range(2))
    v, d_o = (dyadic(-16, 16, 8, B, T, H, Dv).bfloat16() for _ in range(2))
    beta, lam = (dyadic(1, 15, 16, B, T, H) for _ in range(2))
    la = dyadic(-64, 0, 64, B, T, H) if decay else None
    S0 = dyadic(-8, 8, 64, len(lengths) if lengths else B, H, Dv, Dk)
    cu = torch.tensor([0, *lengths], dtype=torch.int32).cumsum(0).to(torch.int32).cuda() if lengths else None
    args = (q, k, v, beta, lam if lam_c is None else lam_c, la, S0)
    o, Sf, saved = qdelta.chunk_fwd(*args, cu_seqlens=cu, save_states=True)
    grads = qdelta.chunk_bwd(*args, saved, d_o, cu_seqlens=cu)
    h = hashlib.sha256()
    for t in (o, Sf, *(grads[key] for key in sorted(grads) if grads[key] is not None)):
        h.update(t.cpu().contiguous().reshape(-1).view(torch.uint8).numpy().tobytes())
    return h.hexdigest()[:16]


@pytest.mark.parametrize("case", list(CASES))
def test_bf16_bits(case):
    assert digest(*case) == CASES[case]
