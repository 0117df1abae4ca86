"""The formulas of the fully recurrent kernels over blocks of 16 tokens, as the
headers of csrc/qd_step.hip (k_rec_fwd) and csrc/qd_rec_bwd.hip state them,
written out in fp64 and checked against the oracle's token recurrence (Sec. 3.3,
Eq. qdelta_decay) and its backpropagation through time.

A slip in any of them (a decay product that is one token off, the wrong
triangle, a row minus a column of the decay sums the other way round, a block
that starts from the wrong stored state) changes a result by far more than the
tolerance."""
import numpy as np
import pytest

from oracle import recurrent

TB = 16


def unit(a):
    return a / np.linalg.norm(a, axis=-1, keepdims=True)


def inputs(T, dk, dv, seed, zeros=()):
    rng = np.random.default_rng(seed)

    def gate(mean=0.0):
        return 1 / (1 + np.exp(-rng.normal(mean, 1.0, T)))

    d = dict(q=unit(rng.standard_normal((T, dk))), k=unit(rng.standard_normal((T, dk))),
             v=rng.standard_normal((T, dv)), beta=gate(), lam=gate(), alpha=gate(1.0),
             S0=0.3 * rng.standard_normal((dv, dk)))
    d["alpha"][[t for t in zeros if t < T]] = 0.0
    return d, rng


def decays(al):
    """g_t = alpha_1..alpha_t, Gam_ti = alpha_{i+1}..alpha_t (i <= t), kb_i = Gam_Ci: products only, so alpha = 0 is exact."""
    n = len(al)
    gam = np.zeros((n, n))
    for i in range(n):
        gam[i:, i] = np.cumprod(np.concatenate([[1.0], al[i + 1:]]))
    return np.cumprod(al), gam, gam[-1].copy()


def block_fwd(S, q, k, v, be, lm, al):
    """One block from entry state S: outputs and exit state (qd_step.hip)."""
    g, gam, kb = decays(al)
    x = k + lm[:, None] * q
    e = np.zeros_like(v)
    o = np.zeros_like(v)
    for t in range(len(q)):
        e[t] = be[t] * (v[t] - g[t] * (S @ x[t])) - sum(be[t] * gam[t, i] * (k[i] @ x[t]) * e[i] for i in range(t))
        o[t] = g[t] * (S @ q[t]) + sum(gam[t, i] * (k[i] @ q[t]) * e[i] for i in range(t + 1))
    return o, g[-1] * S + (kb[:, None] * e).T @ k


def block_bwd(S, G, q, k, v, be, lm, al, dO):
    """One block from entry state S and exit-state gradient G: token gradients and the entry state's (qd_rec_bwd.hip)."""
    g, gam, kb = decays(al)
    x = k + lm[:, None] * q
    xk, qk = x @ k.T, q @ k.T
    A = np.tril(be[:, None] * gam * xk, -1)
    M = np.linalg.inv(np.eye(len(q)) + A)
    P = np.tril(gam * qk)
    sx, sq, gk = x @ S.T, q @ S.T, k @ G.T
    u = v - g[:, None] * sx
    e = M @ (be[:, None] * u)
    w = M.T @ (P.T @ dO + kb[:, None] * gk)
    dA = np.tril(-w @ e.T, -1)
    dG = be[:, None] * gam * dA
    dQK = gam * np.tril(dO @ e.T)
    dx = -(be * g)[:, None] * (w @ S) + dG @ k
    dq = g[:, None] * (dO @ S) + dQK @ k + lm[:, None] * dx
    dk = kb[:, None] * (e @ G) + dQK.T @ q + dG.T @ x + dx
    both = dG * xk + dQK * qk
    rows = both.sum(1) - both.sum(0) + g * ((dO * sq).sum(1) - be * (w * sx).sum(1))
    below = kb * (e * gk).sum(1)
    dla = [rows[j:].sum() + below[:j].sum() + g[-1] * (G * S).sum() for j in range(len(q))]
    z1, z2 = g[:, None] * (dO - (lm * be)[:, None] * w), -(g * be)[:, None] * w
    return dict(dq=dq, dk=dk, dv=be[:, None] * w, dbeta=(w * u).sum(1) + (dA * gam * xk).sum(1), dlam=(q * dx).sum(1),
                dlog_alpha=np.array(dla)), g[-1] * G + z1.T @ q + z2.T @ k


def blocks(T):
    return [slice(a, min(a + TB, T)) for a in range(0, T, TB)]


TOKENS = ("q", "k", "v", "beta", "lam", "alpha")


@pytest.mark.parametrize("T", [1, 15, 16, 17, 70])
def test_block_forward_equals_oracle(T):
    d, _ = inputs(T, 8, 5, 7 + T, zeros=(5, 33, 34))
    S, out = d["S0"], []
    for b in blocks(T):
        o, S = block_fwd(S, *(d[n][b] for n in TOKENS))
        out.append(o)
    sh = {n: d[n][None, :, None] for n in TOKENS}
    o_ref, S_ref = recurrent.fwd(sh["q"], sh["k"], sh["v"], sh["beta"], sh["lam"], None, d["S0"][None, None],
                                 alpha=sh["alpha"])
    assert np.abs(np.concatenate(out) - o_ref[0, :, 0]).max() <= 1e-12 * np.abs(o_ref).max()
    assert np.abs(S - S_ref[0, 0]).max() <= 1e-12 * np.abs(S_ref).max()


@pytest.mark.parametrize("spacing", [1, 2, 3])
@pytest.mark.parametrize("T", [1, 16, 17, 33, 49, 97])
def test_block_backward_equals_oracle_bptt(T, spacing):
    """The reverse walk over blocks, each from the last of the entry states stored every `spacing` blocks."""
    d, rng = inputs(T, 6, 5, 31 + T, zeros=(3, 20))
    dO, dSf = rng.standard_normal(d["v"].shape), rng.standard_normal(d["S0"].shape)
    bl = blocks(T)
    stored, S = {}, d["S0"]
    for c, b in enumerate(bl):
        if c % spacing == 0:
            stored[c] = S
        S = block_fwd(S, *(d[n][b] for n in TOKENS))[1]
    G, parts = dSf, []
    for c in reversed(range(len(bl))):
        S = stored[c // spacing * spacing]
        for b in bl[c // spacing * spacing:c]:
            S = block_fwd(S, *(d[n][b] for n in TOKENS))[1]
        grads, G = block_bwd(S, G, *(d[n][bl[c]] for n in TOKENS), dO[bl[c]])
        parts.insert(0, grads)
    got = {key: np.concatenate([p[key] for p in parts]) for key in parts[0]}
    sh = {n: d[n][None, :, None] for n in TOKENS}
    with np.errstate(divide="ignore"):
        la = np.log(sh["alpha"])
    ref = recurrent.bwd(sh["q"], sh["k"], sh["v"], sh["beta"], sh["lam"], la, d["S0"][None, None],
                        d_o=dO[None, :, None], d_final_state=dSf[None, None])
    for key, val in {**got, "d_initial_state": G}.items():
        r = ref[key][0, 0] if key == "d_initial_state" else ref[key][0, :, 0]
        assert np.abs(val - r).max() <= 1e-11 * max(1.0, np.abs(r).max()), key
