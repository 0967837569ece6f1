"""The default schedule of shadowkv_factorize_keys (plain steps, then shifted ones) against sixteen plain steps asked for with
n_iter, on spectra that converge slowly, fast, after a few strong directions, or not at all (-m gpu)."""
import numpy as np
import pytest
import torch

from paper_2410_21465_amd import shadowkv as S

import parity_util as PU

pytestmark = pytest.mark.gpu


def _scales(kind, D):
    x = torch.arange(D, dtype=torch.float64)
    if kind == "flat":
        return torch.ones(D, dtype=torch.float64)
    if kind == "harmonic":
        return 1.0 / (1.0 + x)
    if kind == "exp60":
        return torch.exp(-x / 60.0)
    if kind == "exp20":
        return torch.exp(-x / 20.0)
    out = torch.exp(-x / 100.0)
    out[:3] *= {"lead": 3e3, "far lead": 1e5}[kind]
    return out


# (spectrum, KV heads, head_dim, tokens, rank): more columns than vectors, from one more to eight times as many
CASES = [("flat", 8, 64, 2048, 160), ("harmonic", 4, 128, 1500, 160), ("exp60", 3, 128, 1500, 48), ("exp20", 4, 64, 900, 96),
         ("lead", 4, 128, 2048, 160), ("far lead", 4, 96, 1200, 48), ("exp60", 2, 64, 1000, 88), ("harmonic", 2, 96, 1000, 152),
         ("flat", 1, 64, 500, 24)]


@pytest.mark.parametrize("kind,h,d,s,r", CASES)
def test_default_steps_come_as_close_as_sixteen_plain_ones(kind, h, d, s, r):
    D = h * d
    print(f"\n[case] {kind} h {h} d {d} s {s} r {r}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(D + r)
    scale = _scales(kind, D)[torch.randperm(D, generator=gen)]
    k = (torch.randn(2, s, D, generator=gen, dtype=torch.float64) * scale).to(torch.bfloat16)
    p = S.Params(batch=2, n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=r, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0)
    out = {n: S.factorize_keys(p, k.cuda(), want_vectors=True, n_iter=n) for n in (0, 16)}
    torch.cuda.synchronize()
    for i in range(2):
        K = k[i].double().numpy()
        G = K.T @ K
        lam = np.linalg.eigvalsh(G)[::-1]
        res, miss = {}, {}
        for n, got in out.items():
            psi, sig = got["psi"][i].cpu().numpy(), got["sigma"][i].cpu().numpy()
            assert np.abs(psi @ psi.T - np.eye(r)).max() < 1e-12
            res[n] = np.linalg.norm(psi @ G - (sig ** 2)[:, None] * psi)
            miss[n] = lam[:r].sum() - np.einsum("ij,ij->", psi @ G, psi)   # energy that the best subspace has more
        print(f"[steps] residual / lam_1 {res[0] / lam[0]:.1e} (16: {res[16] / lam[0]:.1e}), energy {miss[0] / lam[0]:.1e} "
              f"({miss[16] / lam[0]:.1e}), lam_(m+1) / lam_r {lam[min(r + 32, D - 1)] / lam[r - 1]:.2f}", flush=True)
        # rounding: 1e-12 of the largest eigenvalue for sums of a few hundred terms
        assert res[0] <= res[16] + 1e-12 * lam[0]
        assert miss[0] <= miss[16] + 1e-12 * lam[0]


def test_sequences_of_a_batch_pause_by_themselves():
    """Sequences whose shifted steps go without orthonormalisation two at a time, one at a time and not at all, in one batch:
    each as close as after sixteen plain steps (the bounds as above), the first also alone (sums in another order)."""
    h, d, s, r = 4, 128, 1200, 160
    D = h * d
    gen = torch.Generator(device="cpu").manual_seed(7)
    x = torch.arange(D, dtype=torch.float64)
    scales = [torch.exp(-x / 100.0), torch.exp(-x / 14.0), torch.exp(-x / 30.0), torch.ones(D, dtype=torch.float64)]
    k = torch.stack([torch.randn(s, D, generator=gen, dtype=torch.float64) * c for c in scales]).to(torch.bfloat16)

    def run(keys, n):
        p = S.Params(batch=len(keys), n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=r, n_outlier_chunks=0,
                     topk_chunks=1, local_len=0)
        got = S.factorize_keys(p, keys.cuda(), want_vectors=True, n_iter=n)
        return got["psi"].cpu().numpy(), got["sigma"].cpu().numpy()

    many, plain, alone = run(k, 0), run(k, 16), run(k[:1], 0)
    for i in range(len(scales)):
        K = k[i].double().numpy()
        G = K.T @ K
        top = np.linalg.eigvalsh(G)[-1]
        residual = [np.linalg.norm(psi[i] @ G - (sig[i] ** 2)[:, None] * psi[i]) for psi, sig in (many, plain)]
        print(f"[case] sequence {i}: residual / lam_1 {residual[0] / top:.1e} (16: {residual[1] / top:.1e})", flush=True)
        assert np.abs(many[0][i] @ many[0][i].T - np.eye(r)).max() < 1e-12
        assert residual[0] <= residual[1] + 1e-12 * top
    # singular values to rounding: 1e-12 of the largest squared one, as the residuals
    assert np.abs(alone[1][0] ** 2 - many[1][0] ** 2).max() <= 1e-12 * many[1][0][0] ** 2


def _factored(k, h, d, r):
    p = S.Params(batch=len(k), n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=k.shape[1], chunk_size=1, rank=r, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0)
    out = {n: S.factorize_keys(p, k.cuda(), want_vectors=True, n_iter=n) for n in (0, 16)}
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("lead", [1e6, 1e8])
def test_sequences_whose_weakest_pivots_are_rounding_take_sixteen_plain_steps(lead):
    """One direction so far above the others that what it leaves in the last vectors after a step is more than their own length: there
    is no shift to go by, and the default is what n_iter = 16 asks for, bit for bit (the same products in the same order)."""
    h, d, s, r = 4, 128, 1500, 160
    print(f"\n[case] lead {lead}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(int(np.log10(lead)))
    scale = torch.exp(-torch.arange(h * d, dtype=torch.float64) / 100.0)
    scale[0] *= lead
    k = (torch.randn(1, s, h * d, generator=gen, dtype=torch.float64) * scale).to(torch.bfloat16)
    out = _factored(k, h, d, r)
    for name in ("psi", "sigma", "A", "B"):
        assert torch.equal(out[0][name].cpu(), out[16][name].cpu()), name


@pytest.mark.parametrize("h,d,r,level,drop", [(2, 128, 32, 64, 0.117), (2, 128, 32, 74, 0.117), (2, 128, 32, 74, 0.25), (2, 128, 32, 40, 0.25),
                                              (4, 128, 160, 202, 0.117), (4, 128, 160, 192, 0.25), (4, 128, 160, 170, 0.06)])
def test_level_spectra_that_drop(h, d, r, level, drop):
    """`level` equal eigenvalues and the rest `drop` of these, the drop anywhere from inside the r + 32 vectors to beyond them: points of
    [0, b] with b hardly below the r-th eigenvalue would damp next to nothing."""
    D = h * d
    print(f"\n[case] D {D} r {r} level {level} drop {drop}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(level)
    scale = torch.where(torch.arange(D) < level, 1.0, drop ** 0.5).double()
    # orthonormal columns; rounding to storage moves the eigenvalues by some thousandths
    q = torch.linalg.qr(torch.randn(2 * D, D, generator=gen, dtype=torch.float64))[0]
    k = (q * scale[torch.randperm(D, generator=gen)]).to(torch.bfloat16).contiguous()[None]
    out = _factored(k, h, d, r)
    K = k[0].double().numpy()
    G = K.T @ K
    lam = np.linalg.eigvalsh(G)[::-1]
    res, miss = {}, {}
    for n, got in out.items():
        psi, sig = got["psi"][0].cpu().numpy(), got["sigma"][0].cpu().numpy()
        assert np.abs(psi @ psi.T - np.eye(r)).max() < 1e-12
        res[n] = np.linalg.norm(psi @ G - (sig ** 2)[:, None] * psi)
        miss[n] = lam[:r].sum() - np.einsum("ij,ij->", psi @ G, psi)
    print(f"[steps] residual / lam_1 {res[0] / lam[0]:.1e} (16: {res[16] / lam[0]:.1e}), energy {miss[0] / lam[0]:.1e} "
          f"({miss[16] / lam[0]:.1e})", flush=True)
    # rounding: 1e-12 of the largest eigenvalue for sums of a few hundred terms
    assert res[0] <= res[16] + 1e-12 * lam[0]
    assert miss[0] <= miss[16] + 1e-12 * lam[0]
