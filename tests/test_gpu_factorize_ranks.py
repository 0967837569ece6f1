"""shadowkv_factorize_keys over the ranks at which its small linear algebra changes shape (-m gpu): block rows of the
Cholesky factor held per kernel (5 / 12 / 14 / 18 blocks of 16 vectors), vector counts that are no multiple of 16 or 32,
as many vectors as the keys are wide, products of few tiles and of more than 1024 (with ragged edges, sequences apart),
three to five rank tiles per wave of the projection in both storage types, and a spectrum with a few directions above
the rest."""
import numpy as np
import pytest
import torch

from paper_2410_21465_amd import shadowkv as S

import parity_util as PU
from test_gpu_factorize import ulp_distance

pytestmark = pytest.mark.gpu

# (batch, KV heads, head_dim, tokens, rank, leading directions of 30 times the others' scale, storage type)
CASES = [
    (1, 1, 64, 96, 8, 0, 0),         # 40 vectors
    (2, 1, 64, 500, 64, 0, 0),       # as many vectors as columns
    (1, 3, 64, 1500, 48, 2, 0),      # 80 vectors: the last size of the smallest kernel
    (3, 2, 96, 700, 56, 0, 0),       # 88 vectors: the first of the next
    (1, 4, 96, 1111, 160, 3, 0),     # 192 vectors, the default rank
    (1, 4, 128, 2048, 168, 0, 0),    # 200 vectors
    (1, 4, 128, 1024, 192, 3, 0),    # 224 vectors
    (1, 5, 96, 1500, 200, 0, 0),     # 232 vectors
    (2, 6, 64, 1024, 256, 0, 0),     # 288 vectors
    # 200 vectors of 1024 columns in 24 sequences: 5376 tiles of 32 x 32 (X G), 4608 (V X) and 1176 (X X^T, T), which
    # 64 x 64 blocks do not divide
    (24, 8, 128, 1100, 168, 0, 0),
    (16, 8, 128, 1100, 168, 2, 1),   # 3584, 3072 and 784 tiles; FP8 keys with four rank tiles per wave
]


@pytest.mark.parametrize("b,h,d,s,r,lead,kd", CASES)
def test_factors_at_every_shape_of_the_small_algebra(b, h, d, s, r, lead, kd):
    D = h * d
    print(f"\n[case] b {b} h {h} d {d} s {s} r {r} lead {lead} kv_dtype {kd}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(1000 * r + D)
    # columns of graded scale in any order: rounding to storage is relative to each, so the weak ones keep their place in
    # the spectrum (mixed into all columns they would end in the rounding of the strong ones, which is flat)
    scale = torch.exp(-torch.arange(D, dtype=torch.float64) / 32.0)
    scale[:lead] *= 30.0
    k = torch.stack([torch.randn(s, D, generator=gen, dtype=torch.float64) * scale[torch.randperm(D, generator=gen)]
                     for _ in range(b)])
    k = (k * (8.0 / scale.max())).to(torch.float8_e5m2 if kd else torch.bfloat16)
    p = S.Params(batch=b, n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=r, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0, kv_dtype=kd)
    got = S.factorize_keys(p, k.cuda(), want_vectors=True)
    torch.cuda.synchronize()
    psi, sig = got["psi"].cpu().numpy(), got["sigma"].cpu().numpy()
    gA, gB = PU.to_bits(got["A"], kd), PU.to_bits(got["B"], kd)
    for i in range(b):
        K = k[i].double().numpy()
        G = K.T @ K
        lam = np.linalg.eigvalsh(G)[::-1]
        assert np.abs(psi[i] @ psi[i].T - np.eye(r)).max() < 1e-12
        # rounding: 1e-12 of the largest eigenvalue.  Convergence: 16 iterations leave of the directions outside the
        # m = r + 32 vectors a share (lam_{m+1} / lam_r)^16 of the start's, whose angle to a wanted direction has a tangent of
        # order sqrt(D), 100 with room; a Ritz residual goes with that angle, a Ritz value with its square
        m = min(D, r + 32)
        tan = 100.0 * (max(lam[m], 0.0) / lam[r - 1]) ** 16 if m < D else 0.0
        assert tan < 1e-3 and 1e-12 * lam[0] < 1e-3 * lam[r - 1], "bounds that say nothing about the weakest directions"
        resid = np.abs(psi[i] @ G - (sig[i] ** 2)[:, None] * psi[i]).max()
        assert np.abs(sig[i] ** 2 - lam[:r]).max() <= 1e-12 * lam[0] + lam[r - 1] * tan ** 2
        assert resid <= 1e-12 * lam[0] + lam[r - 1] * tan, (resid / lam[0], tan)
        assert np.all(np.diff(sig[i]) <= 0)
        # B and A are the roundings of psi and K psi; a sum in another order may fall on the other side of a boundary
        np.testing.assert_array_equal(gB[i], PU.kv_round(psi[i].reshape(r, h, d).transpose(1, 0, 2), kd))
        far = ulp_distance(gA[i, :s], PU.kv_round(K @ psi[i].T, kd), kd)
        assert far.max() <= 1 and (far > 0).mean() < 1e-3, (far.max(), (far > 0).mean())


@pytest.mark.parametrize("exp2", [-133, 0, 126])
@pytest.mark.parametrize("h,d,s,r", [(1, 64, 300, 64), (2, 96, 1000, 160)])
def test_keys_at_the_ends_of_the_storage_types_range(h, d, s, r, exp2):
    """Keys of 0 and +-2^exp2, from the least bf16 number to nearly the largest, with as many vectors as columns, so that the
    Ritz step alone decides.  What its rotations look at are fourth powers of singular values, and the product of two of
    those leaves the range of fp64 at both ends."""
    D = h * d
    print(f"\n[case] h {h} d {d} s {s} r {r} scale 2^{exp2}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(D)
    K = torch.randint(-1, 2, (s, D), generator=gen).double()
    k = (K * 2.0 ** exp2).to(torch.bfloat16)[None]
    assert torch.equal(k[0].double() * 2.0 ** -exp2, K)
    p = S.Params(batch=1, n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=r, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0)
    got = S.factorize_keys(p, k.cuda(), want_vectors=True)
    torch.cuda.synchronize()
    psi, sig = got["psi"][0].cpu().numpy(), got["sigma"][0].cpu().numpy() * 2.0 ** -exp2
    G = (K.T @ K).numpy()
    lam = np.linalg.eigvalsh(G)[::-1]
    # rounding only, of sums of at most a thousand terms: 1e-12 of the largest eigenvalue
    assert np.abs(psi @ psi.T - np.eye(r)).max() < 1e-12
    assert np.abs(sig ** 2 - lam[:r]).max() <= 1e-12 * lam[0]
    assert np.abs(psi @ G - (sig ** 2)[:, None] * psi).max() <= 1e-12 * lam[0]


# Exponent of column x's scale.  The largest eigenvalue over that of the last vector decides after how many shifted steps vectors
# are made orthonormal again: three up to 10^(13/3), two up to 10^6.5, each beyond.
GRADED = {
    3: lambda x: -min(8, max(0, (x - 128) // 16)),
    2: lambda x: -min(12, x // 20),
    1: lambda x: -min(20, x // 12),
}


@pytest.mark.parametrize("pause", [0, 1, 2, 3])
@pytest.mark.parametrize("end", ["least", -90, 0, 90, "most"])
def test_keys_at_the_ends_of_the_range_with_fewer_vectors_than_columns(pause, end):
    """Keys of 0 and +-2^e with graded (pause > 0) and equal columns, 192 vectors of 512: the steps that follow each other without
    an orthonormalisation take eigenvalues to their third power and the products of vectors to the sixth."""
    h, d, s, r = 4, 128, 1000, 160
    D = h * d
    exps = torch.tensor([GRADED[pause](x) if pause else 0 for x in range(D)], dtype=torch.float64)
    exp2 = {"least": -133 - int(exps.min()), "most": 126}.get(end, end)
    print(f"\n[case] pause {pause} scale 2^{exp2}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(D + pause)
    K = torch.randint(-1, 2, (s, D), generator=gen).double() * torch.exp2(exps)[torch.randperm(D, generator=gen)]
    k = (K * 2.0 ** exp2).to(torch.bfloat16)[None]
    assert torch.equal(k[0].double() * 2.0 ** -exp2, K)
    p = S.Params(batch=1, n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=r, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0)
    got = {n: S.factorize_keys(p, k.cuda(), want_vectors=True, n_iter=n) for n in (0, 16)}
    torch.cuda.synchronize()
    G = (K.T @ K).numpy()
    lam = np.linalg.eigvalsh(G)[::-1]
    ratio = lam[0] / lam[r + 31]
    assert {3: 1.0, 2: 1e13 ** (1 / 3), 1: 1e6 * 10 ** 0.5}.get(pause, 0.0) < ratio < {3: 1e13 ** (1 / 3), 2: 1e6 * 10 ** 0.5}.get(pause, np.inf)
    res = {}
    for n, g in got.items():
        psi, sig = g["psi"][0].cpu().numpy(), g["sigma"][0].cpu().numpy() * 2.0 ** -exp2
        assert np.abs(psi @ psi.T - np.eye(r)).max() < 1e-12
        res[n] = np.linalg.norm(psi @ G - (sig ** 2)[:, None] * psi)
    print(f"[ends] residual / lam_1 {res[0] / lam[0]:.1e} (16 plain steps {res[16] / lam[0]:.1e})", flush=True)
    # rounding, of sums of at most a thousand terms: 1e-12 of the largest eigenvalue
    assert res[0] <= res[16] + 1e-12 * lam[0]
