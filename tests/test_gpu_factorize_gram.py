"""The dense products of shadowkv_factorize_keys (-m gpu), G = K^T K and A = K Psi: formed from 8-bit digits, from lists of
what the keys' digits leave out, or in fp64 for sequences with too much of that; every case says which of these it
is for.  With as many vectors as the keys are wide,
sigma^2 and the right singular vectors give G back, and it is compared with numpy's fp64 product of the same stored keys, A
with the rounding of theirs with the vectors: at the edges of the 128-column blocks, of stages of 64 tokens, blocks of 256 and
the 32768 tokens summed in 32 bits, and for keys of each kind."""
import numpy as np
import pytest
import torch

from paper_2410_21465_amd import shadowkv as S

import parity_util as PU
from test_gpu_factorize import ulp_distance

pytestmark = pytest.mark.gpu


def _keys(kind, b, s, D, kd, gen):
    n = b if b * s * D <= 2 ** 28 else 4          # (very large batches repeat four sequences)
    k = torch.randn(n, s, D, generator=gen, device="cuda")
    if kind == "outliers":        # a row in 500 above the rest: the lists hold several times what normal keys leave out
        k[:, ::500] *= 128.0 if kd else 6.0
    elif kind == "crowded":       # ... more above: one element in 1024 is left out, three quarters of what the lists hold
        k[:, ::500] *= 15.0
    elif kind == "spikes":        # ... far above: the others' last places lie below the digits, more than the lists hold
        k[:, ::500] *= 3000.0
    elif kind == "graded":        # magnitudes over 20 binades in every column: more is left out than the lists hold
        k *= torch.exp2((12.0 if kd else 0.0) - 20.0 * torch.rand(n, s, D, generator=gen, device="cuda"))
    elif kind == "faint":         # a row in 61 whose few elements are all left out by the digits
        faint = torch.zeros(s, 1, device="cuda")
        faint[::61] = 1.0
        some = (torch.arange(D, device="cuda") % 16 == 3).float()
        k = torch.where(faint > 0, k * some * 2.0 ** (-10 if kd else -17), k * 2.0 ** (10 if kd else 0))
    elif kind == "columns":       # columns of very different scale, one of them zero
        k *= torch.exp2(torch.linspace(-12, 8, D, device="cuda"))
        k[:, :, D // 2] = 0.0
    elif kind == "unseen":        # as graded, in tokens that the sample of evenly spaced ones skips: found by full lists
        k[:, s // 4 + 1:s // 4 + 513:2] *= torch.exp2(-20.0 * torch.rand(n, 256, D, generator=gen, device="cuda"))
        k *= 2.0 ** (12 if kd else 0)
    elif kind == "last":          # one element that its digits do not hold, in the last token of a short sequence
        k[:, -1, 3] = 1.125 * 2.0 ** -21
    elif kind == "large":         # beyond 2^22: fp64 (bf16 only)
        k *= 2.0 ** 30
    elif kind == "mixed":         # one sequence of each route
        k[0, ::500] *= 6.0
        k[1] *= torch.exp2(-20.0 * torch.rand(s, D, generator=gen, device="cuda"))
    elif kind == "absent":        # a column far above the others that some tokens do not have: of theirs the weak entries of its
        k *= 2.0 ** (-9 if kd else -4)                           # vectors are all there is
        k[:, :, 3] *= 2.0 ** (20 if kd else 22)
        k[:, ::61, 3] = 0.0
    elif kind == "lone":          # a column that one token has
        k *= 2.0 ** -6
        k[:, :, 5] = 0.0
        k[:, s // 2, 5] = 2.0 ** (15 if kd else 20)
    elif kind == "ones":          # magnitudes with all leading bits set, of either sign
        k = torch.where(k < 0, -255.0, 255.0)
    k = k.clamp(-5.0e4, 5.0e4).to(torch.float8_e5m2) if kd else k.to(torch.bfloat16)
    return k if n == b else k.view(torch.uint8).repeat(b // n, 1, 1).view(k.dtype)


# the last number: which way the sequences go (shadowkv_factorize_plan): 0 digits, 1 fp64 sums, 2 only A in fp64 (fewer tokens
# than vectors: the spare vectors' entries cancel to rounding)
CASES = [(1, 1, 64, 1, "normal", 0, 2), (1, 1, 64, 63, "normal", 0, 2), (2, 1, 64, 65, "normal", 1, 0),
         (1, 1, 96, 513, "normal", 0, 0), (1, 1, 128, 4096, "normal", 0, 0), (3, 3, 64, 1500, "outliers", 0, 0),
         (1, 2, 96, 3001, "outliers", 1, 0), (1, 2, 128, 2049, "outliers", 0, 0), (1, 2, 128, 2000, "graded", 0, 1),
         (2, 2, 64, 1200, "spikes", 0, 1), (1, 2, 128, 4000, "faint", 0, 0), (2, 2, 96, 1000, "faint", 0, 0),
         (1, 4, 64, 1111, "graded", 1, 1), (1, 2, 128, 2500, "faint", 1, 0), (2, 3, 64, 777, "columns", 0, 0),
         (1, 2, 128, 600, "large", 0, 1), (3, 2, 128, 1000, "mixed", 0, (0, 1, 0)), (2, 3, 64, 4096, "unseen", 0, 1),
         (1, 2, 96, 8192, "unseen", 1, 1), (1, 1, 64, 100, "last", 0, 0), (1, 1, 128, 4000, "absent", 0, 0), (2, 2, 96, 3000, "absent", 1, 0),
         (1, 2, 128, 2000, "lone", 0, 2), (2, 3, 64, 1000, "lone", 1, 2), (1, 2, 128, 5000, "ones", 0, 0),
         (1, 1, 64, 70001, "outliers", 0, 0), (40, 4, 64, 600, "graded", 0, 1), (80, 4, 64, 600, "graded", 0, 1),
         (180, 4, 64, 520, "graded", 1, 1),
         (256, 1, 64, 33000, "normal", 0, 0),
         # one token part of more than the 32768 tokens summed in 32 bits, off the diagonal too
         (1024, 3, 64, 33000, "crowded", 0, 0), (2048, 1, 64, 33000, "outliers", 1, 0)]


def test_the_fp64_cases_have_every_number_of_waves():
    waves = {S.factorize_plan(S.Params(batch=b, n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=h * d,
                                       n_outlier_chunks=0, topk_chunks=1, local_len=0, kv_dtype=kd))["fp64_waves"]
             for b, h, d, s, _, kd, route in CASES if route == 1}
    assert waves == {1, 2, 4, 8}


def _left_out(K):
    """Elements of K [s, D] that three 8-bit digits do not hold: no multiples of 2^-22 times a power of two above the column."""
    v = np.ldexp(K, 22 - np.frexp(np.abs(K).max(axis=0))[1])
    return int((v != np.rint(v)).sum())


@pytest.mark.parametrize("b,h,d,s,kind,kd,route", CASES)
def test_gram_matrix_from_the_factors(b, h, d, s, kind, kd, route):
    D = h * d
    print(f"\n[case] b {b} h {h} d {d} s {s} {kind} kv_dtype {kd}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7 * s + D + kd)
    k = _keys(kind, b, s, D, kd, gen)
    p = S.Params(batch=b, n_q_heads=h, n_kv_heads=h, head_dim=d, ctx_len=s, chunk_size=1, rank=D, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0, kv_dtype=kd)
    got = S.factorize_keys(p, k, want_vectors=True)
    again = S.factorize_keys(p, k, want_vectors=True)
    torch.cuda.synchronize()
    assert torch.equal(got["psi"], again["psi"]) and torch.equal(got["sigma"], again["sigma"])   # the same order of sums on every run
    routes, plan = S.factorize_routes(p, got["workspace"]).tolist(), S.factorize_plan(p)
    others = [(i, x) for i, x in enumerate(routes) if x != (route if isinstance(route, int) else route[i])]
    assert not others[:8]
    assert plan["parts"] * plan["tokens_per_part"] >= s and (plan["tokens_per_part"] > 32768) == (b >= 1024), plan
    psi, sig = got["psi"].cpu().numpy(), got["sigma"].cpu().numpy()
    for i in sorted({0, 1 % b, b - 1}):
        K = PU.kv_to_f64(PU.to_bits(k[i].contiguous(), kd))
        if kind in ("outliers", "crowded", "faint"):
            assert _left_out(K) > 0
        G = K.T @ K
        back = (psi[i].T * sig[i] ** 2) @ psi[i]
        # the eigenvectors' rounding: a few D units of the last place of the largest eigenvalue; directions beyond the rank of
        # the keys are rounding as well
        err = np.abs(back - G).max() / np.linalg.norm(G, 2)
        print(f"[gram] sequence {i}: {err:.2e}", flush=True)
        assert err < 32 * D * 2.0 ** -53, err
        # A: fp64 sums of the stored keys times these vectors, rounded once (another order of the sums moves a number across
        # a rounding boundary with a probability of some 2^-40)
        A = K @ psi[i].T
        stored = torch.from_numpy(A).to(k.dtype)     # torch rounds through fp32: a unit of the last place in rare cases
        d = ulp_distance(PU.to_bits(got["A"][i, :s].contiguous(), kd), PU.to_bits(stored, kd), kd)
        big = np.abs(A) > 1e-9 * np.abs(K).max(axis=1, keepdims=True)    # (sums that cancel to rounding have no digits to compare)
        assert d[big].max(initial=0) <= 1 and (d[big] > 0).mean() < 1e-4, (d[big].max(initial=0), (d[big] > 0).mean())


@pytest.mark.parametrize("s,route", [(2 ** 25, 0), (2 ** 25 + 16, 1)])
def test_as_many_tokens_as_a_list_entry_can_name(s, route):
    """An entry of the digits' lists has 25 bits for its token; a longer sequence is summed in fp64."""
    D = 64
    print(f"\n[case] s {s}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(s % 1000)
    k = torch.empty(1, s, D, dtype=torch.bfloat16, device="cuda")
    for part in k[0].split(2 ** 22):
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda"))
    p = S.Params(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=D, ctx_len=s, chunk_size=1, rank=D, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0)
    got = S.factorize_keys(p, k, want_vectors=True)
    assert S.factorize_routes(p, got["workspace"]).tolist() == [route]
    G = torch.zeros(D, D, dtype=torch.float64, device="cuda")
    for part in k[0].split(2 ** 21):
        x = part.double()
        G += x.t().contiguous() @ x
    psi, sig = got["psi"][0].cpu().numpy(), got["sigma"][0].cpu().numpy()
    G = G.cpu().numpy()
    err = np.abs((psi.T * sig ** 2) @ psi - G).max() / np.linalg.norm(G, 2)
    # the eigenvectors' rounding as above; the reference adds 2^21 products at a time in fp64: a random walk of 2^-53 each
    assert err < (32 * D + 2 ** 11) * 2.0 ** -53, err
    for rows in (slice(0, 1000), slice(s - 1000, s)):
        A = PU.kv_to_f64(PU.to_bits(k[0, rows].contiguous(), 0)) @ psi.T
        d = ulp_distance(PU.to_bits(got["A"][0, rows].contiguous(), 0), PU.to_bits(torch.from_numpy(A).to(k.dtype), 0), 0)
        assert d.max() <= 1 and (d > 0).mean() < 1e-3
