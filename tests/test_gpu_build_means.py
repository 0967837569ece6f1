"""Chunk means of shadowkv_build_landmarks where they are rounded in the upper words of fp64 numbers, and where a wave holds
a mean that is not a normal number of the storage type: least and largest numbers, zeros of either sign, infinities (-m gpu).
Bit for bit against the means in fp64 rounded once."""
import numpy as np
import pytest
import torch

from paper_2410_21465_amd import shadowkv as S

import parity_util as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kd", [0, 1])
@pytest.mark.parametrize("c,d", [(4, 64), (4, 96), (4, 128), (8, 64), (8, 128), (16, 64), (16, 96)])
def test_means_are_rounded_once(c, d, kd):
    n_ch = 203
    print(f"\n[case] c {c} d {d} kv_dtype {kd}", flush=True)
    gen = torch.Generator(device="cpu").manual_seed(100 * c + d)
    top = 2.0 ** 14 if kd else 2.0 ** 126
    low = 2.0 ** -16 if kd else 2.0 ** -133
    k = torch.randn(1, 1, n_ch, c, d, generator=gen, dtype=torch.float64)
    k[:, :, 8:12] *= low * 4            # around the least numbers
    k[:, :, 12:16] *= top               # some means round up to infinity
    k[:, :, 16:20] = 0.0
    k[:, :, 20:24] = -0.0
    k[:, :, 24, 1, 3] = float("inf")
    k[:, :, 28:60] *= torch.exp2(torch.randint(-12, 12, (32, c, d), generator=gen).double())   # wide sums: sticky bits
    k[:, :, 60:124, c // 2:] = -k[:, :, 60:124, :c // 2] * (1.0 + torch.exp2(-torch.randint(2, 9, (64, 1, d), generator=gen).double()))
    k = k.to(torch.float8_e5m2 if kd else torch.bfloat16).cuda()
    p = S.Params(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=d, ctx_len=n_ch * c, chunk_size=c, rank=8, n_outlier_chunks=0,
                 topk_chunks=1, local_len=0, kv_dtype=kd)
    got = S.build_landmarks(p, k.view(1, 1, n_ch * c, d).contiguous(), torch.zeros_like(k).view(1, 1, n_ch * c, d))
    torch.cuda.synchronize()
    K = PU.kv_to_f64(PU.to_bits(k, kd)).reshape(n_ch, c, d)
    mean = np.zeros((n_ch, d))
    for t in range(c):
        mean = mean + K[:, t]
    with np.errstate(over="ignore", invalid="ignore"):
        want = PU.kv_round(mean / c, kd)
    np.testing.assert_array_equal(PU.to_bits(got["landmarks"], kd)[0, 0], want)
