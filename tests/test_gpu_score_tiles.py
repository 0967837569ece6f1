"""Logits and selection with one, two and four 16-row tiles per scoring wave, at row counts around the tiles' edges, against
fp64.  Which of them runs follows from the number of workgroups and from the room for the tiles' pairs (16 bytes each, in
4 * topk_chunks * chunk_size bytes per head): the budgets below leave room for 64-row, 128-row or only 256-row workgroups.  Longer
contexts, of more pairs than a wave has lanes, and selections that go through slices and a merge of their survivors."""
import pytest
import torch

from paper_2410_21465_amd import shadowkv as S

pytestmark = pytest.mark.gpu

N_C = [1, 63, 65, 127, 257, 1000]


def _check(d, fp8, G, n_c, c, k):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000 * d + 100 * G + n_c)
    p = S.Params(batch=1, n_q_heads=2 * G, n_kv_heads=2, head_dim=d, ctx_len=n_c * c, chunk_size=c, rank=16,
                 n_outlier_chunks=0, topk_chunks=k, local_len=0, rope_theta=1e4,
                 kv_dtype=S.KV_FP8_E5M2 if fp8 else S.KV_BF16)

    def rnd(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")

    st = p.kv_torch_dtype
    q = rnd(1, 2 * G, d).bfloat16()
    lm = rnd(1, 2, n_c, d).to(st)
    ids = torch.arange(n_c, dtype=torch.int32, device="cuda").repeat(1, 2, 1)
    none = torch.empty(1, 2, 0, d, dtype=st, device="cuda")
    _, got, ws = S.decode_step(p, q, rnd(1, n_c * c, 16).to(st), rnd(1, 2, 16, d).to(st), lm, ids, none, none, none, none,
                               rnd(1, 2, n_c * c, d).to(st), torch.zeros(1, dtype=torch.int32, device="cuda"))
    want = q.cpu().double().view(2, G, d) @ lm.cpu().double()[0].transpose(1, 2) * d ** -0.5
    logits = S.workspace_view(p, ws, "logits").cpu().double().view(2, G, n_c)
    # one rounding to fp32, and fp64 sums of d products in another order
    bound = 2.0 ** -24 * want.abs() + 1e-13 * d
    assert torch.all((logits - want).abs() <= bound)
    score = torch.log_softmax(want, dim=-1).amax(dim=1)
    top = score.sort(dim=-1, descending=True)
    for u in range(2):
        if k < n_c and float(top.values[u, k - 1] - top.values[u, k]) < 1e-6:
            continue                      # a tie, as everywhere
        assert got[0, u].cpu().tolist() == sorted(top.indices[u, :k].tolist())
    return p


@pytest.mark.parametrize("room", ["64", "128", "256"])
@pytest.mark.parametrize("G", [1, 4, 7, 16])
@pytest.mark.parametrize("d,fp8", [(64, False), (96, True), (128, False), (128, True)])
def test_logits_and_selection(d, fp8, G, room):
    for n_c in N_C:
        print(f"[case] d {d} fp8 {fp8} G {G} room {room} n_c {n_c}", flush=True)
        pairs = -(-n_c // int(room))
        c = 4
        k = min(n_c, pairs)                   # 4 k c = 16 k bytes: room for so many pairs and no more
        p = _check(d, fp8, G, n_c, c, k)
        assert S.decode_score_rows(p) == next(rows for rows in (64, 128, 256) if -(-n_c // rows) <= pairs)


@pytest.mark.parametrize("G,fp8,rows,n_c,k", [(4, False, 64, 4161, 86), (4, True, 128, 9000, 90), (7, False, 64, 4999, 104),
                                              (16, False, 64, 4100, 85), (16, True, 256, 33000, 687)])
def test_more_pairs_than_lanes(G, fp8, rows, n_c, k):
    """65 pairs a head and more, on which the softmax normaliser rests."""
    print(f"[case] G {G} fp8 {fp8} n_c {n_c}", flush=True)
    p = _check(64, fp8, G, n_c, 4, k)
    assert S.decode_score_rows(p) == rows


# 9 survivors, 25, 50, 1651, 13151 and, through a middle level, 32468: no multiples of four, a unit's begin at any entry
@pytest.mark.parametrize("n_c,k", [(32769, 1), (32769, 3), (40001, 5), (50003, 127), (50003, 1025), (70000, 7001)])
@pytest.mark.parametrize("G", [2, 16])
def test_survivors_of_slices(n_c, k, G):
    print(f"[case] G {G} n_c {n_c} k {k}", flush=True)
    p = _check(64, False, G, n_c, 1, k)
    assert S.decode_plan(p)["selection_launches"] == (3 if k == 7001 else 2)
