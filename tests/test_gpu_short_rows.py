"""GPU tests of the dense schedule in one kernel (rows of up to 2048 keys, scores kept on chip) at the sizes where it can go
wrong: the edges of its key blocks, of its register forms and of its query groups, against the single pass, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2605_02568_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _problem(seed, B, S, H, D, T, scores):
    g = torch.Generator(device="cpu").manual_seed(seed)
    if scores == "ties":
        q = torch.randint(-1, 2, (B, S, H, D), generator=g).float()
        K = torch.randint(-1, 2, (B, T, D), generator=g).float()
        w = torch.ones((B, S, H))
    else:
        q = torch.randn((B, S, H, D), generator=g)
        K = torch.randn((B, T, D), generator=g)
        w = torch.randn((B, S, H), generator=g) / np.sqrt(H)
    if scores == "equal":
        K[:] = K[:, :1]
    if scores == "negative":  # zeros are the best
        w = -w.abs()
    return q.to(torch.bfloat16).to(DEV), K.to(torch.bfloat16).to(DEV), w.to(DEV)


@pytest.mark.parametrize("scores", ["distinct", "ties", "equal", "negative"])
@pytest.mark.parametrize("B,S,H,D,T,m,k,mask", [
    (1, 9, 64, 128, 1, 1, 5, 0),           # one key
    (2, 9, 5, 32, 255, 1, 16, 0),          # few rows, short lists
    (1, 1537, 33, 64, 63, 1, 64, 0),       # short of a block of keys, lists longer than the row; a group of one query
    (1, 1538, 64, 128, 1024, 4, 512, 0),   # the longest row of the shorter form
    (1, 1539, 64, 128, 1025, 4, 513, 0),   # one key more, one entry more
    (1, 1540, 64, 128, 2048, 4, 1024, 0),  # the longest row
    (1, 1541, 16, 128, 2047, 4, 1000, 0),
    (1, 1541, 32, 128, 65, 4, 17, 0),
    (3, 515, 48, 64, 2048, 4, 512, 0),
    (3, 515, 64, 64, 1023, 4, 4000, 0),    # lists longer than any
    (2, 771, 20, 64, 1500, 4, 300, 0),
    (2, 771, 64, 32, 2000, 4, 700, 0),
    (2, 771, 32, 32, 1030, 4, 512, 0),
    (1, 900, 8, 32, 640, 4, 100, 0),       # fewer rows
    (1, 8, 64, 128, 1024, 4, 512, 0),      # the fewest
    (1, 768, 64, 64, 1025, 4, 700, 0),     # the fewest beyond 1024 keys
    (1, 2049, 64, 128, 2049, 1, 600, 1),   # causal: rows of 1 to 2048 keys, one beyond them all
    (2, 1203, 33, 64, 1203, 1, 300, 1),
    (1, 8190, 4, 32, 5000, 4, 1024, 1),    # a cache longer than any row sees; rows without keys
    (2, 40, 48, 64, 9001, 4, 200, 1),      # rows of 10 keys against a long cache
    (2, 8, 64, 128, 65536, 4, 16, 1),      # of at most 2
    (1, 300, 8, 32, 513, 1, 300, 1),
    (1, 2500, 8, 32, 700, 4, 2048, 1),
])
def test_short_rows_are_bit_identical(B, S, H, D, T, m, k, mask, scores):
    print(f"short rows B={B} S={S} H={H} D={D} T={T} m={m} k={k} mask={mask} {scores}", flush=True)
    if mask == 1 and S // m > 2048:
        S, T = 2048 * m + m - 1, max(T, 2048)
    q, K, w = _problem(S + T + k, B, S, H, D, T, scores)
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    ws = torch.empty(max(P.si_fused_workspace_bytes(B, S, H, D, T, min(k, 2048)), P.si_workspace_bytes(B, S, H, D, T, k, S, T)),
                     dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, mask, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    # one launch that scores and selects
    assert prof["score_tile"][1] == 1 and sum(n for _, n in prof.values()) == 1
    if k <= 2048:
        P.si_indexer_topk_fused(q, K, w, m, k, mask, 0, *out[1], ws)
    else:
        P.si_indexer_topk_tiled(q, K, w, m, k, mask, S, T, *out[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))


@pytest.mark.parametrize("B,S,H,D,T,m,k,mask,one", [
    (1, 1792, 1, 32, 1000, 1, 501, 0, False),  # half the scores are 0, and some are wanted
    (1, 1792, 1, 32, 1000, 1, 500, 0, True),
    (1, 1791, 1, 32, 1000, 1, 501, 0, True),
    (2, 900, 2, 64, 600, 1, 451, 0, False),    # a quarter
    (2, 900, 2, 64, 600, 1, 450, 0, True),
    (1, 1800, 3, 128, 700, 1, 613, 0, False),  # an eighth
    (1, 1800, 4, 128, 700, 1, 690, 0, True),
    (1, 1800, 2, 32, 256, 1, 256, 0, True),    # shorter lists
    (1, 1800, 1, 32, 129, 1, 2000, 0, False),  # every key wanted
    (1, 4001, 1, 32, 5000, 4, 600, 1, False),
    (1, 6001, 1, 32, 1000, 1, 501, 0, True),   # the single pass's workspace does not hold the scores
])
def test_rows_that_end_among_zeros(B, S, H, D, T, m, k, mask, one):
    """Rows of few heads whose best end among scores of exactly 0 are selected by a kernel of their own, where the scores fit."""
    print(f"ends among zeros B={B} S={S} H={H} D={D} T={T} m={m} k={k} mask={mask}", flush=True)
    q, K, w = _problem(S + T + k, B, S, H, D, T, "distinct")
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    ws = torch.empty(P.si_fused_workspace_bytes(B, S, H, D, T, k), dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, mask, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == 1 and sum(n for _, n in prof.values()) == (1 if one else 2)
    P.si_indexer_topk_fused(q, K, w, m, k, mask, 0, *out[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))
