"""GPU tests of the dense schedule (few rows or short key ranges: scores to the workspace, then a
workgroup-level selection) at the sizes where it can go wrong: bit-identical to the single pass or the
tiled schedule, and the selection alone, exactly, against the oracle's sort."""
import numpy as np
import pytest
import torch

import paper_2605_02568_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _problem(seed, B, S, H, D, T, ties):
    g = torch.Generator(device="cpu").manual_seed(seed)
    if ties:
        q = torch.randint(-1, 2, (B, S, H, D), generator=g).float()
        K = torch.randint(-1, 2, (B, T, D), generator=g).float()
        w = torch.ones((B, S, H))
    else:
        q = torch.randn((B, S, H, D), generator=g)
        K = torch.randn((B, T, D), generator=g)
        w = torch.randn((B, S, H), generator=g) / np.sqrt(H)
    return q.to(torch.bfloat16).to(DEV), K.to(torch.bfloat16).to(DEV), w.to(DEV)


@pytest.mark.parametrize("B,S,H,D,T,m,k,mask,ties", [
    (1, 1, 64, 128, 1, 4, 5, 0, False),         # one key
    (3, 1, 1, 32, 4095, 4, 4096, 0, False),     # one query per batch, fewer keys than k
    (2, 2, 33, 64, 33000, 4, 512, 0, False),    # several parts per row, groups of 8 keys, ragged end
    (1, 1, 64, 128, 70001, 4, 512, 0, False),   # groups of 32 keys
    (1, 1, 17, 64, 70001, 4, 512, 0, True),     # ties: the parts' list overflows
    (5, 3, 64, 128, 97, 4, 64, 0, False),       # a query group with an idle wave
    (1, 7, 64, 128, 300, 1, 64, 1, False),      # causal: rows without keys, most rows shorter than T
    (1, 8, 64, 128, 20000, 4, 1000, 0, False),  # shared keys, several parts per row
    (2, 9, 48, 128, 1029, 4, 100, 0, True),
    (1, 2048, 8, 32, 1500, 1, 1100, 1, False),  # causal, one piece
    (1, 1300, 8, 32, 1300, 1, 1025, 1, False),  # causal, key range in pieces: some that a row does not reach
    (2, 2100, 48, 64, 9001, 1, 200, 1, True),   # causal, rows of up to 2100 keys against a longer cache
    (1, 1, 64, 128, 70000, 4, 4096, 0, False),  # the longest list, several parts
    (1, 4200, 8, 32, 1100, 4, 2048, 1, False),  # more rows than the chip has waves
])
def test_dense_schedule_is_bit_identical(B, S, H, D, T, m, k, mask, ties):
    print(f"dense B={B} S={S} H={H} D={D} T={T} m={m} k={k} mask={mask} ties={ties}", flush=True)
    q, K, w = _problem(S + T, B, S, H, D, T, ties)
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    ws = torch.full((max(B * S * T * 4 + (64 << 20), P.si_workspace_bytes(B, S, H, D, T, k, S, 1000)),), 77,
                    dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, mask, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == 1 and prof["finalize"][1] == 1 and prof["compact"][1] == 0
    assert prof["fused"][1] == 0 and prof["fused_narrow"][1] == 0
    if k <= 2048:
        P.si_indexer_topk_fused(q, K, w, m, k, mask, 0, *out[1], ws)
    else:
        P.si_indexer_topk_tiled(q, K, w, m, k, mask, S, min(T, 1000), *out[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))


@pytest.mark.parametrize("B,S,H,D,T,m,k", [
    (1, 4100, 8, 64, 40000, 4, 1025),    # a cache far beyond the last position: rows of 1025 keys
    (2, 1100, 64, 128, 65536, 1, 1090),  # two batches, key range in pieces
    (3, 2, 64, 128, 9000, 4, 5),         # no legal key at all
    (1, 7, 33, 64, 50000, 1, 12),        # one wave per query
])
def test_dense_rows_are_as_long_as_the_longest_legal_row(B, S, H, D, T, m, k):
    """Causal, with a cache longer than S / m: a workspace for B * S rows of S / m scores (and the smallest tile plan)
    is enough for the dense schedule."""
    print(f"dense, long cache B={B} S={S} H={H} D={D} T={T} m={m} k={k}", flush=True)
    q, K, w = _problem(T, B, S, H, D, T, False)
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    size = max(B * S * max(1, S // m) * 4, P.si_workspace_bytes(B, S, H, D, T, k, min(S, 8), 32))
    assert size < B * S * T * 4
    ws = torch.full((size,), 77, dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, 1, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == 1 and prof["finalize"][1] == 1 and prof["compact"][1] == 0
    assert prof["fused"][1] == 0 and prof["fused_narrow"][1] == 0
    big = torch.empty(P.si_fused_workspace_bytes(B, S, H, D, T, k), dtype=torch.uint8, device=DEV)
    P.si_indexer_topk_fused(q, K, w, m, k, 1, 0, *out[1], big)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))


@pytest.mark.parametrize("B,S,H,D,T,m,k,mask,dense", [
    (1, 5000, 8, 32, 5000, 1, 256, 1, True),    # up to 8192 keys per query
    (1, 5000, 7, 32, 5000, 1, 256, 1, False),   # few heads, causal: up to 4096
    (1, 2100, 7, 32, 5000, 1, 256, 0, True),
    (1, 2100, 1, 32, 5000, 1, 256, 0, False),   # one head: also without a mask
    (1, 2100, 1, 128, 4096, 1, 64, 0, True),
    (1, 2100, 64, 64, 5000, 1, 255, 0, False),  # short lists: up to 4096
    (1, 2100, 1, 64, 8000, 1, 1025, 0, True),   # lists beyond the single pass's write-out by bins: up to 8192
    (1, 1544, 2, 32, 65536, 1, 1025, 0, True),   # few rows: up to 2048
    (1, 1544, 2, 32, 65537, 1, 1025, 0, False),  # long lists of more than 65536 keys: up to 1536
    (1, 1536, 2, 32, 65537, 1, 1025, 0, True),
    (1, 1544, 2, 32, 65537, 1, 1024, 0, True),
    (1, 1408, 2, 32, 98305, 1, 1024, 0, True),   # shorter lists: beyond 98304 keys up to 1408
    (1, 1416, 2, 32, 98305, 1, 1024, 0, False),
    (1, 1416, 2, 32, 98304, 1, 1024, 0, True),
    (129, 9, 2, 32, 4097, 4, 300, 0, False),     # 258 groups of eight, 387 of four
    (128, 9, 2, 32, 4097, 4, 300, 0, True),
    (129, 9, 2, 32, 4097, 4, 1025, 0, True),     # long lists
    (171, 12, 2, 32, 4097, 4, 300, 0, True),     # 513 groups of four
    (129, 9, 2, 32, 16385, 4, 300, 0, True),
    (255, 4, 2, 64, 9000, 4, 20, 0, True),       # fewer than 8 queries a batch: by the time of either
    (257, 4, 2, 64, 2500, 4, 20, 0, True),
    (700, 3, 2, 32, 1500, 4, 20, 0, True),
    (240, 4, 33, 128, 7900, 4, 20, 0, False),
    (240, 4, 32, 128, 7900, 4, 20, 0, False),
    (100, 4, 32, 128, 7900, 4, 20, 0, True),
    (130, 7, 2, 128, 16385, 4, 20, 0, False),
    (64, 7, 2, 128, 16385, 4, 20, 0, True),
    (117, 7, 64, 128, 4060, 4, 1227, 0, True),   # lists that the single pass sorts by the network
])
def test_route_by_shape(B, S, H, D, T, m, k, mask, dense):
    """Which schedule a call takes where the two cross, and that both give the same bits."""
    print(f"route B={B} S={S} H={H} D={D} T={T} m={m} k={k} mask={mask}", flush=True)
    q, K, w = _problem(S + T, B, S, H, D, T, False)
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    ws = torch.empty(B * S * T * 4 + (64 << 20), dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, mask, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == int(dense) and prof["compact"][1] == 0
    assert prof["fused"][1] + prof["fused_narrow"][1] == int(not dense)
    P.si_indexer_topk_fused(q, K, w, m, k, mask, 0, *out[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))


def test_dense_schedule_in_row_tiles():
    """k beyond the single pass and a workspace for part of the rows: tiles of rows, the last one ragged."""
    B, S, H, D, T, m, k = 1, 3001, 8, 32, 3001, 1, 2500
    q, K, w = _problem(11, B, S, H, D, T, False)
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    ws = torch.empty(1100 * T * 4, dtype=torch.uint8, device=DEV)  # 1096 rows
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, m, k, 1, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == 3 and prof["finalize"][1] == 3
    big = torch.empty(P.si_workspace_bytes(B, S, H, D, T, k, S, 1024), dtype=torch.uint8, device=DEV)
    P.si_indexer_topk_tiled(q, K, w, m, k, 1, S, 1024, *out[1], big)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))


def _pattern(name, R, n):
    x = torch.randn((R, n), generator=torch.Generator().manual_seed(n + R))
    if name == "ties":
        x = (x * 2).round() * 0.5
    elif name == "equal":
        x = torch.full((R, n), 2.5)
    elif name == "ascending":
        x = torch.arange(n).float().repeat(R, 1)
    elif name == "outliers":
        x[:, ::97] *= 1e30
    elif name == "not_finite":  # -inf and NaN are never selected, +inf ties in index order
        x[:, ::5] = float("inf")
        x[:, 1::7] = -float("inf")
        x[:, 2::11] = float("nan")
    elif name == "lowest":
        x[:] = -float("inf")
        x[:, :3] = torch.tensor([1.0, torch.finfo(torch.float32).min, 0.0])[:min(3, n)]
    elif name == "denormal":
        x = x * 1e-42
    elif name == "clump":
        x[:, n // 2:n // 2 + 600] += 50
    elif name == "few_above_equals":  # the equals begin inside the best k, and a wave's, workgroup's and chunk's border is among them
        x = x.clamp(max=0.25)
        x[:, n // 3:n // 3 + 15] = torch.arange(15).float() + 1
    elif name == "many_above_equals":  # in few groups
        x = x.clamp(max=0)
        x[:, 4096:4096 + 3000] = x[:, 4096:4096 + 3000] ** 2 + 1
    elif name == "relu":  # the zeros are the worst
        x = x.clamp(min=0)
    elif name == "relu_negative":  # the zeros are the best
        x = x.clamp(max=0)
    return x


@pytest.mark.parametrize("name", ["normal", "ties", "equal", "ascending", "outliers", "not_finite", "lowest",
                                  "denormal", "clump", "relu", "relu_negative"])
@pytest.mark.parametrize("R,n,k", [(1, 1, 3), (3, 70, 64), (2, 4096, 1024), (2, 4097, 1000), (3, 8193, 2048),
                                   (2, 8200, 4096), (1, 140001, 1500)])
def test_selection_at_its_edges(oracle, name, R, n, k):
    print(f"selection {name} R={R} n={n} k={k}", flush=True)
    x = _pattern(name, R, n)
    legal = torch.tensor([n, n + 5, max(0, n - 3)][:R], dtype=torch.int32)
    for lg in (None, legal):
        idx = torch.full((R, k), -7, dtype=torch.int32, device=DEV)
        val = torch.full((R, k), 9.0, dtype=torch.float32, device=DEV)
        ws = torch.full((P.si_workspace_bytes(1, R, 1, 32, n, k, R, 8192),), 77, dtype=torch.uint8, device=DEV)
        P.si_topk_from_scores(x.to(DEV), None if lg is None else lg.to(DEV), k, 8192, idx, val, ws)
        torch.cuda.synchronize()
        for r in range(R):
            row = x[r, :n if lg is None else min(n, int(lg[r]))].double().numpy()
            place = np.flatnonzero(row > -np.inf)  # (False for NaN)
            ri, rs = oracle.sort_topk(row[place], k)
            c = min(k, len(place))
            gi, gs = idx[r].cpu().numpy(), val[r].cpu().numpy()
            assert np.array_equal(gi[:c], place[ri[:c]]) and np.all(gi[c:] == -1)
            assert np.array_equal(gs[:c], rs[:c].astype(np.float32) + 0.0) and np.all(np.isneginf(gs[c:]))


@pytest.mark.parametrize("name", ["normal", "ties", "equal", "outliers", "not_finite", "lowest", "clump", "relu",
                                  "relu_negative"])
@pytest.mark.parametrize("R,n,k", [
    (3, 300, 16), (2100, 512, 600),                        # one wave, 8 scores a lane
    (2100, 513, 512), (2100, 1024, 1024),                  # 16
    (2100, 2048, 512), (2100, 1025, 1000),                 # 32
    (2100, 4096, 1024), (2100, 2049, 17),                  # two waves
    (3, 8192, 2048), (3, 1500, 1025),                      # 512 threads, 16 scores each
    (3, 8193, 1030), (3, 16384, 4096), (3, 4000, 4096),    # 32
    (3, 16385, 4096),                                      # beyond the registers
    (1800, 5000, 512), (1800, 20000, 1025),                # many rows by the list
    (3, 140000, 2100),                                     # several parts, the longer list
])
def test_selection_from_registers_at_its_edges(oracle, name, R, n, k):
    """Every form of the selection from registers at its shortest and longest rows; rows repeat every three."""
    print(f"short selection {name} R={R} n={n} k={k}", flush=True)
    x = _pattern(name, 3, n)
    legal = torch.tensor([n, n - 1, n // 3], dtype=torch.int32)
    rep = (R + 2) // 3
    idx = torch.full((R, k), -7, dtype=torch.int32, device=DEV)
    val = torch.full((R, k), 9.0, dtype=torch.float32, device=DEV)
    ws = torch.full((P.si_workspace_bytes(1, R, 1, 32, n, k, R, 1024),), 77, dtype=torch.uint8, device=DEV)
    P.si_topk_from_scores(x.repeat(rep, 1)[:R].to(DEV), legal.repeat(rep)[:R].to(DEV), k, 1024, idx, val, ws)
    torch.cuda.synchronize()
    for r in range(3):
        row = x[r, :int(legal[r])].double().numpy()
        place = np.flatnonzero(row > -np.inf)
        ri, rs = oracle.sort_topk(row[place], k)
        c = min(k, len(place))
        gi, gs = idx[r].cpu().numpy(), val[r].cpu().numpy()
        assert np.array_equal(gi[:c], place[ri[:c]]) and np.all(gi[c:] == -1)
        assert np.array_equal(gs[:c], rs[:c].astype(np.float32) + 0.0) and np.all(np.isneginf(gs[c:]))
        assert bool((idx[r::3] == idx[r]).all()) and bool((val[r::3] == val[r]).all())


def _least_ms(x, k, c_T, size=None):
    R, n = x.shape
    idx = torch.empty((R, k), dtype=torch.int32, device=DEV)
    val = torch.empty((R, k), dtype=torch.float32, device=DEV)
    ws = torch.empty(size or P.si_workspace_bytes(1, R, 1, 32, n, k, R, c_T), dtype=torch.uint8, device=DEV)
    times = []
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        P.si_topk_from_scores(x, None, k, c_T, idx, val, ws)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("R,n,k", [(16384, 1024, 512), (2000, 2048, 1024), (4096, 4096, 1024), (1024, 16384, 4096)])
def test_equal_scores_do_not_multiply_the_time_of_a_selection(R, n, k):
    """Rows of which half are exactly 0 (one head, ReLU) against rows of distinct scores: measured 1.2 to 2.3 times the
    time, and 4.9 to 10 times with a list that is cut again for every few equal scores."""
    x = torch.randn((R, n), generator=torch.Generator(device=DEV).manual_seed(n), device=DEV)
    distinct, worst, best = _least_ms(x, k, 1024), _least_ms(x.clamp(min=0), k, 1024), _least_ms(x.clamp(max=0), k, 1024)
    print(f"selection R={R} n={n} k={k}: {distinct:.3f} ms, zeros last {worst:.3f}, zeros first {best:.3f}", flush=True)
    assert max(worst, best) < 4.0 * distinct


@pytest.mark.parametrize("R,n,k,c_T", [(1, 49152, 300, 700), (50, 49152, 300, 700), (16, 65536, 512, 16384), (1, 262144, 4096, 16384)])
def test_equal_scores_in_rows_of_several_workgroups(R, n, k, c_T):
    """Rows whose best are all exactly 0 overflow the list that a row's workgroups share: measured 1.4 to 2.0 times the time of
    distinct scores, and 3.8 to 5.4 times with a last workgroup that cuts its list again and again."""
    x = torch.randn((R, n), generator=torch.Generator(device=DEV).manual_seed(n), device=DEV)
    distinct, best = _least_ms(x, k, c_T), _least_ms(x.clamp(max=0), k, c_T)
    print(f"several workgroups R={R} n={n} k={k} c_T={c_T}: {distinct:.4f} ms, zeros first {best:.4f}", flush=True)
    assert best < 3.0 * distinct


def test_few_equal_scores_in_rows_of_several_workgroups():
    """Equal scores that overflow the shared list but not the one on chip: measured 3.5 to 4.4 times the time of distinct ones, 7
    with a pass that looks for equals in every chunk."""
    x = torch.randn((3, 278614), generator=torch.Generator(device=DEV).manual_seed(4), device=DEV)
    distinct, rounded = _least_ms(x, 471, 4096), _least_ms((x * 8).round() / 8, 471, 4096)
    print(f"several workgroups, rounded: {distinct:.4f} ms, rounded {rounded:.4f}", flush=True)
    assert rounded < 5.0 * distinct


def test_maxima_of_large_groups_are_shared_by_waves():
    """A workspace with room for the maxima of groups of 1024 only: measured 1.0 to 1.2 times the time of groups of 32, 3 times by
    one wave for 64 such groups."""
    x = torch.randn((14, 76484), generator=torch.Generator(device=DEV).manual_seed(5), device=DEV)
    small, ample = _least_ms(x, 36, 512), _least_ms(x, 36, 16384)
    print(f"maxima of large groups: {small:.4f} ms, of groups of 32 {ample:.4f}", flush=True)
    assert small < 1.8 * ample


@pytest.mark.parametrize("B,S,H,D,T,k,tiles", [
    (45, 1, 8, 32, 60000, 64, 2),    # one query a batch
    (70, 4, 20, 64, 30001, 100, 5),  # four
    (9, 7, 33, 64, 70001, 64, 3),    # seven, several workgroups per row
    (11, 2, 64, 128, 100003, 64, 2),
    (300, 1, 8, 32, 38062, 595, 2),  # tiles of more rows, without joint lists, have room for more batches
    (93, 7, 64, 128, 11952, 51, 0),  # many queries a batch, whose waves take the keys to each: the single pass
    (122, 7, 8, 64, 35079, 100, 0),
])
def test_dense_schedule_in_batch_tiles(B, S, H, D, T, k, tiles):
    """Few queries of many batches in the single pass's workspace, which holds the scores of some batches only."""
    print(f"batch tiles B={B} S={S} H={H} D={D} T={T} k={k}", flush=True)
    q, K, w = _problem(B + T, B, S, H, D, T, False)
    out = [(torch.full((B, S, k), -7, dtype=torch.int32, device=DEV), torch.full((B, S, k), 5.0, device=DEV))
           for _ in range(2)]
    ws = torch.full((P.si_fused_workspace_bytes(B, S, H, D, T, k),), 77, dtype=torch.uint8, device=DEV)
    assert ws.numel() < B * S * T * 4
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_indexer_topk(q, K, w, 4, k, 0, *out[0], ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["score_tile"][1] == prof["finalize"][1] == tiles
    assert prof["fused_narrow"][1] + prof["fused"][1] == int(tiles == 0)
    P.si_indexer_topk_fused(q, K, w, 4, k, 0, 0, *out[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))


@pytest.mark.parametrize("n,k,list_keys", [(1 << 20, 4096, 5300), (1 << 20, 3500, 4500)])
def test_a_joint_list_too_short_for_the_groups_a_bound_comes_from(n, k, list_keys):
    """Long lists, whose bound comes from fewer groups than there are maxima: a workspace with room for the maxima of all groups
    of 32 and for 1.3 k keys gets larger groups and a longer list instead of one that ordinary scores overflow."""
    x = torch.randn((1, n), generator=torch.Generator(device=DEV).manual_seed(n), device=DEV)
    small, ample = _least_ms(x, k, 1024, n // 32 * 4 + list_keys * 8 + 1024), _least_ms(x, k, 1024, 1 << 20)
    print(f"joint list n={n} k={k} keys={list_keys}: {small:.4f} ms, ample workspace {ample:.4f}", flush=True)
    assert small < 2.0 * ample


@pytest.mark.parametrize("R,n,k,c_T,several", [
    (64, 32768, 300, 16384, True),   # groups of 32 entries, four workgroups a row
    (64, 32767, 300, 16384, False),
    (64, 36864, 255, 16384, True),   # short lists
    (64, 36863, 255, 16384, False),
    (65, 40960, 300, 16384, True),   # three
    (65, 40959, 300, 16384, False),
    (128, 49152, 300, 16384, True),  # two
    (128, 49151, 300, 16384, False),
    (1, 46422, 375, 4096, True),     # a list of 4096 just fits
    (1, 46422, 375, 4000, False),
    (4, 49151, 20, 700, False),      # larger groups
    (4, 49152, 20, 700, True),
    (1, 32768, 513, 16384, False),   # fewer groups than 2 k
])
def test_selection_by_one_or_several_workgroups(oracle, R, n, k, c_T, several):
    print(f"one or several workgroups R={R} n={n} k={k} c_T={c_T}", flush=True)
    x = _pattern("normal", R, n)
    legal = torch.tensor([n, n - 1, n // 3, 5 * n // 7] * R, dtype=torch.int32)[:R]
    idx = torch.full((R, k), -7, dtype=torch.int32, device=DEV)
    val = torch.full((R, k), 9.0, dtype=torch.float32, device=DEV)
    ws = torch.full((P.si_workspace_bytes(1, R, 1, 32, n, k, R, c_T),), 77, dtype=torch.uint8, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_topk_from_scores(x.to(DEV), legal.to(DEV), k, c_T, idx, val, ws)
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["init"][1] == int(several) and prof["filter_scores"][1] == 1
    for r in sorted({0, R // 2, R - 1}):
        ri, rs = oracle.sort_topk(x[r, :int(legal[r])].double().numpy(), k)
        assert np.array_equal(idx[r].cpu().numpy(), ri) and np.array_equal(val[r].cpu().numpy(), rs.astype(np.float32))


@pytest.mark.parametrize("name", ["normal", "ties", "ascending", "not_finite", "lowest", "clump", "relu_negative", "equal",
                                  "few_above_equals", "many_above_equals"])
@pytest.mark.parametrize("R,n,k,c_T", [
    (3, 49152, 20, 700),      # the shortest rows of several workgroups; a list shorter than the usual one
    (3, 140001, 100, 1024),   # groups of 64 and more
    (2, 300007, 1500, 5000),  # groups of 32, a shorter list
])
def test_selection_by_several_workgroups_in_a_small_workspace(oracle, name, R, n, k, c_T):
    print(f"selection, small workspace {name} R={R} n={n} k={k} c_T={c_T}", flush=True)
    x = _pattern(name, R, n)
    legal = torch.tensor([n, n - 3, n // 3][:R], dtype=torch.int32)
    size = P.si_workspace_bytes(1, R, 1, 32, n, k, R, c_T)
    guard = torch.full((size + 4096,), 77, dtype=torch.uint8, device=DEV)
    idx = torch.full((R, k), -7, dtype=torch.int32, device=DEV)
    val = torch.full((R, k), 9.0, dtype=torch.float32, device=DEV)
    P.si_profile_reset()
    P.si_profile_enable(True)
    P.si_topk_from_scores(x.to(DEV), legal.to(DEV), k, c_T, idx, val, guard[:size])
    prof = P.si_profile_read()
    P.si_profile_enable(False)
    assert prof["init"][1] == 1  # the maxima: by several workgroups
    assert bool((guard[size:] == 77).all())
    for r in range(R):
        row = x[r, :int(legal[r])].double().numpy()
        place = np.flatnonzero(row > -np.inf)
        ri, rs = oracle.sort_topk(row[place], k)
        c = min(k, len(place))
        gi, gs = idx[r].cpu().numpy(), val[r].cpu().numpy()
        assert np.array_equal(gi[:c], place[ri[:c]]) and np.all(gi[c:] == -1)
        assert np.array_equal(gs[:c], rs[:c].astype(np.float32) + 0.0) and np.all(np.isneginf(gs[c:]))
