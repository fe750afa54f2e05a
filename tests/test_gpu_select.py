"""Token selection at the sizes where its kernels change course (paper Section 3, "KV Pruning"):
prefixes around the pooling tiles of 4096 candidates (one kernel up to three of them, a pooling kernel of several
workgroups before it beyond), around the groups of eight candidates whose codes share 16 bytes, pooling
windows up to the widest, cuts in the lowest score bin, and candidates around the cut that do not
fit the list in LDS.  Indices against the checker, which scores in binary64."""
import numpy as np
import pytest
import torch

from paper_2412_12706_amd import kvqp, synth
from tests.gpu_util import dev
from tests.test_gpu_compress import check_indices

pytestmark = pytest.mark.gpu


def select(orc, P, W, pool, budget, Gq=2, Hkv=2, sm_scale=None, outlier=10.0, keys=None, seed=60):
    L, Hq = P + W, Hkv * Gq
    q_obs, k, v = synth.prompt_host(1, Hq, Hkv, L, W, 128, outlier=outlier, config=seed)
    if keys is not None:
        keys(k)
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hq, n_kv_heads=Hkv, seq_len=L, window=W, pool_kernel=pool, budget=budget, bits=16,
                   sm_scale=sm_scale or 128 ** -0.5)
    _, idx, pooled = orc.compress(q_obs, k, v, window=W, pool=pool, budget=budget, bits=16, G=32, sm_scale=float(np.float32(cfg.sm_scale)))
    gc = kvqp.alloc_cache(cfg)
    got = torch.full((1, Hkv, cfg.n_kept), -1, dtype=torch.int32, device="cuda")
    unrefined = torch.full((Hkv,), -1, dtype=torch.int32, device="cuda")
    kvqp.compress(cfg, dev(q_obs), dev(k), dev(v), gc, idx_out=got, unrefined_out=unrefined)
    torch.cuda.synchronize()
    return got.cpu().numpy(), idx, pooled, unrefined.cpu().tolist()


def check_heads(got, idx, pooled, unrefined):
    """Every head by itself: the checker's survivors where the cut was refined in binary64; where binary32 decided, nothing but the
    order within 2e-5 of the cut is open (the band of scores that its rounding, a few 1e-7, could move, with room to spare)."""
    for g, loose in enumerate(unrefined):
        if not loose:
            check_indices(got[:, g:g + 1], idx[:, g:g + 1], pooled[:, g:g + 1])
            continue
        own, scores = got[0, g], pooled[0, g]
        assert np.all(np.diff(own) > 0) and own[0] >= 0 and own[-1] < scores.size
        cut = np.sort(scores)[-own.size]
        kept = np.zeros(scores.size, bool)
        kept[own] = True
        assert kept[scores > cut * (1 + 2e-5)].all() and not kept[scores < cut * (1 - 2e-5)].any(), g


def row_statistics(cfg, ws, rows_pad):
    """(m, 1/Z) and the binary64 Z of every window row, out of a workspace of the stated size: they lie before the votes, the
    pooled scores' codes (beyond three pooling tiles), the survivors (each padded to 256 bytes) and room for all pooled scores (the same)."""
    heads, P, rows = cfg.batch * cfg.n_kv_heads, cfg.seq_len - cfg.window, cfg.n_q_heads // cfg.n_kv_heads * cfg.window

    def padded(n):
        return -(-n // 256) * 256
    eighths = -(-P // 8) if P > 12288 else 0
    at = kvqp.workspace_bytes(cfg)[0] - heads * eighths * 32 - sum(padded(heads * n) for n in (cfg.n_kept * 4, eighths * 16, P * 4, rows_pad * 16))
    host = ws.cpu().numpy()
    stats = host[at:at + heads * rows_pad * 8].view(np.float32).reshape(heads, rows_pad, 2)[:, :rows]
    zsum = host[at + heads * rows_pad * 8:at + heads * rows_pad * 16].view(np.float64).reshape(heads, rows_pad)[:, :rows]
    return stats.astype(np.float64), zsum


@pytest.mark.parametrize("P,pool,budget", [
    (2, 1, 1), (7, 3, 3), (9, 7, 8), (64, 63, 10), (1025, 5, 1024), (4095, 7, 1000), (4096, 63, 4095), (4096, 1, 1),
    (4097, 7, 1), (4104, 1, 4103), (8191, 13, 2000), (8193, 63, 513), (12289, 3, 6000), (40001, 7, 9001)])
def test_survivors_match_the_checker(orc, P, pool, budget):
    print(f"case P={P} pool={pool} budget={budget}", flush=True)
    got, idx, pooled, unrefined = select(orc, P, 8, pool, budget, seed=60 + P % 7)
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("P,pool,budget", [(4097, 63, 4096), (8192, 7, 3000), (8193, 1, 8192), (9001, 5, 1), (12288, 63, 2500), (12289, 7, 12288)])
def test_prefixes_of_two_and_three_pooling_tiles(orc, P, pool, budget):
    """Up to three tiles the selection pools and counts by itself, beyond them a kernel before it does: both sides of
    each line, windows that reach into the next tile, cuts at either end."""
    print(f"case tiles P={P} pool={pool} budget={budget}", flush=True)
    got, idx, pooled, unrefined = select(orc, P, 8, pool, budget, seed=90 + P % 5)
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("P,budget", [(3000, 2850), (9000, 8700)])
def test_cut_in_the_lowest_score_bin(orc, P, budget):
    """A single sharp row spreads its votes over ninety factors of two: the cut lies below 2^-55, where
    all scores share one bin, and the list of candidates around it is long."""
    print(f"case low cut P={P} budget={budget}", flush=True)
    got, idx, pooled, unrefined = select(orc, P, 1, 1, budget, Gq=1, sm_scale=0.7, outlier=1.0, seed=71)
    assert all(np.sort(pooled[0, g])[-budget] < 2.0 ** -55 for g in range(2))
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("P,budget,distinct", [(6000, 1500, 1), (9000, 4000, 2), (4090, 100, 1)])
def test_more_ties_than_the_list_holds(orc, P, budget, distinct):
    """Prefixes of one or two distinct key rows: thousands of scores tie at the cut exactly, more than
    the list in LDS and the binary64 re-scoring hold; the lowest positions win and the call says how
    many candidates binary32 decided."""
    print(f"case ties P={P} budget={budget} distinct={distinct}", flush=True)

    def keys(k):
        for d in range(distinct):
            k[:, :, d:P:distinct] = k[:, :, d:d + 1]
    got, idx, _, unrefined = select(orc, P, 8, 1, budget, keys=keys, seed=73)
    assert np.array_equal(got, idx)
    assert unrefined == [-(-P // distinct)] * 2


def test_clustered_scores_beyond_the_list_are_still_refined(orc):
    """Six thousand scores within one percent of the cut but few within the band that binary32 could
    misplace: the candidates do not fit the list, and the cut is binary64's all the same."""
    P = 6500

    def keys(k):
        base = k[:, :, :1].astype(np.float32)
        k[:, :, :P] = (base + 0.005 * k[:, :, :P].astype(np.float32)).astype(np.float16)
    print("case clustered", flush=True)
    got, idx, pooled, unrefined = select(orc, P, 8, 1, 3000, outlier=1.0, keys=keys, seed=75)
    for g in range(2):
        kth = np.sort(pooled[0, g])[-3000]
        assert (np.abs(pooled[0, g] / kth - 1) < 0.004).sum() > 3840
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("P,pool,budget", [(4096, 1, 1500), (4000, 63, 900), (12288, 5, 7000), (13001, 1, 4001), (30011, 31, 9000)])
@pytest.mark.parametrize("noise", [1.0, 0.2, 0.05, 0.02])
def test_lists_around_the_cut_of_any_length(orc, P, pool, budget, noise):
    """From a dozen candidates around the cut to more than the list holds: up to 64 that one wave finishes, more that a radix pass
    thins out first, and more than 64 left by it (plateaus of a wide pooling window, scores that cluster)."""
    print(f"case list P={P} pool={pool} budget={budget} noise={noise}", flush=True)

    def keys(k):
        base = k[:, :, :1].astype(np.float32)
        k[:, :, :P] = (base + noise * k[:, :, :P].astype(np.float32)).astype(np.float16)
    got, idx, pooled, unrefined = select(orc, P, 8, pool, budget, outlier=1.0, keys=keys, seed=101)
    kth = [np.sort(pooled[0, g])[-budget] for g in range(2)]
    print("around", [int((np.abs(pooled[0, g] / kth[g] - 1) < 0.008).sum()) for g in range(2)], "unrefined", unrefined, flush=True)
    for g in range(2):
        in_band = int((np.abs(pooled[0, g] / kth[g] - 1) <= 1.9e-5).sum())
        assert unrefined[g] == 0 or in_band > 256, (unrefined, in_band)
    check_heads(got, idx, pooled, unrefined)


@pytest.mark.parametrize("Gq,W", [(4, 64), (8, 17), (4, 32), (1, 5)])
def test_scores_that_leave_the_first_keys_far_behind(orc, Gq, W):
    """Keys that grow fourteenfold halfway through the prompt: row maxima of later workgroups pass those of
    earlier ones by more than 2^60, and the statistics of the latter vanish in the merge."""
    P = 4500
    print(f"case growing keys Gq={Gq} W={W}", flush=True)

    def keys(k):
        k[:, :, P // 2:P] = (k[:, :, P // 2:P].astype(np.float32) * 14).astype(np.float16)
    got, idx, pooled, unrefined = select(orc, P, W, 7, 300, Gq=Gq, Hkv=2, outlier=1.0, keys=keys, seed=77)
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("P,Gq,W", [(1, 8, 32), (63, 4, 64), (191, 8, 17), (257, 8, 31), (4097, 4, 33)])
def test_wide_windows_at_the_edges_of_a_step(orc, P, Gq, W):
    """More than 128 window rows: key counts around the 64 keys of a wave's step, row counts that do not
    fill a tile of 16."""
    print(f"case wide P={P} Gq={Gq} W={W}", flush=True)
    got, idx, pooled, unrefined = select(orc, P, W, 5, max(1, P // 3), Gq=Gq, seed=79)
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("L,Gq,W", [(9, 1, 5), (64, 2, 17), (65, 4, 8), (127, 8, 16), (129, 4, 31), (193, 2, 64), (4159, 4, 16), (4161, 4, 32), (20011, 1, 33)])
def test_scores_at_the_edges_of_a_chunk(orc, L, Gq, W):
    """Up to 128 window rows: key counts around the chunks of 64 that take turns in LDS (one, two and more of them
    per workgroup), row counts that do not fill the one, two or four slabs of 32 rows."""
    print(f"case chunks L={L} Gq={Gq} W={W}", flush=True)
    P = L - W
    got, idx, pooled, unrefined = select(orc, P, W, 3, max(1, P // 4), Gq=Gq, seed=83)
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


FEW_PARTS = [(L, parts) for L, parts in ((128, 1), (129, 2), (1024, 8), (1025, 9), (2048, 16), (2049, 17), (3000, 24), (3969, 32), (4096, 32), (4097, 33))]


@pytest.mark.parametrize("Hkv,Gq,W,L,parts", [(64, 4, 32, 1030, 6), (16, 4, 31, 2100, 17), (2, 4, 32, 4290, 34), (3, 2, 30, 2111, 17), (3, 1, 20, 517, 5),
                                              (3, 1, 20, 600, 5)] + [(2, *rows, *p) for rows in ((1, 20), (4, 16), (4, 32)) for p in FEW_PARTS])
def test_row_statistics_merged_by_the_vote_pass(orc, Hkv, Gq, W, L, parts):
    """One, two, up to eight, nine, sixteen and more, up to 32 statistics per row, which the vote pass merges itself (the form for
    eight and the one for 32), and just more of them, which a kernel before it does, for one, two and four slabs of
    rows; keys that grow late, so that the parts differ by many factors of two.  Up to three pooling tiles the workspace has, besides votes,
    survivors and the rows' totals, the parts alone: the count is read off its size."""
    print(f"case parts Hkv={Hkv} Gq={Gq} W={W} L={L}", flush=True)
    c = kvqp.Cfg(batch=1, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=L, window=W, budget=(L - W) // 5, bits=16)
    rows_pad = 32 if Gq * W <= 32 else 64 if Gq * W <= 64 else 128
    rest = sum(-(-Hkv * n // 256) * 256 for n in (c.n_kept * 4, (L - W) * 4, rows_pad * 16))
    assert kvqp.workspace_bytes(c)[0] - rest == parts * Hkv * rows_pad * 8
    P = L - W

    def keys(k):
        k[:, :, P // 2:P] = (k[:, :, P // 2:P].astype(np.float32) * 3).astype(np.float16)
    got, idx, pooled, unrefined = select(orc, P, W, 3, P // 5, Gq=Gq, Hkv=Hkv, outlier=4.0, keys=keys, seed=95)
    check_indices(got, idx, pooled)
    assert unrefined == [0] * Hkv


@pytest.mark.parametrize("where,word", [("query", float("nan")), ("key", float("nan")), ("query", float("inf")), ("key", -float("inf"))])
@pytest.mark.parametrize("P,Gq,W,pool,budget", [(700, 2, 8, 7, 100), (4096, 4, 32, 1, 4095), (5000, 2, 8, 7, 513), (9001, 4, 64, 63, 2000)])
def test_votes_that_are_not_numbers_still_give_every_survivor(P, Gq, W, pool, budget, where, word):
    """Such inputs have no defined scores, but every head still gets its count of ascending positions
    of the prefix (the quantizer gathers at them), and the other heads are not touched.  A row of a
    head that is not finite takes all its votes away (query, NaN) or leaves them at zero: the lowest positions."""
    print(f"case {where} {word} P={P} Gq={Gq} W={W} pool={pool} budget={budget}", flush=True)
    L, Hkv = P + W, 3
    q_obs, k, v = (dev(t) for t in synth.prompt_host(1, Hkv * Gq, Hkv, L, W, 128, config=81))
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=L, window=W, pool_kernel=pool, budget=budget, bits=4, group_size=32)

    def survivors():
        got = torch.full((1, Hkv, budget), -1, dtype=torch.int32, device="cuda")
        kvqp.compress(cfg, q_obs, k, v, kvqp.alloc_cache(cfg), idx_out=got)
        torch.cuda.synchronize()
        return got.cpu()[0]
    clean = survivors()
    if where == "query":
        q_obs[0, Gq:2 * Gq, :, 5] = word
    else:
        k[0, 1, P // 3, 9] = word
    got = survivors()
    assert torch.equal(got[0], clean[0]) and torch.equal(got[2], clean[2])
    assert bool((got[1].diff() > 0).all()) and int(got[1, 0]) >= 0 and int(got[1, -1]) < P
    if word != word:
        assert torch.equal(got[1], torch.arange(budget, dtype=torch.int32))


@pytest.mark.parametrize("Gq,W", [(4, 64), (8, 24), (4, 32), (8, 8), (4, 8)])
@pytest.mark.parametrize("key", [5.0, 14.0, 24.0, 38.0])
def test_row_sums_keep_their_precision_when_a_late_key_dominates(Gq, W, key):
    """Statistics of the window rows (the divisors of every vote, in the re-scoring too) when one key, the
    last of a wave's share, beats all earlier ones by 4 to 55 factors of two.  One channel is in use, so
    the products are exact and only exponentials and sums are rounded: with arguments up to 8 (a
    reference never lags further) 2^-22 ln 2 for the rounding of the argument, 2^-23 for the exponential and 2^-24
    for each of at most eleven additions behind the large term, together 9.4e-7 of the sum.  Arguments of 32
    to 64, as a reference left at the first keys gives, are rounded to 1.3e-6 alone.  (Up to 64 rows a lane's sum and what follows
    are 64 bits wide and rounded once.)"""
    B, Hkv, P, budget = 8, 8, 4500, 100
    heads, rows = B * Hkv, Gq * W
    rows_pad = 32 if rows <= 32 else 64 if rows <= 64 else 128 if rows <= 128 else 256
    print(f"case late key {key} Gq={Gq} W={W}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q = torch.zeros(B, Hkv * Gq, W, 128, dtype=torch.float16, device="cuda")
    q[..., 0] = (0.5 + 0.5 * torch.rand(B, Hkv * Gq, W, generator=gen, device="cuda")).half()
    k = torch.zeros(B, Hkv, P + W, 128, dtype=torch.float16, device="cuda")
    k[:, :, 8 * 64 + 51, 0] = key
    cfg = kvqp.Cfg(batch=B, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=P + W, window=W, pool_kernel=1, budget=budget, bits=16, sm_scale=1.0)
    ws = kvqp.alloc_workspace(kvqp.workspace_bytes(cfg)[0])
    kvqp.compress(cfg, q, k, torch.zeros_like(k), kvqp.alloc_cache(cfg), workspace=ws)
    torch.cuda.synchronize()

    stats, zsum = row_statistics(cfg, ws, rows_pad)
    arg = q[..., 0].cpu().numpy().astype(np.float64).reshape(heads, rows) * key * np.float64(np.float32(np.log2(np.e)))
    others = P + np.arange(rows) % W                                             # visible keys of score 0
    assert np.ptp(arg) > 0.4 * key
    err = zsum / (others[None] * np.exp2(-stats[..., 0]) + np.exp2(arg - stats[..., 0])) - 1
    worst = np.abs(err).max()
    print(f"worst {worst:.2e} rms {np.sqrt((err ** 2).mean()):.2e}", flush=True)
    assert worst < 9.4e-7
    assert np.allclose(stats[..., 1] * zsum, 1, rtol=1.2e-7)


@pytest.mark.parametrize("Gq,W", [(1, 7), (4, 8), (2, 32), (4, 32)])
def test_row_sums_of_the_key_strips_are_added_in_64_bits(Gq, W):
    """A row whose sum is 1 in one strip of 16 keys of a chunk and 0.75 * 2^-24 in each of the other three: every strip's sum is exact,
    and their total reaches the workspace rounded once (2^-24).  Added one after the other in 32 bits all three would be lost,
    2.25 * 2^-24.  Products and scale are whole numbers, so no exponential is rounded.  (Up to 32 window rows there are four strips to a
    chunk, up to 64 two, beyond them one, where a lane's own sum has the same bound.)"""
    B, Hkv, P, budget = 1, 2, 3000, 100
    heads, rows = B * Hkv, Gq * W
    rows_pad = 32 if rows <= 32 else 64 if rows <= 64 else 128
    print(f"case strips Gq={Gq} W={W}", flush=True)
    scale = np.float32(np.log(2.0))
    assert np.float32(scale * np.float32(1.4426950408889634)) == 1.0
    q = torch.zeros(B, Hkv * Gq, W, 128, dtype=torch.float16, device="cuda")
    q[..., 0] = 1.0
    k = torch.zeros(B, Hkv, P + W, 128, dtype=torch.float16, device="cuda")
    k[..., 0] = -2000.0
    at = 10 * 64
    k[:, :, at + 5, 0] = 0.0
    for strip in (1, 2, 3):
        k[:, :, at + 16 * strip + 2, 0] = -25.0
        k[:, :, at + 16 * strip + 9, 0] = -26.0
    cfg = kvqp.Cfg(batch=B, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=P + W, window=W, pool_kernel=1, budget=budget, bits=16, sm_scale=float(scale))
    ws = kvqp.alloc_workspace(kvqp.workspace_bytes(cfg)[0])
    kvqp.compress(cfg, q, k, torch.zeros_like(k), kvqp.alloc_cache(cfg), workspace=ws)
    torch.cuda.synchronize()
    stats, zsum = row_statistics(cfg, ws, rows_pad)
    err = zsum / ((1 + 2.25 * 2.0 ** -24) * np.exp2(-stats[..., 0].astype(np.float64))) - 1
    print(f"worst {np.abs(err).max():.2e}", flush=True)
    assert np.abs(err).max() <= 2.0 ** -24 * (1 + 2.0 ** -20)


@pytest.mark.parametrize("P,pool,budget,noise", [(12301, 63, 5000, 0.0), (8192, 5, 8191, 0.0), (40003, 13, 9000, 0.0), (13001, 31, 4000, 0.003),
                                                 (20481, 1, 12000, 0.002)])
def test_more_candidates_around_the_cut_than_the_list_holds_under_wide_windows(orc, P, pool, budget, noise):
    """Prompts whose keys are alike (or nearly): the candidates around the cut are visited in the threads' own scores (up to
    three tiles) or by pooling the prefix once more, tile by tile, and their windows reach across the tiles' edges."""
    print(f"case alike P={P} pool={pool} budget={budget} noise={noise}", flush=True)

    def keys(k):
        base = k[:, :, :1].astype(np.float32)
        k[:, :, :P] = (base + noise * k[:, :, :P].astype(np.float32)).astype(np.float16)
    got, idx, pooled, unrefined = select(orc, P, 8, pool, budget, outlier=1.0, keys=keys, seed=83)
    if noise == 0.0:
        assert np.array_equal(got[0], np.tile(np.arange(budget), (2, 1))) and unrefined == [P, P]
    else:
        for g in range(2):
            kth = np.sort(pooled[0, g])[-budget]
            assert (np.abs(pooled[0, g] / kth - 1) < 0.004).sum() > 3840
            assert unrefined[g] == 0 or unrefined[g] > 512
        check_heads(got, idx, pooled, unrefined)


@pytest.mark.parametrize("P,pool,budget", [(12289, 5, 3000), (13003, 5, 5000), (40003, 13, 9000)])
def test_a_compress_workspace_without_room_for_all_pooled_scores_gives_the_same_survivors(P, pool, budget):
    """Beyond three pooling tiles the stated size has four bytes per candidate for prompts whose scores cluster around the cut (more
    candidates there than the list holds); a workspace that holds everything else is taken, and a smaller one is not."""
    print(f"case smaller compress workspace P={P}", flush=True)
    W, Hkv = 8, 2
    q_obs, k, v = (dev(t) for t in synth.prompt_host(1, Hkv * 2, Hkv, P + W, W, 128, outlier=1.0, config=85))
    k[:, :, :P] = (k[:, :, :1].float() + 0.002 * k[:, :, :P].float()).half()
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * 2, n_kv_heads=Hkv, seq_len=P + W, window=W, pool_kernel=pool, budget=budget, bits=4, group_size=32)
    stated = kvqp.workspace_bytes(cfg)[0]
    least = stated - Hkv * -(-P // 8) * 32
    got = []
    for size in (stated, least):
        idx = torch.full((1, Hkv, budget), -1, dtype=torch.int32, device="cuda")
        kvqp.compress(cfg, q_obs, k, v, kvqp.alloc_cache(cfg), idx_out=idx, workspace=kvqp.alloc_workspace(stated)[:size])
        torch.cuda.synchronize()
        got.append(idx)
    assert torch.equal(got[0], got[1]) and bool((got[0].diff() > 0).all())
    with pytest.raises(kvqp.KvqpError):
        kvqp.compress(cfg, q_obs, k, v, kvqp.alloc_cache(cfg), workspace=kvqp.alloc_workspace(stated)[:least - 16])


@pytest.mark.parametrize("where", ["workspace", "query"])
def test_a_survivor_list_over_memory_that_dies_during_the_call(where):
    """The selection writes the caller's list itself; a list laid over the workspace or the queries, which are read
    until the list is complete, still comes out as one in memory of its own, and so does the cache."""
    print(f"case list over {where}", flush=True)
    P, W, Hkv, Gq, budget = 5000, 16, 2, 4, 700
    q_obs, k, v = (dev(t) for t in synth.prompt_host(1, Hkv * Gq, Hkv, P + W, W, 128, config=87))
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=P + W, window=W, budget=budget, bits=4, group_size=32)
    ws = kvqp.alloc_workspace(kvqp.workspace_bytes(cfg)[0])
    want = torch.empty((1, Hkv, budget), dtype=torch.int32, device="cuda")
    ca, cb = kvqp.alloc_cache(cfg), kvqp.alloc_cache(cfg)
    kvqp.compress(cfg, q_obs, k, v, ca, idx_out=want, workspace=ws)
    over = ws if where == "workspace" else q_obs.view(torch.uint8).view(-1)
    got = over[:4 * Hkv * budget].view(torch.int32).view(1, Hkv, budget)
    kvqp.compress(cfg, q_obs, k, v, cb, idx_out=got, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert all(torch.equal(ca.buffers[n], cb.buffers[n]) for n in ca.buffers)


def test_unusual_cuts_beyond_three_tiles(orc):
    """The lowest score bin, ties beyond the list and votes that are not numbers, where codes and counts pass through memory."""
    test_cut_in_the_lowest_score_bin(orc, 13500, 13100)
    test_more_ties_than_the_list_holds(orc, 14000, 4000, 2)
    test_votes_that_are_not_numbers_still_give_every_survivor(13001, 4, 32, 7, 4000, "query", float("nan"))


@pytest.mark.parametrize("over", ["k_codes", "v_scale", "tail_k"])
def test_a_survivor_list_over_a_buffer_of_the_cache(over):
    """The caller's list is written and never read: laid over a buffer of the cache it is lost, the cache is not."""
    print(f"case list over {over}", flush=True)
    P, W, Hkv, Gq, budget = 5000, 16, 2, 4, 700
    q_obs, k, v = (dev(t) for t in synth.prompt_host(1, Hkv * Gq, Hkv, P + W, W, 128, config=87))
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=P + W, window=W, budget=budget, bits=4, group_size=32)
    ca, cb = kvqp.alloc_cache(cfg), kvqp.alloc_cache(cfg)
    for c in (ca, cb):
        for t in c.buffers.values():
            t.fill_(0xA5)
    kvqp.compress(cfg, q_obs, k, v, ca)
    kvqp.compress(cfg, q_obs, k, v, cb, idx_out=cb.buffers[over][:4 * Hkv * budget].view(torch.int32).view(1, Hkv, budget))
    torch.cuda.synchronize()
    assert all(torch.equal(ca.buffers[n], cb.buffers[n]) for n in ca.buffers)


def test_calls_on_two_streams_may_share_a_survivor_list_that_nobody_reads():
    """Prompts of two lengths, each with its own cache and workspace, one list for both."""
    print("case one list for two streams", flush=True)
    W, Hkv, budget = 16, 2, 120
    waste = torch.empty((1, Hkv, budget), dtype=torch.int32, device="cuda")
    calls = []
    for L in (9000, 200):
        t = [dev(x) for x in synth.prompt_host(1, Hkv * 2, Hkv, L, W, 128, config=L)]
        cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * 2, n_kv_heads=Hkv, seq_len=L, window=W, budget=budget, bits=4, group_size=32)
        want, got = kvqp.alloc_cache(cfg), kvqp.alloc_cache(cfg)
        kvqp.compress(cfg, *t, want)
        calls.append((cfg, t, want, got, kvqp.alloc_workspace(kvqp.workspace_bytes(cfg)[0]), torch.cuda.Stream()))
    torch.cuda.synchronize()
    for _ in range(20):
        for cfg, t, _, got, ws, stream in calls:
            kvqp.compress(cfg, *t, got, idx_out=waste, workspace=ws, stream=stream)
    torch.cuda.synchronize()
    for cfg, _, want, got, _, _ in calls:
        assert all(torch.equal(want.buffers[n], got.buffers[n]) for n in want.buffers)


@pytest.mark.parametrize("Gq,W,L", [(1, 9, 700), (4, 8, 4133), (8, 8, 3001), (4, 32, 2065), (4, 64, 1500), (4, 30, 13000)])
@pytest.mark.parametrize("shift", [1, 4])
def test_prompts_at_any_address(Gq, W, L, shift):
    """Queries, keys and values that begin at the address of any binary16 number (2 and 8 bytes past a multiple of 16 here): the same
    survivors and the same cache as from aligned copies, for one, two and four slabs of window rows and for more."""
    print(f"case address Gq={Gq} W={W} L={L} shift={shift}", flush=True)
    Hkv, budget = 2, L // 5
    t = [dev(x) for x in synth.prompt_host(1, Hkv * Gq, Hkv, L, W, 128, config=96)]
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=L, window=W, budget=budget, bits=4, group_size=32, outlier_threshold=6.0,
                   outlier_overflow_cap=budget)
    got = []
    for s in (0, shift):
        moved = []
        for x in t:
            room = torch.zeros(x.numel() + 8, dtype=x.dtype, device="cuda")
            moved.append(room[s:s + x.numel()].view(x.shape))
            moved[-1].copy_(x)
            assert moved[-1].data_ptr() % 16 == 2 * s
        idx = torch.full((1, Hkv, budget), -1, dtype=torch.int32, device="cuda")
        cache = kvqp.alloc_cache(cfg)
        for b in cache.buffers.values():
            b.fill_(0xA5)
        kvqp.compress(cfg, *moved, cache, idx_out=idx)
        torch.cuda.synchronize()
        got.append((idx, cache))
    assert torch.equal(got[0][0], got[1][0])
    assert all(torch.equal(got[0][1].buffers[n], got[1][1].buffers[n]) for n in got[0][1].buffers)


@pytest.mark.parametrize("P,pool,budget", [(32768, 7, 9000), (32769, 7, 9000), (32777, 1, 1), (32961, 5, 4000), (40961, 63, 40960), (65543, 5, 20000), (131072, 7, 30000), (131071, 13, 1)])
def test_prefixes_whose_codes_several_workgroups_sweep(orc, P, pool, budget):
    """Beyond 32768 candidates a head's codes are swept by up to sixteen workgroups, the last of which goes on: both sides of the
    line, the shortest last share (793 groups of eight, the others have 832), sixteen full ones, cuts at either end."""
    print(f"case shares P={P} pool={pool} budget={budget}", flush=True)
    got, idx, pooled, unrefined = select(orc, P, 8, pool, budget, seed=103 + P % 5)
    check_indices(got, idx, pooled)
    assert unrefined == [0, 0]


@pytest.mark.parametrize("P,pool,budget,noise", [(33001, 1, 9000, 0.05), (50001, 7, 12000, 0.02), (40009, 1, 39000, 0.002), (45000, 5, 20000, 0.0)])
def test_long_and_overlong_lists_of_several_workgroups(orc, P, pool, budget, noise):
    print(f"case shares, list P={P} pool={pool} budget={budget} noise={noise}", flush=True)

    def keys(k):
        base = k[:, :, :1].astype(np.float32)
        k[:, :, :P] = (base + noise * k[:, :, :P].astype(np.float32)).astype(np.float16)
    got, idx, pooled, unrefined = select(orc, P, 8, pool, budget, outlier=1.0, keys=keys, seed=105)
    if noise == 0.0:
        assert np.array_equal(got[0], np.tile(np.arange(budget), (2, 1))) and unrefined == [P, P]
    else:
        assert all(n == 0 or n > 512 for n in unrefined)
        check_heads(got, idx, pooled, unrefined)


def test_counts_per_head_and_replays_where_several_workgroups_sweep():
    """Heads that keep nothing, everything or some of 40000 candidates, in one call; the same again eagerly and as replays of a
    captured call with other work on the workspace between them: what counts the workgroups' arrivals is reset by the call itself."""
    print("case shares, counts and replays", flush=True)
    P, W, Hkv = 40000, 8, 4
    q_obs, k, v = (dev(t) for t in synth.prompt_host(1, Hkv * 2, Hkv, P + W, W, 128, config=107))
    cfg = kvqp.Cfg(batch=1, n_q_heads=Hkv * 2, n_kv_heads=Hkv, seq_len=P + W, window=W, budget=P, bits=4, group_size=32)
    ws = kvqp.alloc_workspace(kvqp.workspace_bytes(cfg)[0])
    counts = [0, P, 9001, 1]

    def call(idx, un, stream=None):
        kvqp.compress_ragged(cfg, q_obs, k, v, counts, kvqp.alloc_cache(cfg, ragged=True), idx_out=idx, workspace=ws, unrefined_out=un, stream=stream)
    want, un = torch.full((1, Hkv, P), -1, dtype=torch.int32, device="cuda"), torch.full((Hkv,), -1, dtype=torch.int32, device="cuda")
    call(want, un)
    torch.cuda.synchronize()
    assert un.tolist() == [0] * Hkv
    for h, n in enumerate(counts):
        alone = kvqp.Cfg(batch=1, n_q_heads=2, n_kv_heads=1, seq_len=P + W, window=W, budget=max(n, 1), bits=4, group_size=32)
        got = torch.empty((1, 1, max(n, 1)), dtype=torch.int32, device="cuda")
        kvqp.compress(alone, q_obs[:, 2 * h:2 * h + 2].contiguous(), k[:, h:h + 1].contiguous(), v[:, h:h + 1].contiguous(), kvqp.alloc_cache(alone), idx_out=got)
        torch.cuda.synchronize()
        assert torch.equal(want[0, h, :n], got[0, 0, :n])
    idx, un2 = want.clone(), un.clone()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    cache = kvqp.alloc_cache(cfg, ragged=True)
    with torch.cuda.graph(graph, stream=side):
        kvqp.compress_ragged(cfg, q_obs, k, v, counts, cache, idx_out=idx, workspace=ws, unrefined_out=un2, stream=side)
    for _ in range(4):
        idx.fill_(-1)
        un2.fill_(-1)
        ws.fill_(0xA5)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(idx[0, h, :n], want[0, h, :n]) for h, n in enumerate(counts)) and un2.tolist() == [0] * Hkv
        again = torch.full_like(want, -1)
        call(again, un)
        torch.cuda.synchronize()
        assert torch.equal(again, want)


@pytest.mark.parametrize("Hkv,P,counts,noise", [(52, 33001, "equal", 1.0), (33, 65521, "own", 1.0), (17, 131072, "own", 1.0), (17, 131071, "equal", 0.05),
                                                (17, 131072, "equal", 0.0)])
def test_long_prefixes_of_many_heads_are_swept_by_one_workgroup_each(Hkv, P, counts, noise):
    """More heads than leave each sweeping workgroup a CU: one workgroup takes all groups of codes of a head, up to sixteen per
    thread, and lists up to 16384 of them (all keys alike).  The same survivors and the same word on what binary32 decided as from a call on
    the head alone, whose codes several workgroups sweep."""
    print(f"case one workgroup Hkv={Hkv} P={P} counts={counts} noise={noise}", flush=True)
    assert Hkv * -(-(-(-P // 8)) // 1024) > 256
    W, pool = 8, 5
    gen = torch.Generator(device="cuda").manual_seed(P + Hkv)
    q_obs = torch.randn(1, Hkv, W, 128, generator=gen, device="cuda").half()
    k = torch.randn(1, Hkv, P + W, 128, generator=gen, device="cuda", dtype=torch.float16)
    if noise < 1.0:
        k[:, :, 1:P] = (k[:, :, :1].float() + noise * k[:, :, 1:P].float()).half()
    budget = P // 6
    n = [budget] * Hkv if counts == "equal" else [(0, P, 1, budget, P - 1)[h % 5] for h in range(Hkv)]

    def call(heads, n):
        rows = slice(heads[0], heads[-1] + 1)
        cfg = kvqp.Cfg(batch=1, n_q_heads=len(heads), n_kv_heads=len(heads), seq_len=P + W, window=W, pool_kernel=pool, budget=max(n + [1]), bits=2, group_size=128)
        idx = torch.full((1, len(heads), cfg.n_kept), -1, dtype=torch.int32, device="cuda")
        un = torch.full((len(heads),), -1, dtype=torch.int32, device="cuda")
        kk = k[:, rows].contiguous()
        if counts == "equal":
            kvqp.compress(cfg, q_obs[:, rows].contiguous(), kk, kk, kvqp.alloc_cache(cfg), idx_out=idx, unrefined_out=un)
        else:
            kvqp.compress_ragged(cfg, q_obs[:, rows].contiguous(), kk, kk, n, kvqp.alloc_cache(cfg, ragged=True), idx_out=idx, unrefined_out=un)
        torch.cuda.synchronize()
        return idx[0], un.tolist()
    sees = torch.arange(P + W, device="cuda") <= P + torch.arange(W, device="cuda")[:, None]

    def pooled(h):      # scores in 64 bits
        logit = (q_obs[0, h].double() @ k[0, h].double().T) * float(np.float32(128 ** -0.5))
        vote = torch.softmax(logit.masked_fill(~sees, -torch.inf), dim=1)[:, :P].sum(0)
        return torch.nn.functional.max_pool1d(vote[None], pool, 1, pool // 2)[0].cpu().numpy()
    got, un = call(list(range(Hkv)), n)
    assert got.shape[1] == max(n)
    for h in range(Hkv):
        want, alone = call([h], [n[h]])
        if n[h] == 0:
            assert un[h] == alone[0] == 0
            continue
        if noise == 0.0:
            assert un[h] == alone[0] == P and torch.equal(got[h], want[0]) and torch.equal(got[h], torch.arange(budget, dtype=torch.int32, device="cuda"))
            continue
        scores = pooled(h)
        best = np.sort(np.lexsort((np.arange(P), -scores))[:n[h]])
        assert un[h] == alone[0] == 0
        for list_ in (got[h, :n[h]], want[0, :n[h]]):
            check_heads(list_.cpu().numpy()[None, None], best[None, None], scores[None, None], [0])
