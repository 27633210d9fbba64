"""Prefill attention of launches with few workgroups (keys split over the wave halves of a workgroup and over workgroups
with a merge) and with many (no split; a loose length bound makes the same sequences such a launch).  Query tiles of 128 with one row, full and one over; a wave whose first key block lies wholly behind some
of its queries (cached rows that are no multiple of 32); splits beyond a short sequence's keys; empty, skipped and
single-token sequences; contiguous and block-table caches; the fused decoder.

Reference: the oracle's functions on the rows the caches hold.  Bounds: the bf16 tolerances of the parity gate, the
max-abs one scaled by the largest reference value."""
import numpy as np
import pytest
import torch

import gpu_util as U
from oracle import gta_oracle as orc
from paper_2506_17286_amd import binding as B, workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {"1b": W.WORKLOADS[1], "paper": W.PAPER_WORKLOADS[0],
          "mid": W.scaled(W.WORKLOADS[1], n_heads=4, n_qgroups=2, n_kgroups=1, latent_dim=128),
          "slim": W.scaled(W.PAPER_WORKLOADS[0], n_heads=8, n_qgroups=8, n_kgroups=2, n_cgroups=2, latent_dim=64)}

WIDE = W.WORKLOADS[4]

def _setup(shape, tokens):
    wl = W.scaled(SHAPES.get(shape, WIDE), d_model=128, seed=7300)
    if shape in ("paper", "slim"):
        wl = W.scaled(wl, d_model=256)
    rng = W.make_rng(wl)
    # scores of a few nats, so that the softmax is neither flat nor one-hot
    w = W.draw_weights(wl, rng, std=wl.d_model ** -0.5)
    return wl, w, W.draw_hidden(wl, rng, tokens), rng


def _check(wl, w, x, k, c, prefix, out, what):
    """out rows of one sequence against the oracle on its first `prefix` cached rows and its own new rows"""
    cfg, ow = U.oracle_config(wl), U.oracle_weights(w)
    n = len(x)
    pos = np.arange(prefix, prefix + n)
    Q, K, C, G = orc.project_tokens(cfg, ow, x, pos)
    K = np.concatenate([k[:prefix].reshape(prefix, wl.n_kgroups, wl.head_dim), K])
    C = np.concatenate([c[:prefix].reshape(prefix, wl.n_cgroups, wl.latent_dim), C])
    L = np.empty((n, wl.n_qgroups, wl.latent_dim))
    for g in range(wl.n_qgroups):
        L[:, g] = orc.attention_map_rows(cfg, Q[:, g], pos, K[:, cfg.k_of_group(g)]) @ C[:, cfg.c_of_group(g)]
    ref = orc.decode_heads(cfg, ow, L, G)
    U.assert_close(out, ref, "bf16", what, max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("bound", [257, 70000])
@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("lens", [[129], [128], [1, 300, 31], [257, 0, 160], [2048]], ids=str)
def test_fresh(shape, lens, bound):
    wl, w, x, _ = _setup(shape, sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "bf16"), x, cu, max_seqlen=max(max(lens), bound)))
    none = np.zeros((0, 1))
    for b in range(len(lens)):
        if lens[b]:
            _check(wl, w, x[cu[b]:cu[b + 1]], none, none, 0, out[cu[b]:cu[b + 1]], f"{shape} {lens} sequence {b}")


@pytest.mark.parametrize("lens", [[1000, 300, 129, 1, 700, 640, 900], [1030] * 6], ids=["ragged", "alike"])
def test_paired_workgroups(lens):
    """257 to 512 workgroups of four waves: those behind the first 256 go backwards.  All (level, sequence) pairs on the chip at once:
    short ragged prompts (448 workgroups), and prompts of one length, which stay with four waves beyond 1024 keys (432)."""
    wl, w, x, _ = _setup("1b", sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "bf16"), x, cu))
    none = np.zeros((0, 1))
    for b in range(len(lens)) if len(set(lens)) > 1 else (0, 3):
        _check(wl, w, x[cu[b]:cu[b + 1]], none, none, 0, out[cu[b]:cu[b + 1]], f"{lens} sequence {b}")
    if len(set(lens)) == 1:   # every row is written
        assert (np.abs(out).max(axis=1) > 0).all()


@pytest.mark.parametrize("chunk", [False, True])
@pytest.mark.parametrize("lens", [[1000, 129, 300, 1, 640, 0, 257, 128, 400, 145], [1000, 900, 1, 640, 1000, 128, 897, 600, 1000, 774]],
                         ids=["in turn", "dealt"])
def test_paired_workgroups_of_ranked_tiles(lens, chunk):
    """More pairs than the chip holds (640 workgroups), so that tiles are ranked, and a bound of 33 tiles (264 workgroups, to the XCDs
    in turn) and of 64 (512, eight tiles at a time), more than there are tiles; chunks with the workgroups that set the lengths behind
    them."""
    wl, w, x, r2 = _setup("1b", sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    prefix, cap = [0, 40, 500, 300, 127, 9, 128, 0, 33, 470] if chunk else [0] * 10, 1408
    k, c = W.draw_cache(wl, r2, 10, cap)
    cache = U.DeviceCache(wl, 10, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    run = U.run_prefill_chunk if chunk else U.run_prefill
    out = U.f64(run(wl, U.upload_weights(w, "bf16"), x, cu, cache=cache))
    assert cache.seq_lens.tolist() == [p + n for p, n in zip(prefix, lens)]
    for b in range(10):
        if lens[b]:
            _check(wl, w, x[cu[b]:cu[b + 1]], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[cu[b]:cu[b + 1]],
                   f"sequence {b}: {lens[b]} behind {prefix[b]}")


@pytest.mark.parametrize("chunk", [False, True])
@pytest.mark.parametrize("batch", [3, 63, 64, 65, 130])
@pytest.mark.parametrize("shape", ["1b", "paper"])
def test_every_tile_is_found(shape, batch, chunk):
    """The kernels number the query tiles of ragged sequences themselves, 64 sequences at a time: one tile more or less,
    empty sequences, levels that only a few or only late sequences reach, cached rows that lift a sequence's tiles."""
    rng = np.random.default_rng(batch)
    lens = [int(n) for n in rng.choice([0, 1, 2, 40, 127, 128, 129, 200], batch)]
    lens[-1], lens[batch // 2] = 390, 257
    prefix = [int(n) for n in rng.choice([0, 1, 127, 128, 500], batch)] if chunk else [0] * batch
    cap = 896
    wl, w, x, r2 = _setup(shape, sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    k, c = W.draw_cache(wl, r2, batch, cap)
    cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    if chunk:
        cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
        out = U.f64(U.run_prefill_chunk(wl, U.upload_weights(w, "bf16"), x, cu, cache))
    else:
        out = U.f64(U.run_prefill(wl, U.upload_weights(w, "bf16"), x, cu, cache=cache))
    for b in range(batch):
        if lens[b]:
            _check(wl, w, x[cu[b]:cu[b + 1]], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[cu[b]:cu[b + 1]],
                   f"{shape} sequence {b}: {lens[b]} behind {prefix[b]}")


@pytest.mark.parametrize("chunk", [False, True])
@pytest.mark.parametrize("lengths", ["ragged", "alike", "one_tile", "two_tiles", "equal", "no_offsets", "loose_bound"])
@pytest.mark.parametrize("shape,batch", [("1b", 65), ("paper", 256), ("paper", 257), ("1b", 1000), ("paper", 4097)])
def test_tiles_of_many_sequences(shape, batch, lengths, chunk):
    """More sequences than a wave has lanes: ranked four to a lane (to 256), two and three rounds of the search for a tile's
    sequence, or an id for every (level, sequence).  Every row is written; some sequences are compared with the oracle."""
    rng = np.random.default_rng(batch)
    some = lambda *choices: [int(n) for n in rng.choice(choices, batch)]
    lens = {"ragged": some(0, 1, 2, 17, 40, 127, 128, 129), "alike": some(130, 140, 150), "one_tile": some(0, 1, 33, 127, 128), "two_tiles": some(0, 1, 100, 129, 200),
            "loose_bound": some(0, 1, 2, 17, 40, 127, 128, 129)}.get(lengths, [129] * batch)
    if lengths == "ragged":
        lens[-1], lens[batch // 2] = 390, 257
    prefix, cap = some(0, 1, 127, 128, 200) if chunk else [0] * batch, 592
    wl, w, x, r2 = _setup(shape, sum(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wdev, bound = U.upload_weights(w, "bf16"), 500 if lengths == "loose_bound" else max(lens)
    gen = torch.Generator(device="cuda").manual_seed(3)
    k, c = (torch.randn((batch, cap, width), device="cuda", generator=gen, dtype=torch.bfloat16) for width in wl.kv_width)
    cache = U.DeviceCache(wl, batch, cap, k.clone(), c.clone())
    offsets = None if lengths == "no_offsets" else cu
    if chunk:
        cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
        out = U.run_prefill_chunk(wl, wdev, x, offsets, cache, max_chunk=bound, batch=batch)
    else:
        out = U.run_prefill(wl, wdev, x, offsets, batch=batch, max_seqlen=bound, cache=cache)
    assert bool(torch.isfinite(out).all()) and bool(out.any(dim=1).all())
    assert cache.seq_lens.tolist() == [p + n for p, n in zip(prefix, lens)]
    for b in sorted({0, batch - 1, batch // 2, 63, 64, *(int(i) for i in rng.integers(0, batch, 24))}):
        if lens[b]:
            _check(wl, w, x[cu[b]:cu[b + 1]], U.f64(k[b]), U.f64(c[b]), prefix[b], U.f64(out[cu[b]:cu[b + 1]]),
                   f"{shape} {lengths} sequence {b}: {lens[b]} behind {prefix[b]}")


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_chunks_behind_cached_rows(shape, paged):
    lens, prefix, cap = [1, 33, 128, 70, 129, 40], [1500, 2047, 31, 0, 33, 2300], 2304   # the last one does not fit
    wl, w, x, rng = _setup(shape, sum(lens))
    k, c = W.draw_cache(wl, rng, len(lens), cap)
    if paged:
        cache = U.PagedDeviceCache(wl, len(lens), 32, cap // 32, seed=4)
        cache.store(B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    else:
        cache = U.DeviceCache(wl, len(lens), cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = U.f64(U.run_prefill_chunk(wl, U.upload_weights(w, "bf16"), x, cu, cache))
    for b in range(len(lens) - 1):
        _check(wl, w, x[cu[b]:cu[b + 1]], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[cu[b]:cu[b + 1]],
               f"{shape} {lens[b]} behind {prefix[b]}")
    assert not out[cu[-2]:].any() and cache.status.tolist() == [0] * 5 + [B.GTA_ERR_CACHE_FULL]
    assert cache.seq_lens.tolist() == [n + p for n, p in zip(lens[:-1], prefix[:-1])] + [prefix[-1]]


@pytest.mark.parametrize("prefix", [(472, 473), (2000, 10), (7900, 1100), (8100, 3000)], ids=str)   # 16 tiles, 17; 4 splits, none; most and fewer
@pytest.mark.parametrize("shape", ["1b", "mid", "slim"])
def test_chunks_in_large_slots(shape, prefix):
    """Sequences that use fewer splits than the launch has room for, and none."""
    lens, cap = [40, 40], 8192
    wl, w, x, rng = _setup(shape, sum(lens))
    k, c = W.draw_cache(wl, rng, 2, cap)
    cache = U.DeviceCache(wl, 2, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    out = U.f64(U.run_prefill_chunk(wl, U.upload_weights(w, "bf16"), x, np.array([0, 40, 80]), cache))
    for b in range(2):
        _check(wl, w, x[40 * b:40 * b + 40], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[40 * b:40 * b + 40],
               f"{shape} behind {prefix[b]}")


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_chunks_of_many_workgroups(shape, paged):
    """A loose bound on the chunks' lengths and enough sequences that no key halves or splits are taken: every tile shape
    walks more key tiles than it has stages in cache mode."""
    lens, prefix, cap = [1, 33, 128, 70, 129, 2, 300] * 2 + [40], [1500, 2047, 31, 0, 33, 700, 1000] * 2 + [2300], 2304
    wl, w, x, rng = _setup(shape, sum(lens))
    assert cap // 128 * len(lens) * wl.n_qgroups > 512
    k, c = W.draw_cache(wl, rng, len(lens), cap)
    if paged:
        cache = U.PagedDeviceCache(wl, len(lens), 64, cap // 64, seed=4)
        cache.store(B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    else:
        cache = U.DeviceCache(wl, len(lens), cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = U.f64(U.run_prefill_chunk(wl, U.upload_weights(w, "bf16"), x, cu, cache, max_chunk=cap))
    for b in range(len(lens) - 1):
        _check(wl, w, x[cu[b]:cu[b + 1]], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[cu[b]:cu[b + 1]],
               f"{shape} {lens[b]} behind {prefix[b]}")
    assert not out[cu[-2]:].any() and cache.status.tolist() == [0] * 14 + [B.GTA_ERR_CACHE_FULL]


@pytest.mark.parametrize("n", [1, 40])
@pytest.mark.parametrize("where", ["query", "keys"])
def test_nan_passes_the_merge(where, n):
    """Scores that are all NaN (a NaN in W_Q or in every cached key of a group) leave no maximum in any split; the heads of
    that group have no result all the same, the others keep theirs.  Without the gate, which would be NaN of itself."""
    wl, w, x, rng = _setup("1b", n)
    cap, prefix = 2304, 2200
    k, c = W.draw_cache(wl, rng, 1, cap)
    if where == "query":
        w["wq"][0, 5] = np.nan
    else:
        k[0, :prefix, 5] = np.nan
        w["wk"][:, 5] = np.nan
    cache = U.DeviceCache(wl, 1, cap, *(torch.from_numpy(a).to("cuda", torch.bfloat16) for a in (k, c)))
    cache.seq_lens.fill_(prefix)
    dev = {name: torch.from_numpy(a).to("cuda", torch.bfloat16) for name, a in w.items() if a is not None}
    out = U.f64(U.run_prefill_chunk(wl, dev, x, np.array([0, n]), cache, gate=False)).reshape(n, wl.n_qgroups, -1)
    assert np.isnan(out[:, 0]).all() and np.isfinite(out[:, 1:]).all()


@pytest.mark.parametrize("bound", [None, 2304])          # key splits, one key half
@pytest.mark.parametrize("shape", list(SHAPES))
def test_how_far_a_nan_token_reaches_back(shape, bound):
    """A NaN token behind a prefix that is no multiple of 32: rows at least 64 tokens before it, and the other sequences of
    the call, are not affected."""
    lens, prefix, bad, cap = [150, 40] + [1] * 13, [1500, 41] + [9] * 13, 120, 2304
    wl, w, x, rng = _setup(shape, sum(lens))
    k, c = W.draw_cache(wl, rng, len(lens), cap)
    cache = U.DeviceCache(wl, len(lens), cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    cu, xd = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), B.to_device(x, "bf16")
    xd[bad] = float("nan")
    cfg, cut = B.config_of(wl), torch.from_numpy(cu).cuda()
    most = max(lens) if bound is None else bound
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_PREFILL_CHUNK, len(lens), len(x), most))
    out = torch.empty((len(x), wl.n_heads * wl.head_dim), dtype=torch.bfloat16, device="cuda")
    weights = U.upload_weights(w, "bf16")
    B.gta_prefill_chunk(cfg, B.make_weights(weights), xd, cut, len(lens), len(x), most, cache.struct, None, out, ws)
    got = U.f64(out)
    _check(wl, w, x[:bad - 63], k[0].astype(np.float64), c[0].astype(np.float64), prefix[0], got[:bad - 63], f"{shape} before")
    assert np.isnan(got[bad:lens[0]]).all()
    _check(wl, w, x[cu[1]:cu[2]], k[1].astype(np.float64), c[1].astype(np.float64), prefix[1], got[cu[1]:cu[2]], f"{shape} beside")


@pytest.mark.parametrize("chunk,batch", [(False, 15), (False, 16), (True, 16), (True, 17)])
def test_latent_tile_changes_over(chunk, batch):
    """Either side of the rule that gives launches of few workgroups latent tiles of 128 columns: 15 (240 workgroups of 256
    columns) and 16 prompts of two query tiles, 16 and 17 chunks of one, with full, partial and single-row tiles."""
    lens = [40 if chunk else 129] * batch
    lens[1], lens[2] = 1, 128
    prefix, cap = [7 * b for b in range(batch)] if chunk else [0] * batch, 320
    wl, w, x, rng = _setup("1b", sum(lens))
    k, c = W.draw_cache(wl, rng, batch, cap)
    cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    wdev = U.upload_weights(w, "bf16")
    if chunk:
        cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
        out = U.f64(U.run_prefill_chunk(wl, wdev, x, cu, cache, max_chunk=128))
    else:
        out = U.f64(U.run_prefill(wl, wdev, x, cu, cache=cache))
    for b in range(batch):
        _check(wl, w, x[cu[b]:cu[b + 1]], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[cu[b]:cu[b + 1]],
               f"sequence {b}: {lens[b]} behind {prefix[b]}")


@pytest.mark.parametrize("shape,batch", [("paper", 3), ("paper", 9), ("mid", 3), ("mid", 9), ("1b", 32), ("1b", 33), ("wide", 9), ("wide", 17)])
def test_chunks_of_one_tile(shape, batch):
    """Chunks of at most 128 tokens: the XCDs take workgroups in a row, 15 and 45 (paper) do not divide by eight; more than the
    chip holds at once (1b 33, wide) are ranked and dealt to the XCDs by tile, below 16 by workgroup; some chunks are empty,
    some full."""
    lens, cap = ([128, 0, 1, 40, 77, 2, 127, 33, 64] * 4)[:batch], 1216
    prefix = [int(p) for p in np.random.default_rng(3).integers(0, cap - 128, batch)]
    wl, w, x, rng = _setup(shape, sum(lens))
    k, c = W.draw_cache(wl, rng, batch, cap)
    cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = U.f64(U.run_prefill_chunk(wl, U.upload_weights(w, "bf16"), x, cu, cache))
    for b in range(batch):
        if lens[b]:
            _check(wl, w, x[cu[b]:cu[b + 1]], k[b].astype(np.float64), c[b].astype(np.float64), prefix[b], out[cu[b]:cu[b + 1]],
                   f"{shape} {lens[b]} behind {prefix[b]}")
