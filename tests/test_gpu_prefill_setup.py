"""What a prefill call derives from offsets, lengths and page tables before its GEMMs: sequences of more than 64 pages (a
wave looks at 64 table entries at a time), a missing page behind the first 64, several tokens per wave.

Reference: the same tokens as a fresh prompt into contiguous caches.  Both calls run the same projection on the same
bf16 inputs with the same angles, so the cached rows are equal bit by bit."""
import numpy as np
import pytest
import torch

import gpu_util as U
from paper_2506_17286_amd import binding as B, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,page,chunk", [([2201, 2198, 7], 32, True), ([2201, 2198, 7], 32, False), ([1030, 1030, 7], 16, False)])
def test_sequences_of_many_pages(lens, page, chunk):
    wl = W.scaled(W.WORKLOADS[1], d_model=128, n_heads=4, n_qgroups=2, n_kgroups=1, latent_dim=128, seed=9100)
    rng = W.make_rng(wl)
    w, x = W.draw_weights(wl, rng, std=wl.d_model ** -0.5), W.draw_hidden(wl, rng, sum(lens))
    wdev, cu = U.upload_weights(w, "bf16"), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    plain = U.DeviceCache(wl, 3, 2560)
    U.run_prefill(wl, wdev, x, cu, cache=plain)
    paged = U.PagedDeviceCache(wl, 3, page, 2560 // page, seed=1, missing=[(1, lens[1] // page)])
    (U.run_prefill_chunk if chunk else U.run_prefill)(wl, wdev, x, cu, cache=paged)
    assert paged.seq_lens.tolist() == [lens[0], 0, lens[2]] and paged.status.tolist() == [0, B.GTA_ERR_CACHE_FULL, 0]
    k, c = paged.logical()
    for s in (0, 2):
        assert torch.equal(k[s, :lens[s]], plain.k[s, :lens[s]]) and torch.equal(c[s, :lens[s]], plain.c[s, :lens[s]])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("call", ["prefill", "chunk", "decode"])
def test_rope_base_below_one(dtype, call):
    """A base of 2^-64 makes frequencies up to 2^62, far outside what a two-part reduction by pi/2 takes.  At such angles one
    unit in the last place of a frequency is many turns, so no two implementations rotate alike; but every one rotates:
    the lengths of the pairs (j, j + d_h/2) of the stored keys are those of the unrotated projection (bounds of the parity
    gate)."""
    wl = W.scaled(W.PAPER_WORKLOADS[1], d_model=128, dtype=dtype, rope_base=2. ** -64, seed=9200)
    rng, n = W.make_rng(wl), 100
    w, x = W.draw_weights(wl, rng, std=wl.d_model ** -0.5), W.draw_hidden(wl, rng, n)
    wdev, cu = U.upload_weights(w, dtype), np.array([0, n], dtype=np.int32)
    if call == "decode":     # token b behind b rows, one slot each
        cache = U.DeviceCache(wl, n, n)
        cache.seq_lens.copy_(torch.arange(n))
        U.run_decode(wl, wdev, x, cache)
        rows = cache.k[torch.arange(n), torch.arange(n)]
    else:
        cache = U.DeviceCache(wl, 1, n)
        (U.run_prefill if call == "prefill" else U.run_prefill_chunk)(wl, wdev, x, cu, cache=cache)
        rows = cache.k[0]
    pairs = lambda k: np.hypot(k[:, :wl.head_dim // 2], k[:, wl.head_dim // 2:])
    ref = pairs(x.astype(np.float64) @ w["wk"].astype(np.float64))
    U.assert_close(pairs(U.f64(rows)), ref, dtype, call, max(1.0, float(ref.max())))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lens", [[5], [33, 64], [0, 7, 0, 0, 3, 0], [3, 1, 4, 1, 5, 9, 2, 6, 5, 3, 5, 8, 9, 7, 9, 3], [4] * 17, [6, 6]],
                         ids=["one", "two", "empty", "sixteen", "seventeen", "no_offsets"])
def test_prompts_without_a_setup_launch(dtype, lens):
    """Up to 16 short prompts (of 17 a launch in front works out rows, sines and lengths): sequences without tokens at either
    end, a missing page, no offsets.  Chunks behind nothing take the table; their rows are equal bit by bit, and so are
    lengths and flags."""
    wl = W.scaled(W.PAPER_WORKLOADS[1], d_model=128, dtype=dtype, seed=9300)
    rng = W.make_rng(wl)
    w, x = W.draw_weights(wl, rng, std=wl.d_model ** -0.5), W.draw_hidden(wl, rng, sum(lens))
    wdev, cu = U.upload_weights(w, dtype), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    last, page = len(lens) - 1, 32
    plain, paged, chunk = (U.DeviceCache(wl, len(lens), 128), U.PagedDeviceCache(wl, len(lens), page, 4, seed=1, missing=[(last, 0)]),
                           U.DeviceCache(wl, len(lens), 128))
    out = U.run_prefill(wl, wdev, x, None if lens == [6, 6] else cu, cache=plain, batch=len(lens))
    U.run_prefill(wl, wdev, x, cu, cache=paged)
    ref = U.run_prefill_chunk(wl, wdev, x, cu, cache=chunk)
    assert plain.seq_lens.tolist() == lens and plain.status.tolist() == [0] * len(lens)
    full = lens[last] > 0                                  # a sequence without tokens needs no page
    assert paged.seq_lens.tolist() == lens[:-1] + [0 if full else lens[last]]
    assert paged.status.tolist() == [0] * last + [B.GTA_ERR_CACHE_FULL if full else 0]
    k, c = paged.logical()
    for s, n in enumerate(lens):
        assert torch.equal(plain.k[s, :n], chunk.k[s, :n]) and torch.equal(plain.c[s, :n], chunk.c[s, :n])
        if s != last:
            assert torch.equal(k[s, :n], chunk.k[s, :n]) and torch.equal(c[s, :n], chunk.c[s, :n])
    U.assert_close(U.f64(out), U.f64(ref), dtype, "outputs")
