"""The fp32 MFMA kernels against the oracle at the edges of their tiles: row tiles of 32 (few rows) and 64 (many),
32-key blocks dealt to four waves, latent slices of 64 and 128 columns, 16-row decode steps, splits without rows,
contiguous and block-table caches, full slots.

Bound: the fp32 tolerances of the parity gate (max-abs 1e-5, relative RMS 1e-5); sums of at most 1280 fp32 products
stay a factor of ten below them, of 3904 in 16 partial sums a factor of five."""
import numpy as np
import pytest
import torch

import gpu_util as U
from oracle import gta_oracle as orc
from paper_2506_17286_amd import workloads as W

pytestmark = pytest.mark.gpu

PAPER = dict(d_model=128, n_heads=20, n_qgroups=5, n_kgroups=1, n_cgroups=1, head_dim=64, latent_dim=128)
SHAPES = {
    "paper": PAPER,
    "paper_nq3": dict(PAPER, n_heads=12, n_qgroups=3),
    "paper_h1": dict(PAPER, n_heads=16, n_qgroups=16),                   # as many maps as a step has columns
    "heads32": dict(d_model=64, n_heads=8, n_qgroups=2, n_kgroups=2, n_cgroups=1, head_dim=32, latent_dim=64),
    "heads16": dict(d_model=64, n_heads=8, n_qgroups=4, n_kgroups=4, n_cgroups=2, head_dim=16, latent_dim=32),
    "latent192": dict(d_model=192, n_heads=4, n_qgroups=2, n_kgroups=1, n_cgroups=1, head_dim=64, latent_dim=192),
    "latent256": dict(d_model=64, n_heads=4, n_qgroups=4, n_kgroups=2, n_cgroups=2, head_dim=64, latent_dim=256),
    "heads128": dict(d_model=64, n_heads=2, n_qgroups=2, n_kgroups=1, n_cgroups=1, head_dim=128, latent_dim=128),
}
# paired: 360 attention workgroups of the paper's shape, those behind the first 256 in reverse (the others: none, or too many)
LENS = {"short": [1, 31, 32, 33, 97], "long": [513, 2, 160], "paired": [545, 2, 160, 33]}


def _wl(shape, **kw):
    return W.Workload(name=f"f32_{shape}", kind="prefill", batch=1, seqlen=64, dtype="f32", rope=True, seed=4100,
                      **dict(SHAPES[shape], **kw))


def _inputs(wl, tokens, with_wo):
    rng = W.make_rng(wl)
    # weights of standard deviation 1/sqrt(H): scores and gates of order one at these small widths
    w = W.draw_weights(wl, rng, with_wo=with_wo, std=wl.d_model ** -0.5)
    return w, W.draw_hidden(wl, rng, tokens)


def _scale(ref):
    return max(1.0, float(np.abs(ref).max()))


@pytest.mark.parametrize("with_wo", [False, True])
@pytest.mark.parametrize("lens", list(LENS))
@pytest.mark.parametrize("shape", list(SHAPES))
def test_prefill(shape, lens, with_wo):
    wl, lens = _wl(shape), LENS[lens]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    w, x = _inputs(wl, int(cu[-1]), with_wo)
    cache = U.DeviceCache(wl, len(lens), max(lens) + 3, fill=7.0)
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "f32"), x, cu, cache=cache))
    for b, n in enumerate(lens):
        ref, k, c = orc.prefill_sequence(U.oracle_config(wl), U.oracle_weights(w), x[cu[b]:cu[b + 1]])
        U.assert_close(out[cu[b]:cu[b + 1]], ref, "f32", f"{shape} sequence {b}", _scale(ref))
        U.assert_close(U.f64(cache.k[b, :n]), k.reshape(n, -1), "f32", "keys", _scale(k))
        U.assert_close(U.f64(cache.c[b, :n]), c.reshape(n, -1), "f32", "latents", _scale(c))
        assert bool((cache.k[b, n:] == 7.0).all()) and int(cache.seq_lens[b]) == n


@pytest.mark.parametrize("splits", [0, 1, 5, 40])          # 40: more than the one-round-trip tail takes
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("shape", ["paper", "paper_nq3", "paper_h1"])
def test_decode(shape, paged, splits):
    """Contexts around the 16-row step, an empty slot, a full slot; two steps in a row."""
    wl = _wl(shape)
    ctx = [0, 1, 15, 16, 17, 255, 300, 336]
    cap = 336                                              # the last slot is full
    w, x = _inputs(wl, 2 * len(ctx), True)
    wdev, (kw, cw) = U.upload_weights(w, "f32"), wl.kv_width
    rng = np.random.default_rng(5)
    k0 = rng.standard_normal((len(ctx), cap, kw)).astype(np.float32)
    c0 = rng.standard_normal((len(ctx), cap, cw)).astype(np.float32)
    if paged:
        cache = U.PagedDeviceCache(wl, len(ctx), 16, cap // 16, seed=3)
        cache.store(torch.from_numpy(k0).cuda(), torch.from_numpy(c0).cuda())
    else:
        cache = U.DeviceCache(wl, len(ctx), cap, torch.from_numpy(k0).cuda(), torch.from_numpy(c0).cuda())
    cache.seq_lens.copy_(torch.tensor(ctx, dtype=torch.int32))
    kr, cr = k0.astype(np.float64), c0.astype(np.float64)
    lens, status = np.array(ctx, dtype=np.int32), np.zeros(len(ctx), dtype=np.int32)
    for step in range(2):
        xs = x[step * len(ctx):(step + 1) * len(ctx)]
        ref = orc.decode(U.oracle_config(wl), U.oracle_weights(w), xs, kr, cr, lens, status, range(len(ctx)))
        out = U.f64(U.run_decode(wl, wdev, xs, cache, num_splits=splits))
        assert not out[-1].any()                           # the full slot
        U.assert_close(out, ref, "f32", f"{shape} step {step}", _scale(ref))
        kd, cd = cache.logical() if paged else (cache.k, cache.c)
        U.assert_close(U.f64(kd), kr, "f32", "keys", _scale(kr))
        U.assert_close(U.f64(cd), cr, "f32", "latents", _scale(cr))
        np.testing.assert_array_equal(cache.seq_lens.cpu().numpy(), lens)
        np.testing.assert_array_equal(cache.status.cpu().numpy(), status)


@pytest.mark.parametrize("splits", [1, 5, 40])
@pytest.mark.parametrize("shape", ["paper", "paper_nq3", "paper_h1"])
def test_decode_gate_of_large_pre_activations(shape, splits):
    """The Sigmoid alone, as the ratio of a gated and an ungated step, on pre-activations up to 40 that are exact (one-hot
    tokens pick rows of W_G).  Bound: exponential, sum, quotient and two products of at most one unit in the last place
    each, 6 x 2^-24."""
    wl, batch = _wl(shape), 5
    rng = W.make_rng(wl)
    w = W.draw_weights(wl, rng, std=wl.d_model ** -0.5)
    w["wg"] = rng.uniform(-40., 40., w["wg"].shape).astype(np.float32)
    x = np.eye(batch, wl.d_model, dtype=np.float32)
    k, c = W.draw_cache(wl, rng, batch, 200)
    outs = []
    for gate in (True, False):
        cache = U.DeviceCache(wl, batch, 200, torch.from_numpy(k).cuda(), torch.from_numpy(c).cuda())
        cache.seq_lens.copy_(torch.tensor([0, 15, 64, 100, 199], dtype=torch.int32))
        outs.append(U.f64(U.run_decode(wl, U.upload_weights(w, "f32"), x, cache, num_splits=splits, gate=gate)))
    got, ref = outs[0] / outs[1], orc.sigmoid(w["wg"][:batch])
    assert np.abs(got / ref - 1.).max() <= 6 * 2. ** -24


@pytest.mark.parametrize("shape", ["paper", "paper_nq3"])
def test_decode_and_chunk_store_the_same_keys(shape):
    """A token's key row does not depend on the call that stored it: one new token behind 64 prefixes, as a decode step and
    as a chunk, both on the projection that splits K.  Sums and angles are the same in both and the sines are rounded once
    from fp64, so that rows may differ only where the two frequencies (a power on the host, one on the device) round apart
    and the sine lies at the edge of a rounding: by one unit of the larger term, in less than one value in a thousand."""
    wl, batch, cap = _wl(shape), 64, 6000
    w, x = _inputs(wl, batch, False)
    wdev, prefix = U.upload_weights(w, "f32"), np.random.default_rng(8).integers(0, cap, batch)
    keys = []
    for chunk in (True, False):
        cache = U.DeviceCache(wl, batch, cap)
        cache.seq_lens.copy_(torch.from_numpy(prefix.astype(np.int32)))
        if chunk:
            U.run_prefill_chunk(wl, wdev, x, np.arange(batch + 1), cache)
        else:
            U.run_decode(wl, wdev, x, cache)
        keys.append(U.f64(cache.k[torch.arange(batch), torch.from_numpy(prefix)]))
    assert (keys[0] != keys[1]).mean() < 1e-3 and np.abs(keys[0] - keys[1]).max() <= 2 ** -23 * np.abs(keys[0]).max()


@pytest.mark.parametrize("batch", [33, 256, 257, 300])
def test_decode_of_many_sequences(batch):
    """Several row tiles of the kernel for few rows, and the decode epilogue in the one for many."""
    wl, cap = _wl("paper"), 80
    w, x = _inputs(wl, batch, True)
    k, c = W.draw_cache(wl, W.make_rng(wl), batch, cap)
    ctx = np.random.default_rng(batch).integers(0, cap, batch).astype(np.int32)
    ctx[batch // 2] = cap                                  # full
    cache = U.DeviceCache(wl, batch, cap, torch.from_numpy(k).cuda(), torch.from_numpy(c).cuda())
    cache.seq_lens.copy_(torch.from_numpy(ctx))
    out = U.f64(U.run_decode(wl, U.upload_weights(w, "f32"), x, cache))
    kr, cr, lens, status = k.astype(np.float64), c.astype(np.float64), ctx.copy(), np.zeros(batch, dtype=np.int32)
    ref = orc.decode(U.oracle_config(wl), U.oracle_weights(w), x, kr, cr, lens, status, range(batch))
    U.assert_close(out, ref, "f32", "out", _scale(ref))
    U.assert_close(U.f64(cache.k), kr, "f32", "keys", _scale(kr))
    U.assert_close(U.f64(cache.c), cr, "f32", "latents", _scale(cr))
    np.testing.assert_array_equal(cache.seq_lens.cpu().numpy(), lens)
    np.testing.assert_array_equal(cache.status.cpu().numpy(), status)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("lens", [[33, 1, 64, 5, 20], [33, 300, 1, 64, 20]], ids=str)   # projection of few, of many rows
@pytest.mark.parametrize("shape", ["paper", "heads32", "heads16"])
def test_chunk(shape, lens, paged):
    """Per-token RoPE rows behind uneven prefixes; the last chunk does not fit."""
    wl, prefix, cap = _wl(shape), [0, 37, 100, 255, 390], 400
    cfg, cu = U.oracle_config(wl), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    w, x = _inputs(wl, int(cu[-1]), False)
    k, c = W.draw_cache(wl, W.make_rng(wl), len(lens), cap)
    if paged:
        cache = U.PagedDeviceCache(wl, len(lens), 16, cap // 16, seed=3)
        cache.store(torch.from_numpy(k).cuda(), torch.from_numpy(c).cuda())
    else:
        cache = U.DeviceCache(wl, len(lens), cap, torch.from_numpy(k).cuda(), torch.from_numpy(c).cuda())
    cache.seq_lens.copy_(torch.tensor(prefix, dtype=torch.int32))
    out = U.f64(U.run_prefill_chunk(wl, U.upload_weights(w, "f32"), x, cu, cache))
    kd, cd = (U.f64(t) for t in (cache.logical() if paged else (cache.k, cache.c)))
    ow = U.oracle_weights(w)
    for b, (n, p) in enumerate(zip(lens, prefix)):
        rows, pos = slice(cu[b], cu[b + 1]), np.arange(p, p + n)
        if p + n > cap:
            assert not out[rows].any() and int(cache.seq_lens[b]) == p
            continue
        Q, K, C, G = orc.project_tokens(cfg, ow, x[rows], pos)
        K = np.concatenate([k[b, :p].reshape(p, wl.n_kgroups, wl.head_dim), K])
        C = np.concatenate([c[b, :p].reshape(p, wl.n_cgroups, wl.latent_dim), C])
        L = np.stack([orc.attention_map_rows(cfg, Q[:, g], pos, K[:, cfg.k_of_group(g)]) @ C[:, cfg.c_of_group(g)]
                      for g in range(wl.n_qgroups)], axis=1)
        ref = orc.decode_heads(cfg, ow, L, G)
        U.assert_close(out[rows], ref, "f32", f"{shape} {n} behind {p}", _scale(ref))
        U.assert_close(kd[b, :p + n], K.reshape(p + n, -1), "f32", "keys", _scale(K))
        U.assert_close(cd[b, :p + n], C.reshape(p + n, -1), "f32", "latents", _scale(C))
        assert int(cache.seq_lens[b]) == p + n


@pytest.mark.parametrize("gate", ["silu", "relu2", False])
@pytest.mark.parametrize("shape", ["paper", "heads32"])
def test_gates(shape, gate):
    """The other gates in the decoder epilogues (few and many rows) and in the decode tails (5 and 40 splits)."""
    wl = _wl(shape)
    for lens in LENS.values():
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        w, x = _inputs(wl, int(cu[-1]), False)
        ref, _, _ = orc.prefill(U.oracle_config(wl, gate), U.oracle_weights(w), x, cu)
        U.assert_close(U.f64(U.run_prefill(wl, U.upload_weights(w, "f32"), x, cu, gate=gate)), ref, "f32", f"{lens}", _scale(ref))
    ctx = np.array([0, 20, 130], dtype=np.int32)
    w, x = _inputs(wl, 3, False)
    k, c = W.draw_cache(wl, W.make_rng(wl), 3, 160)
    ref = orc.decode(U.oracle_config(wl, gate), U.oracle_weights(w), x, k.astype(np.float64), c.astype(np.float64), ctx.copy(),
                     np.zeros(3, dtype=np.int32), range(3))
    for splits in (5, 40):
        cache = U.DeviceCache(wl, 3, 160, torch.from_numpy(k).cuda(), torch.from_numpy(c).cuda())
        cache.seq_lens.copy_(torch.from_numpy(ctx))
        out = U.f64(U.run_decode(wl, U.upload_weights(w, "f32"), x, cache, num_splits=splits, gate=gate))
        U.assert_close(out, ref, "f32", f"{splits} splits", _scale(ref))


@pytest.mark.parametrize("longest", [4, 5, 6, 7])
@pytest.mark.parametrize("shape", ["paper", "heads32", "latent256", "heads128"])
def test_prefill_of_many_tiny_prompts(shape, longest):
    """Both sides of the lengths up to which such a batch stays on the kernel with a wave per row."""
    wl, lens = _wl(shape), [longest] + list(np.random.default_rng(longest).integers(1, longest + 1, 599))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    w, x = _inputs(wl, int(cu[-1]), False)
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "f32"), x, cu))
    ref, _, _ = orc.prefill(U.oracle_config(wl), U.oracle_weights(w), x, cu)
    U.assert_close(out, ref, "f32", shape, _scale(ref))


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 64, 65, 145, 256])
@pytest.mark.parametrize("shape", ["paper", "heads32", "heads16"])
def test_gemms_of_few_rows(shape, rows):
    """Row counts around the three tiles of the few-row GEMMs (paper: 16 x 16 up to 32 rows, 32 x 16 up to 64, 32 x 32 behind;
    the narrow shapes change over at 144): rotated tiles narrower than a head, as wide, and wider, and partial row tiles."""
    wl = _wl(shape)
    w, x = _inputs(wl, rows, True)
    cache = U.DeviceCache(wl, 1, rows + 3, fill=7.0)
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "f32"), x, [0, rows], cache=cache))
    ref, k, c = orc.prefill_sequence(U.oracle_config(wl), U.oracle_weights(w), x)
    U.assert_close(out, ref, "f32", f"{shape} {rows} rows", _scale(ref))
    U.assert_close(U.f64(cache.k[0, :rows]), k.reshape(rows, -1), "f32", "keys", _scale(k))
    U.assert_close(U.f64(cache.c[0, :rows]), c.reshape(rows, -1), "f32", "latents", _scale(c))
    assert bool((cache.k[0, rows:] == 7.0).all())


@pytest.mark.parametrize("rows", [16, 64, 70])            # 16 x 16, 32 x 16 and 32 x 32 tiles
@pytest.mark.parametrize("d_model", [640, 1216, 1280, 1344, 2560, 2624, 3904])
def test_rounds_of_a_contraction(d_model, rows):
    """16 waves take five groups of the contraction each before they ask for more: part of a round, one, two and more, and some
    groups over."""
    wl = W.scaled(_wl("paper"), d_model=d_model)
    w, x = _inputs(wl, rows, True)
    cache = U.DeviceCache(wl, 1, rows)
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "f32"), x, [0, rows], cache=cache))
    ref, k, c = orc.prefill_sequence(U.oracle_config(wl), U.oracle_weights(w), x)
    U.assert_close(out, ref, "f32", f"{d_model} wide, {rows} rows", _scale(ref))
    U.assert_close(U.f64(cache.k[0, :rows]), k.reshape(rows, -1), "f32", "keys", _scale(k))
    U.assert_close(U.f64(cache.c[0, :rows]), c.reshape(rows, -1), "f32", "latents", _scale(c))
