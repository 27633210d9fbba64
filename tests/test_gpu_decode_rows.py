"""Decode steps through the few-row GEMMs (K split inside the workgroup) and the split counts of short contexts: row
tiles of 32, K shorter than one round of the 16 waves and longer than two, rotated tiles of heads of 64 and 128, W_O,
full slots; and the fixed scratch array where the library's own split count would not fit it.

Bounds: the bf16 tolerances of the parity gate, the max-abs one scaled by the largest reference value."""
import numpy as np
import pytest
import torch

import gpu_util as U
from oracle import gta_oracle as orc
from paper_2506_17286_amd import binding as B, workloads as W

pytestmark = pytest.mark.gpu

CASES = [("paper", 128, 1), ("paper", 128, 33), ("paper", 1408, 32), ("paper", 1408, 128), ("paper", 128, 129),
         ("1b", 128, 1), ("1b", 2176, 8), ("1b", 256, 9)]


def _wl(family, d_model):
    base = W.PAPER_WORKLOADS[1] if family == "paper" else W.WORKLOADS[3]
    return W.scaled(base, d_model=d_model, seed=5200)


@pytest.mark.parametrize("with_wo", [False, True])
@pytest.mark.parametrize("family,d_model,batch", CASES)
def test_decode_rows(family, d_model, batch, with_wo):
    wl, cap = _wl(family, d_model), 200
    rng = W.make_rng(wl)
    w = W.draw_weights(wl, rng, with_wo=with_wo, std=d_model ** -0.5)
    x = W.draw_hidden(wl, rng, batch)
    k, c = W.draw_cache(wl, rng, batch, cap)
    ctx = rng.integers(0, cap, size=batch).astype(np.int32)
    ctx[-1] = cap if batch > 1 else 63                      # the last slot is full
    cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.from_numpy(ctx))
    out = U.f64(U.run_decode(wl, U.upload_weights(w, "bf16"), x, cache))
    kr, cr, lens, status = k.astype(np.float64), c.astype(np.float64), ctx.copy(), np.zeros(batch, dtype=np.int32)
    ref = orc.decode(U.oracle_config(wl), U.oracle_weights(w), x, kr, cr, lens, status, range(batch))
    U.assert_close(out, ref, "bf16", "out", max(1.0, float(np.abs(ref).max())))
    U.assert_close(U.f64(cache.k), kr, "bf16", "keys", float(np.abs(kr).max()))
    U.assert_close(U.f64(cache.c), cr, "bf16", "latents", float(np.abs(cr).max()))
    np.testing.assert_array_equal(cache.seq_lens.cpu().numpy(), lens)
    np.testing.assert_array_equal(cache.status.cpu().numpy(), status)


def test_static_scratch_takes_coarser_splits_where_its_own_do_not_fit():
    wl, batch, cap = W.scaled(W.WORKLOADS[4], kind="decode", d_model=256, seed=5300), 58, 256
    cfg = B.config_of(wl)
    assert B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, batch, 0, cap) > B.GTA_STATIC_SCRATCH_BYTES
    assert B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, batch, 0, cap, 1) <= B.GTA_STATIC_SCRATCH_BYTES
    rng = W.make_rng(wl)
    wdev = U.upload_weights(W.draw_weights(wl, rng), "bf16")
    x = B.to_device(W.draw_hidden(wl, rng, batch), "bf16")
    k, c = (B.to_device(a, "bf16") for a in W.draw_cache(wl, rng, batch, cap))
    lens = torch.full((batch,), 200, dtype=torch.int32, device="cuda")
    outs = []
    for static in (True, False):
        cache = U.DeviceCache(wl, batch, cap, k.clone(), c.clone(), lens.clone())
        out = torch.full((batch, wl.n_heads * wl.head_dim), float("nan"), dtype=torch.bfloat16, device="cuda")
        if static:
            B.gta_decode_static(cfg, B.make_weights(wdev), x, batch, cache.struct, None, out, 0)
        else:
            ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, batch, 0, cap, 1))
            B.gta_decode(cfg, B.make_weights(wdev), x, batch, cache.struct, None, out, 1, ws)
        torch.cuda.synchronize()
        outs.append((out, cache.k, cache.c, cache.seq_lens))
    assert all(torch.equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("most,cap", [(64, 2048), (128, 512), (256, 256)])
def test_workspace_of_a_full_batch_serves_fewer_sequences(most, cap):
    """fp32 steps: 63 sequences take more splits each than 64; slices of at least 256 rows fit the workspace of 64 all the
    same."""
    wl = W.scaled(_wl("paper", 128), dtype="f32")
    cfg = B.config_of(wl)
    rng = W.make_rng(wl)
    w, x = W.draw_weights(wl, rng, std=wl.d_model ** -0.5, with_wo=True), W.draw_hidden(wl, rng, most)
    wdev, lens = U.upload_weights(w, "f32"), torch.from_numpy(rng.integers(0, cap, most).astype(np.int32)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(1)
    k, c = (torch.randn((most, cap, width), device="cuda", generator=gen) for width in wl.kv_width)
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, most, 0, cap))
    assert any(B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, n, 0, cap) > ws.numel() for n in range(1, most))
    for batch in (most, most - 1, most // 2 + 1, 2):
        cache = U.DeviceCache(wl, most, cap, k.clone(), c.clone(), lens.clone())
        out = torch.empty((batch, wl.d_model), device="cuda")
        B.gta_decode(cfg, B.make_weights(wdev), B.to_device(x[:batch], "f32"), batch, cache.struct, None, out, 0, ws)
        again = U.DeviceCache(wl, most, cap, k, c, lens.clone())
        ref = U.f64(U.run_decode(wl, wdev, x[:batch], again))
        U.assert_close(U.f64(out), ref, "f32", f"{batch} sequences", max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("splits", [4, 80])             # 80: more than the one-round-trip tails take
@pytest.mark.parametrize("family,dtype,batch", [("paper", "f32", 5), ("tiny", "f32", 5), ("paper", "bf16", 5), ("1b", "bf16", 5),
                                                ("1b", "bf16", 64), ("1b", "bf16", 256), ("wide", "bf16", 5)])
def test_a_context_split_of_nothing_but_nan(family, dtype, batch, splits):
    """NaN keys that fill whole splits (256 rows in 4, 1280 in 80) and a NaN query leave their sequence without a result,
    whichever merge follows, and no other sequence is affected."""
    base = {"paper": W.PAPER_WORKLOADS[1], "1b": W.WORKLOADS[3], "wide": W.WORKLOADS[4], "tiny": W.WORKLOADS[0]}[family]
    wl = W.scaled(base, kind="decode", d_model=256, dtype=dtype, seed=5400)
    rng, cap = W.make_rng(wl), 256 if splits == 4 else 1280
    wdev = U.upload_weights(W.draw_weights(wl, rng, std=wl.d_model ** -0.5), dtype)
    x, gen = W.draw_hidden(wl, rng, batch), torch.Generator(device="cuda").manual_seed(1)
    k, c = (torch.randn((batch, cap, width), device="cuda", generator=gen).to(torch.float32 if dtype == "f32" else torch.bfloat16)
            for width in wl.kv_width)
    lens = torch.full((batch,), cap - 1, dtype=torch.int32, device="cuda")

    def step(x):
        return U.run_decode(wl, wdev, x, U.DeviceCache(wl, batch, cap, k.clone(), c.clone(), lens.clone()), num_splits=splits, gate=False)
    clean = step(x)
    k[1, 64:128 if splits == 4 else 96] = float("nan")
    x[3] = np.nan
    out = step(x)
    assert torch.isfinite(clean).all() and torch.isnan(out[1]).all() and torch.isnan(out[3]).all()
    others = [b for b in range(batch) if b not in (1, 3)]
    assert torch.equal(out[others], clean[others])


@pytest.mark.parametrize("splits", [0, 1, 3])
@pytest.mark.parametrize("d_model", [128, 1664])          # queries and new rows finished by the projection, by the stream
@pytest.mark.parametrize("maps,latents,paged", [(3, 1, False), (5, 1, True), (6, 1, False), (6, 2, True), (10, 2, False)])
def test_narrow_rows_around_a_step(maps, latents, paged, d_model, splits):
    """The stream over narrow rows takes 16 rows a step, two steps in flight in each of four waves: contexts around one step,
    one round and two rounds of the waves, an empty and a full slot, slices without rows; what lies behind a context is NaN."""
    wl = W.scaled(_wl("paper", d_model), n_heads=2 * maps, n_qgroups=maps, n_cgroups=latents)
    ctx = np.array([0, 1, 14, 15, 16, 17, 62, 63, 64, 65, 127, 128, 129, 200, 272], dtype=np.int32)   # the last slot is full
    batch, cap = len(ctx), 272
    rng = W.make_rng(wl)
    w = W.draw_weights(wl, rng, with_wo=True, std=d_model ** -0.5)
    x = W.draw_hidden(wl, rng, batch)
    k, c = W.draw_cache(wl, rng, batch, cap)
    for b, n in enumerate(ctx):
        k[b, n:] = c[b, n:] = np.nan
    if paged:
        cache = U.PagedDeviceCache(wl, batch, 16, cap // 16, seed=2)
        cache.store(B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    else:
        cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.from_numpy(ctx))
    out = U.f64(U.run_decode(wl, U.upload_weights(w, "bf16"), x, cache, num_splits=splits))
    kr, cr, lens, status = k.astype(np.float64), c.astype(np.float64), ctx.copy(), np.zeros(batch, dtype=np.int32)
    ref = orc.decode(U.oracle_config(wl), U.oracle_weights(w), x, kr, cr, lens, status, range(batch))
    U.assert_close(out, ref, "bf16", "out", max(1.0, float(np.abs(ref).max())))
    np.testing.assert_array_equal(cache.seq_lens.cpu().numpy(), lens)
    np.testing.assert_array_equal(cache.status.cpu().numpy(), status)
    k2, c2 = cache.logical() if paged else (cache.k, cache.c)
    for b in range(batch - 1):
        U.assert_close(U.f64(k2[b, ctx[b]]), kr[b, ctx[b]], "bf16", "new key", max(1.0, float(np.abs(kr[b, ctx[b]]).max())))
        U.assert_close(U.f64(c2[b, ctx[b]]), cr[b, ctx[b]], "bf16", "new latent", max(1.0, float(np.abs(cr[b, ctx[b]]).max())))


@pytest.mark.parametrize("with_wo", [False, True])
@pytest.mark.parametrize("splits", [0, 1, 5, 8, 9])        # 4 at a time; 9: another tail
@pytest.mark.parametrize("batch", [32, 33, 64, 255])      # 32: another tail; one row in the last tile, full tiles, 15 rows
def test_tail_of_sixteen_sequences(batch, splits, with_wo):
    """Contexts from none to full, among them ones that leave splits without rows."""
    wl, cap = _wl("1b", 256), 640
    rng = W.make_rng(wl)
    w = W.draw_weights(wl, rng, with_wo=with_wo, std=wl.d_model ** -0.5)
    x = W.draw_hidden(wl, rng, batch)
    k, c = W.draw_cache(wl, rng, batch, cap)
    ctx = rng.integers(0, cap, size=batch).astype(np.int32)
    ctx[:4] = 0, 1, 3, cap
    cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.from_numpy(ctx))
    out = U.f64(U.run_decode(wl, U.upload_weights(w, "bf16"), x, cache, num_splits=splits))
    kr, cr, lens, status = k.astype(np.float64), c.astype(np.float64), ctx.copy(), np.zeros(batch, dtype=np.int32)
    ref = orc.decode(U.oracle_config(wl), U.oracle_weights(w), x, kr, cr, lens, status, range(batch))
    U.assert_close(out, ref, "bf16", "out", max(1.0, float(np.abs(ref).max())))
    np.testing.assert_array_equal(cache.seq_lens.cpu().numpy(), lens)
    np.testing.assert_array_equal(cache.status.cpu().numpy(), status)


@pytest.mark.parametrize("splits", [1, 5])
@pytest.mark.parametrize("batch", [32, 33])                # one sequence a workgroup, sixteen
def test_merged_outputs_keep_fp32(batch, splits):
    """Two latent columns whose means over 1024 rows of equal weight, exact in fp32, differ by 2^-19 at a value of 1.001; the
    decoder subtracts them.  An error of one in 2^23 of either is one in 16 of the difference."""
    wl, n = _wl("1b", 256), 1024
    rng = W.make_rng(wl)
    w = W.draw_weights(wl, rng)
    w["wp"][:] = 0.0
    w["wp"][:, 0, 0], w["wp"][:, 1, 0] = -1.0, 1.0
    k, c = np.zeros((batch, n, wl.kv_width[0]), dtype=np.float32), np.zeros((batch, n, wl.kv_width[1]), dtype=np.float32)
    c[:, :, :2], c[:, 0, :2], c[:, 1, :2] = 1.0, 4.0, 0.25
    c[:, 1, 1] += 2.0 ** -9
    cache = U.DeviceCache(wl, batch, n, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.fill_(n - 1)                             # the new row is 0, as are all scores
    x = np.zeros((batch, wl.d_model), dtype=np.float32)
    out = U.f64(U.run_decode(wl, U.upload_weights(w, "bf16"), x, cache, num_splits=splits, gate=False))
    heads = out.reshape(batch, wl.n_heads, wl.head_dim)
    np.testing.assert_allclose(heads[:, :, 0], 2.0 ** -19, rtol=2.0 ** -4)
    assert not heads[:, :, 1:].any()


@pytest.mark.parametrize("where", ["latents", "matrix"])
@pytest.mark.parametrize("splits", [1, 5])
@pytest.mark.parametrize("batch", [32, 33])                # one sequence a workgroup, sixteen
def test_infinities_in_the_tail(batch, splits, where):
    """An infinite latent or decoder weight gives the infinities of the float64 reference, and nothing else changes."""
    wl, n = _wl("1b", 256), 200
    rng = W.make_rng(wl)
    w, x = W.draw_weights(wl, rng), W.draw_hidden(wl, rng, batch)
    k, c = W.draw_cache(wl, rng, batch, n)
    lens = rng.integers(50, n, size=batch).astype(np.int32)

    def step():
        cache = U.DeviceCache(wl, batch, n, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
        cache.seq_lens.copy_(torch.from_numpy(lens))
        return U.f64(U.run_decode(wl, U.upload_weights(w, "bf16"), x, cache, num_splits=splits, gate=False))
    clean = step()
    if where == "latents":
        c[1, 7, 3], c[batch - 1, 40, 500] = np.inf, -np.inf
    else:
        w["wp"][0, 3, 5], w["wp"][15, 500, 100] = np.inf, -np.inf
    got = step()
    with np.errstate(invalid="ignore"):
        ref = orc.decode(U.oracle_config(wl, False), U.oracle_weights(w), x, k.astype(np.float64), c.astype(np.float64), lens.copy(),
                         np.zeros(batch, dtype=np.int32), range(batch))
    bad = ~np.isfinite(ref)
    assert bad.sum() == (2 * wl.n_heads * wl.head_dim if where == "latents" else 2 * batch) and not np.isnan(ref).any()
    np.testing.assert_array_equal(got[bad], ref[bad])
    np.testing.assert_array_equal(got[~bad], clean[~bad])


NARROW = [(3, 1), (5, 1), (6, 1), (6, 2), (10, 2)]         # maps, latents


@pytest.mark.parametrize("splits", [1, 5])
@pytest.mark.parametrize("n", [1, 15, 16, 33, 300])
@pytest.mark.parametrize("maps,latents", NARROW)
def test_infinite_latents_of_narrow_rows(maps, latents, n, splits):
    """The stream and the merge alone; with one row the weight is exactly 1."""
    wl = W.scaled(_wl("paper", 128), n_heads=2 * maps, n_qgroups=maps, n_cgroups=latents)
    rng = np.random.default_rng(n)
    q, k, c = (W.round_to_dtype(rng.standard_normal(s).astype(np.float32), "bf16") for s in
               ((1, maps, wl.head_dim), (1, n, wl.head_dim), (1, n, latents * wl.latent_dim)))
    c[0, -1, 7], c[0, n // 2, -1] = np.inf, -np.inf
    cache = U.DeviceCache(wl, 1, n, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.fill_(n)
    cfg = B.config_of(wl)
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, 1, 0, n, splits))
    out = torch.empty((maps, wl.latent_dim), device="cuda")
    B.gta_decode_attention(cfg, torch.from_numpy(q.reshape(1, -1).copy()).cuda(), cache.struct, None, 1, splits, ws)
    B.gta_decode_combine(cfg, cache.struct, None, 1, splits, ws, out)
    got, oc = U.f64(out), U.oracle_config(wl)
    c64 = c[0].astype(np.float64).reshape(n, latents, -1)
    ref = np.stack([(orc.attention_map_rows(oc, q[:, g].astype(np.float64), np.array([n - 1]), k[0].astype(np.float64)) @ c64[:, oc.c_of_group(g)])[0]
                    for g in range(maps)])
    bad = ~np.isfinite(ref)
    assert bad.any() and not np.isnan(ref).any()
    np.testing.assert_array_equal(got[bad], ref[bad])
    U.assert_close(got[~bad], ref[~bad], "bf16", "finite columns", max(1.0, float(np.abs(ref[~bad]).max())))


@pytest.mark.parametrize("d_model", [128, 1664])          # new rows finished by the projection, by the stream
@pytest.mark.parametrize("maps,latents", [(5, 1), (10, 2)])
def test_new_latent_that_overflows(maps, latents, d_model):
    """Into an empty slot and behind 20 rows: 1e10 times 1e30 is an infinity in 16 bits, and so are the outputs that it reaches."""
    wl = W.scaled(_wl("paper", d_model), n_heads=2 * maps, n_qgroups=maps, n_cgroups=latents)
    rng, batch, cap = W.make_rng(wl), 3, 64
    w, x = W.draw_weights(wl, rng, std=d_model ** -0.5), W.draw_hidden(wl, rng, batch)
    k, c = W.draw_cache(wl, rng, batch, cap)
    for name in ("wq", "wk", "wc", "wg"):
        w[name][0] = 0.0
    w["wc"][0, 7], w["wc"][0, -1] = W.round_to_dtype(np.array([1e30, -1e30], dtype=np.float32), "bf16")
    x[:, 0] = W.round_to_dtype(np.array([1e10, 1e10, 0.0], dtype=np.float32), "bf16")
    lens = np.array([0, 20, 20], dtype=np.int32)
    cache = U.DeviceCache(wl, batch, cap, B.to_device(k, "bf16"), B.to_device(c, "bf16"))
    cache.seq_lens.copy_(torch.from_numpy(lens))
    got = U.f64(U.run_decode(wl, U.upload_weights(w, "bf16"), x, cache, gate=False))
    ref = orc.decode(U.oracle_config(wl, False), U.oracle_weights(w), x, k.astype(np.float64), c.astype(np.float64), lens.copy(),
                     np.zeros(batch, dtype=np.int32), range(batch))
    assert (np.abs(ref[:2]) > 1e30).all()
    if latents == 2:                                        # one infinity in each latent
        np.testing.assert_array_equal(got[:2], np.sign(ref[:2]) * np.inf)
    else:                                                   # both in one: the sum of two infinities
        w7, w_last = (np.sign(w["wp"][:, i].reshape(-1)) for i in (7, -1))
        same = w7 == -w_last
        np.testing.assert_array_equal(got[:2, same], np.broadcast_to(w7[same] * np.inf, (2, same.sum())))
        assert np.isnan(got[:2, ~same]).all()
    U.assert_close(got[2], ref[2], "bf16", "without", max(1.0, float(np.abs(ref[2]).max())))
