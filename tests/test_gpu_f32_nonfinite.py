"""Prefill and decode in fp32 on values that are not finite: a token that holds NaN or infinities (uninitialised padding at the
tail of equal-length sequences) reaches the rows that see it and no earlier one; keys whose score overflows to -inf have
weight 0, also where they fill a whole block.

Reference: float64, every row on the keys it sees only.  Bounds: the fp32 tolerances of the parity gate on what is
finite there; what is not finite there has to be the same infinity or a NaN."""
import numpy as np
import pytest
import torch

import gpu_util as U
from oracle import gta_oracle as orc
from paper_2506_17286_amd import binding as B, workloads as W

pytestmark = pytest.mark.gpu

PAPER = dict(d_model=128, n_heads=20, n_qgroups=5, n_kgroups=1, n_cgroups=1, head_dim=64, latent_dim=128)
SHAPES = {
    "paper": PAPER,
    "heads32": dict(d_model=64, n_heads=8, n_qgroups=2, n_kgroups=2, n_cgroups=1, head_dim=32, latent_dim=64),
    "latent192": dict(d_model=192, n_heads=4, n_qgroups=2, n_kgroups=1, n_cgroups=1, head_dim=64, latent_dim=192),
    "latent256": dict(d_model=64, n_heads=4, n_qgroups=4, n_kgroups=2, n_cgroups=2, head_dim=64, latent_dim=256),
    "heads128": dict(d_model=64, n_heads=2, n_qgroups=2, n_kgroups=1, n_cgroups=1, head_dim=128, latent_dim=128),
}


def _wl(shape):
    return W.Workload(name=f"f32_{shape}", kind="prefill", batch=1, seqlen=64, dtype="f32", rope=True, seed=4300, **SHAPES[shape])


def _same(got, ref, what):
    finite = np.isfinite(ref)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref), what)
    np.testing.assert_array_equal(got[np.isinf(ref)], ref[np.isinf(ref)], what)
    U.assert_close(got[finite], ref[finite], "f32", what, max(1.0, float(np.abs(ref[finite]).max())))


@pytest.mark.parametrize("bad", [(97, 32), (70, 33), (40, 0), (33, 65)], ids=str)   # first padding token of the two sequences
@pytest.mark.parametrize("shape", list(SHAPES))
def test_prefill_with_uninitialised_padding(shape, bad):
    wl, n = _wl(shape), 100
    rng = W.make_rng(wl)
    w, x = W.draw_weights(wl, rng, std=wl.d_model ** -0.5), W.draw_hidden(wl, rng, 2 * n)
    for b in range(2):
        pad = x[b * n + bad[b]:(b + 1) * n]
        pad[:] = np.nan
        pad[1::2] = np.inf
    out = U.f64(U.run_prefill(wl, U.upload_weights(w, "f32"), x, batch=2))
    for b in range(2):
        rows = slice(b * n, b * n + bad[b])
        if bad[b]:
            ref, _, _ = orc.prefill_sequence(U.oracle_config(wl), U.oracle_weights(w), x[rows])
            U.assert_close(out[rows], ref, "f32", f"{shape} sequence {b}", max(1.0, float(np.abs(ref).max())))
        assert np.isnan(out[b * n + bad[b]:(b + 1) * n]).all()


@pytest.mark.parametrize("row", [0, 31, 37, 64, 99])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_infinite_latents(shape, row):
    """The attention stage alone: one latent row with an infinity and a NaN, the last row (re-read past the end) among them."""
    wl, n = _wl(shape), 100
    rng = np.random.default_rng(row)
    q, k, c = (rng.standard_normal((n, groups, width)).astype(np.float32) for groups, width in
               ((wl.n_qgroups, wl.head_dim), (wl.n_kgroups, wl.head_dim), (wl.n_cgroups, wl.latent_dim)))
    c[row, :, 3], c[row, :, -1], c[row, :, 20] = np.inf, -np.inf, np.nan
    cfg, dev = U.oracle_config(wl), [torch.from_numpy(a.reshape(n, -1)).cuda() for a in (q, k, c)]
    out = torch.empty((n, wl.n_qgroups * wl.latent_dim), device="cuda")
    B.gta_prefill_attention(B.config_of(wl), *dev, None, 1, n, n, out)
    got = U.f64(out).reshape(n, wl.n_qgroups, wl.latent_dim)
    for g in range(wl.n_qgroups):
        kg, cg = k[:, cfg.k_of_group(g)].astype(np.float64), c[:, cfg.c_of_group(g)].astype(np.float64)
        m = orc.attention_map_rows(cfg, q[:, g].astype(np.float64), np.arange(n), kg)
        with np.errstate(invalid="ignore"):
            ref = np.stack([m[i, :i + 1] @ cg[:i + 1] for i in range(n)])
        _same(got[:, g], ref, f"{shape} group {g}")


def _overflowing(groups, width, rows, bad):
    """q [1, 1, width] and keys [rows, groups, width] whose products are below -FLT_MAX for the rows `bad`, small elsewhere"""
    rng = np.random.default_rng(rows)
    k = rng.standard_normal((rows, groups, width)).astype(np.float32) * np.float32(1e-20)
    k[bad] = -1e20
    return np.full((1, 1, width), 1e20, dtype=np.float32), k


@pytest.mark.parametrize("block", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_prefill_block_of_overflowed_scores(shape, block):
    wl, n = _wl(shape), 150
    q, k = _overflowing(wl.n_kgroups, wl.head_dim, n, slice(32 * block, 32 * block + 32))
    q = np.broadcast_to(q, (n, wl.n_qgroups, wl.head_dim))
    c = np.random.default_rng(1).standard_normal((n, wl.n_cgroups, wl.latent_dim)).astype(np.float32)
    cfg, dev = U.oracle_config(wl), [torch.from_numpy(a.reshape(n, -1).copy()).cuda() for a in (q, k, c)]
    out = torch.empty((n, wl.n_qgroups * wl.latent_dim), device="cuda")
    B.gta_prefill_attention(B.config_of(wl), *dev, None, 1, n, n, out)
    got = U.f64(out).reshape(n, wl.n_qgroups, wl.latent_dim)
    first = 32 if block == 0 else 0                   # rows without any other key are 0 / 0
    for g in range(wl.n_qgroups):
        kg, cg = k[:, cfg.k_of_group(g)].astype(np.float64), c[:, cfg.c_of_group(g)].astype(np.float64)
        ref = orc.attention_map_rows(cfg, q[first:, g].astype(np.float64), np.arange(first, n), kg) @ cg
        U.assert_close(got[first:, g], ref, "f32", f"{shape} group {g}", max(1.0, float(np.abs(ref).max())))


def _decode_stage(wl, q, k, c, splits):
    """gta_decode_attention and gta_decode_combine on caches that hold k, c [batch, rows, width]"""
    batch, rows = k.shape[:2]
    cache = U.DeviceCache(wl, batch, rows, torch.from_numpy(k).cuda(), torch.from_numpy(c).cuda())
    cache.seq_lens.fill_(rows)
    cfg = B.config_of(wl)
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_DECODE, batch, 0, rows, splits))
    out = torch.empty((batch, wl.n_qgroups, wl.latent_dim), device="cuda")
    B.gta_decode_attention(cfg, torch.from_numpy(q.reshape(batch, -1).copy()).cuda(), cache.struct, None, batch, splits, ws)
    B.gta_decode_combine(cfg, cache.struct, None, batch, splits, ws, out)
    return U.f64(out)


@pytest.mark.parametrize("splits", [1, 5, 40])
@pytest.mark.parametrize("shape,first,last", [("paper", 0, 16), ("paper", 16, 32), ("paper", 48, 64), ("heads32", 0, 64)])   # blocks of 16, 64
def test_decode_step_of_overflowed_scores(shape, first, last, splits):
    wl, n = _wl(shape), 300
    q, k = _overflowing(wl.n_kgroups, wl.head_dim, n, slice(first, last))
    q = np.broadcast_to(q, (1, wl.n_qgroups, wl.head_dim))
    c = np.random.default_rng(2).standard_normal((n, wl.latent_dim)).astype(np.float32)
    got = _decode_stage(wl, q, k.reshape(1, n, -1), c[None], splits)
    cfg = U.oracle_config(wl)
    for g in range(wl.n_qgroups):
        kg = k[:, cfg.k_of_group(g)].astype(np.float64)
        ref = orc.attention_map_rows(cfg, q[:, g].astype(np.float64), np.array([n - 1]), kg) @ c.astype(np.float64)
        U.assert_close(got[:, g], ref, "f32", f"group {g}", max(1.0, float(np.abs(ref).max())))


@pytest.mark.parametrize("splits", [1, 5, 40])
@pytest.mark.parametrize("n", [1, 15, 16, 33, 300])
def test_decode_infinite_latent_in_the_newest_row(n, splits):
    """Rows past the end re-read the newest one with weight 0."""
    wl, rng = _wl("paper"), np.random.default_rng(n)
    q, k, c = (rng.standard_normal(s).astype(np.float32) for s in
               ((1, wl.n_qgroups, wl.head_dim), (1, n, wl.head_dim), (1, n, wl.latent_dim)))
    c[0, -1, 7], c[0, -1, 100], c[0, 0, 50] = np.inf, -np.inf, np.nan
    got = _decode_stage(wl, q, k, c, splits)
    for g in range(wl.n_qgroups):
        m = orc.attention_map_rows(U.oracle_config(wl), q[:, g].astype(np.float64), np.array([n - 1]), k[0].astype(np.float64))
        _same(got[:, g], m @ c[0].astype(np.float64), f"{n} rows, group {g}")


@pytest.mark.parametrize("splits", [1, 5, 40])          # 40: more than the one-round-trip tail takes
@pytest.mark.parametrize("dtype,gate", [("f32", True), ("f32", False), ("bf16", True)])
def test_decode_step_with_a_nan_key(dtype, gate, splits):
    """A sequence with a NaN among its keys has no result, the others (and a full slot) are not affected."""
    wl = W.scaled(_wl("paper"), dtype=dtype)
    rng, cap, batch = W.make_rng(wl), 300, 4
    w, x = W.draw_weights(wl, rng, std=wl.d_model ** -0.5), W.draw_hidden(wl, rng, batch)
    k, c = W.draw_cache(wl, rng, batch, cap)
    k[1, 20] = np.nan
    cache = U.DeviceCache(wl, batch, cap, *(torch.from_numpy(a).to("cuda", torch.float32 if dtype == "f32" else torch.bfloat16) for a in (k, c)))
    cache.seq_lens.copy_(torch.tensor([250, 250, 17, cap], dtype=torch.int32))
    out = U.f64(U.run_decode(wl, U.upload_weights(w, dtype), x, cache, num_splits=splits, gate=gate))
    assert np.isnan(out[1]).all() and not out[3].any()
    lens, status = np.array([250, 250, 17, cap], dtype=np.int32), np.zeros(batch, dtype=np.int32)
    with np.errstate(invalid="ignore"):
        ref = orc.decode(U.oracle_config(wl, gate), U.oracle_weights(w), x, k.astype(np.float64), c.astype(np.float64), lens, status, range(batch))
    for b in (0, 2):
        U.assert_close(out[b], ref[b], dtype, f"sequence {b}", max(1.0, float(np.abs(ref[b]).max())))
