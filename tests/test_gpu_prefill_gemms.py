"""The prefill's GEMMs at the edges of their tiles: the few-row kernel, the 64-row tiles that split K over their waves
(three stages of 64: contractions of one, two and more) and the stream of 256 x 256 tiles (eight waves; X in three stages of 64, weights in
four of 32).  One valid row in the last row tile and full row tiles, contractions that leave the stages at each phase, two heads side by side in a weight tile, several heads and one, the packed weights, every gate.

Reference: float64 on the same bf16 inputs.  Bounds: the bf16 tolerances of the parity gate, the max-abs one scaled by
the largest reference value (the outputs carry one bf16 rounding, 2^-9 of their size)."""
import numpy as np
import pytest
import torch

import gpu_util as U
from paper_2506_17286_amd import binding as B, workloads as W

pytestmark = pytest.mark.gpu


def _wl(**kw):
    base = dict(name="big", kind="prefill", batch=1, seqlen=64, d_model=256, n_heads=4, n_qgroups=2, n_kgroups=2, n_cgroups=1,
                head_dim=128, latent_dim=256, dtype="bf16", rope=True, seed=6100)
    return W.Workload(**dict(base, **kw))


def _close(got, ref, what):
    r = ref.cpu().numpy()
    U.assert_close(U.f64(got), r, "bf16", what, max(1.0, float(np.abs(r).max())))


LAYERS = {
    "k256": _wl(), "k384": _wl(d_model=384, latent_dim=384), "k640": _wl(d_model=640, n_heads=8, latent_dim=512),
    "k128": _wl(d_model=128), "slim": _wl(head_dim=64, n_heads=8, n_qgroups=4, latent_dim=64),
    "packed": _wl(head_dim=64, n_heads=20, n_qgroups=5, n_kgroups=1, latent_dim=128, d_model=256),
    "multi128": _wl(latent_dim=128), "single128": _wl(n_qgroups=4, latent_dim=128),   # several heads of 128 per tile, one
}


@pytest.mark.parametrize("gate", [True, False])
@pytest.mark.parametrize("rows", [33, 64, 65, 449, 24832, 24833])
@pytest.mark.parametrize("layer", list(LAYERS))
def test_prefill_gemms(layer, rows, gate):
    _check(LAYERS[layer], rows, gate)


@pytest.mark.parametrize("gate", ["silu", "relu2"])
@pytest.mark.parametrize("rows", [65, 24833])
@pytest.mark.parametrize("layer", list(LAYERS))
def test_other_gates(layer, rows, gate):
    _check(LAYERS[layer], rows, gate)


@pytest.mark.parametrize("layer,rows", [("packed", 576), ("packed", 577), ("k256", 1600), ("k256", 1601)])
def test_second_tile_on_a_cu(layer, rows):
    """252 and 280 tiles of 64 x 64, 250 and 260 of 64 x 128 in the projection: two stages a step or one."""
    _check(LAYERS[layer], rows, True)


@pytest.mark.parametrize("rows", [3200, 3201])
def test_packed_weights_of_long_contractions(rows):
    """Heads of 128, 2048 rows of packed weights: 700 tiles of 64 x 128, the last on those, and 714, the first on 256 x 256 tiles."""
    _check(_wl(d_model=2048, n_heads=8, n_qgroups=4, n_kgroups=1, latent_dim=128), rows, True)


@pytest.mark.parametrize("layer,rows", [("k256", 3264), ("k256", 3265), ("k256", 4993), ("k256", 13057), ("k256", 19457), ("packed", 9345),
                                        ("packed", 13825), ("ten", 11137)])
def test_rounds_of_tiles(layer, rows):
    """510 and 520 tiles of 64 x 128 in the projection: the last on those, the first on 256 x 256 tiles.  256 x 256 tiles on 256 CUs:
    100: less than a round, every tile shared by two workgroups; 260: a round and four to
    share, of the last strip's one row only the first half exists; 385: 129 behind the round are too many to share; 7 columns
    in panels of 4 and 3, 259 and 385 tiles; 10 columns in panels of 4, 4 and 2, a last band of 4 strips, 440 tiles."""
    _check(dict(LAYERS, ten=_wl(n_heads=12, latent_dim=512))[layer], rows, True)


ROTATED = {"packed64": _wl(head_dim=64, n_heads=20, n_qgroups=5, n_kgroups=1, latent_dim=128), "packed128": _wl(n_heads=10, n_qgroups=5, n_kgroups=1),
           "matrices": _wl()}


@pytest.mark.parametrize("layer", list(ROTATED))
def test_rotation_bits(layer):
    """Rows of X with a single one give weights as values before the rotation, exactly, and the rotation is one product rounded to fp32
    and one fused multiply-add.  Which product comes first is part of the result's last fp32 bit: hi cos first against packed
    weights, lo sin first against the four matrices."""
    wl, rows = ROTATED[layer], 9000
    H, dh, nq, nk, nh, dl = wl.d_model, wl.head_dim, wl.n_qgroups, wl.n_kgroups, wl.n_heads, wl.latent_dim
    g = torch.Generator(device="cuda")
    g.manual_seed(wl.seed)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    w = {"wq": rand(H, nq * dh), "wk": rand(H, nk * dh), "wc": rand(H, dl), "wg": rand(H, nh * dh), "wp": rand(nh, dl, dh), "wo": None}
    at = torch.arange(rows, device="cuda") % H
    x = torch.zeros((rows, H), dtype=torch.bfloat16, device="cuda")
    x[torch.arange(rows, device="cuda"), at] = 1.
    mk = lambda n: torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    out = {"q": mk(nq * dh), "k": mk(nk * dh), "c": mk(dl), "g": mk(nh * dh)}
    cfg = B.config_of(wl)
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_PREFILL, 1, rows, rows))
    B.gta_prefill_projection(cfg, B.make_weights(w), x, None, 1, rows, rows, out["q"], out["k"], out["c"], out["g"], ws)
    ang = torch.arange(rows, device="cuda", dtype=torch.float64)[:, None] * \
        wl.rope_base ** (-torch.arange(dh // 2, device="cuda", dtype=torch.float64) * 2 / dh)
    c, s = ang.cos().float()[:, None], ang.sin().float()[:, None]
    fma = lambda a, b, z: (a.double() * b.double() + z.double()).float()   # the product is exact
    for name, groups in (("q", nq), ("k", nk)):
        lo, hi = w["w" + name][at].float().view(rows, groups, dh).split(dh // 2, dim=-1)
        ref = torch.cat([fma(lo, c, -(hi * s)), fma(hi, c, lo * s) if layer == "matrices" else fma(lo, s, hi * c)], dim=-1)
        ref = ref.bfloat16().view(rows, -1)
        # a cosine or sine may lie next to a tie of its own rounding to fp32 (2^-29 of them, as its 64-bit error), and so may a result
        assert int((out[name] != ref).sum()) <= 2, f"{name}: {int((out[name] != ref).sum())} of {ref.numel()} differ"
    for name in ("c", "g"):
        assert torch.equal(out[name], w["w" + name][at])


@pytest.mark.parametrize("rows", [100, 1400, 2700, 9000])
def test_infinite_weights_stay_in_their_columns(rows):
    """Q and K end in the middle of a wave's 128 columns (320 of 256 + 64), so that latent columns go through the rotation's
    epilogue: a column of infinities must not reach the one that would be its partner.  24, 264, 516 and 1692 tiles of 64 x 128."""
    wl = _wl(head_dim=64, n_heads=16, n_qgroups=4, n_kgroups=1, latent_dim=128)
    H, dh, nq, nk, nh, dl = wl.d_model, wl.head_dim, wl.n_qgroups, wl.n_kgroups, wl.n_heads, wl.latent_dim
    g = torch.Generator(device="cuda")
    g.manual_seed(wl.seed + rows)
    rand = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).bfloat16()
    w = {"wq": rand(H, nq * dh, std=H ** -0.5), "wk": rand(H, nk * dh, std=H ** -0.5), "wc": rand(H, dl, std=H ** -0.5),
         "wg": rand(H, nh * dh, std=H ** -0.5), "wp": rand(nh, dl, dh), "wo": None}
    x = rand(rows, H).abs() + 1.
    w["wc"][3, 5] = w["wc"][7, 40] = float("inf")
    w["wg"][9, 70] = float("-inf")
    mk = lambda n: torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    out = {"q": mk(nq * dh), "k": mk(nk * dh), "c": mk(dl), "g": mk(nh * dh)}
    cfg = B.config_of(wl)
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_PREFILL, 1, rows, rows))
    B.gta_prefill_projection(cfg, B.make_weights(w), x, None, 1, rows, rows, out["q"], out["k"], out["c"], out["g"], ws)
    inf = {"q": {}, "k": {}, "c": {5: float("inf"), 40: float("inf")}, "g": {70: float("-inf")}}
    for name in ("c", "g"):
        for col, v in inf[name].items():
            assert bool((out[name][:, col] == v).all()), f"{name} column {col}"
        rest = [i for i in range(out[name].shape[1]) if i not in inf[name]]
        _close(out[name][:, rest], x.double() @ w["w" + name][:, rest].double(), name)
    assert torch.isfinite(out["q"].float()).all() and torch.isfinite(out["k"].float()).all()


def _check(wl, rows, gate):
    cfg = B.config_of(wl)
    cfg.gate = B.GATE_CODES[gate]
    g = torch.Generator(device="cuda")
    g.manual_seed(wl.seed + rows)
    rand = lambda *s, std=1.0: (torch.randn(s, generator=g, device="cuda") * std).bfloat16()
    H, dh, dl, nq, nk, nh = wl.d_model, wl.head_dim, wl.latent_dim, wl.n_qgroups, wl.n_kgroups, wl.n_heads
    w = {"wq": rand(H, nq * dh, std=H ** -0.5), "wk": rand(H, nk * dh, std=H ** -0.5), "wc": rand(H, dl, std=H ** -0.5),
         "wg": rand(H, nh * dh, std=H ** -0.5), "wp": rand(nh, dl, dh, std=dl ** -0.5), "wo": rand(nh * dh, H, std=(nh * dh) ** -0.5)}
    gw, x = B.make_weights(w), rand(rows, H)
    mk = lambda n: torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    out = {"q": mk(nq * dh), "k": mk(nk * dh), "c": mk(dl), "g": mk(nh * dh)}
    ws = B.alloc_workspace(B.gta_workspace_bytes(cfg, B.GTA_MODE_PREFILL, 1, rows, rows))
    B.gta_prefill_projection(cfg, gw, x, None, 1, rows, rows, out["q"], out["k"], out["c"], out["g"], ws)
    ang = torch.arange(rows, device="cuda", dtype=torch.float64)[:, None] * \
        wl.rope_base ** (-torch.arange(dh // 2, device="cuda", dtype=torch.float64) * 2 / dh)
    for name, groups in (("q", nq), ("k", nk), ("c", 0), ("g", 0)):
        ref = x.double() @ w["w" + name].double()
        if groups:
            lo, hi = ref.view(rows, groups, dh).split(dh // 2, dim=-1)
            c, s = ang.cos()[:, None], ang.sin()[:, None]
            ref = torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1).reshape(rows, -1)
        _close(out[name], ref, name)
    L, z, heads = rand(rows, nq * dl), rand(rows, nh * dh), mk(nh * dh)
    B.gta_prefill_decoder(cfg, gw, L, z, rows, heads)
    ref = torch.cat([L[:, h // (nh // nq) * dl:][:, :dl].double() @ w["wp"][h].double() for h in range(nh)], dim=1)
    zd = z.double()
    _close(heads, ref * {True: torch.sigmoid(zd), False: 1., "silu": zd * torch.sigmoid(zd), "relu2": zd.clamp(min=0.) ** 2}[gate],
           "decoder")
    o = mk(H)
    B.gta_output_projection(cfg, gw, heads, rows, o)
    _close(o, heads.double() @ w["wo"].double(), "output projection")
