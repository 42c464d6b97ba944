"""The table scatter's pair lists (pair_lists.h): every kind of list level (tight and loose
hashed tiles, modulo hashing, dense levels dealt line by line), levels with too many tiles
for lists (masks), chunk and batch boundaries, one and two corner sets, against the
oracle; and, on the CPU, the rule that keeps every call that fits the static workspace
within it."""
import numpy as np
import pytest

from oracle import hash4d_oracle as O
from paper_2507_19141_amd import _lib, synth
from tests.util import RTOL_GRAD, mlp_backward_scale, needs_gpu, scaled_close

# name: (F, space resolutions, time resolutions, T)
GRIDS = {
    "tight": (2, [40, 128], [8, 30], 1 << 14),
    "loose": (2, [300, 2048], [9, 20], 1 << 12),          # 2 N_s above the 256 rows of a tile
    "loose_f1": (1, [2047], [3], 1 << 11),
    "modulo": (2, [16, 33], [5, 9], 5003),                # T no power of two
    "dense": (2, [1, 3, 7], [1, 2, 5], 1 << 13),          # 8 .. 384 lines
    "dense_32": (4, [31], [3], 1 << 17),                  # lines a multiple of 32 long
    "mixed": (8, [3, 31, 600], [4, 7, 11], 1 << 13),
    "masks": (8, [512], [40], 1 << 21),                   # 512 tiles: no lists
}


def _inputs(n, seed, crowded):
    rng = np.random.default_rng(seed)
    x = synth.uniform_xyzt(n, rng)
    if crowded:  # every query in a few cells, one timestamp
        x = (0.5 + 0.01 * (x - 0.5)).astype(np.float32)
        x[:, 3] = np.float32(0.25)
    edges = np.array([[0, 0, 0, 0], [1, 1, 1, 1], [np.nan, 0.5, 2.0, -1.0], [0.25, 0.5, 0.75, 1.0]], np.float32)
    x[: min(n, 4)] = edges[: min(n, 4)]
    return rng, x


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [_lib.F32, _lib.F64], ids=["f32", "f64"])
@pytest.mark.parametrize("name", GRIDS)
@pytest.mark.parametrize("n,crowded", [(1, False), (513, False), (2048, True), (4097, False)])
def test_scatter_every_list_kind(name, dt, n, crowded):
    needs_gpu()
    import torch
    F, rs, rt, T = GRIDS[name]
    L = len(rs)
    og = O.make_grid(L, F, rs, rt, T)
    lg = _lib.h4d_grid_init(L, F, rs, rt, T)
    rng, x = _inputs(n, 7 * n + len(name), crowded)
    gf = synth.upstream(n, L * F, rng)
    real = np.float64 if dt == _lib.F64 else np.float32
    wb = _lib.hash4d_encode_backward_workspace_bytes(lg, n)
    ws = torch.full((wb,), 0xA5, dtype=torch.uint8, device="cuda")   # nothing is read before it is written
    d_table = torch.full((og.E, F), float("nan"), dtype=torch.float64 if dt == _lib.F64 else torch.float32,
                         device="cuda")
    _lib.hash4d_encode_backward(lg, dt, _dev(x), n, _dev(gf.astype(real)), 0.5, d_table, ws, wb,
                                _lib.QUERY_MAJOR | _lib.GRAD_OVERWRITE)
    torch.cuda.synchronize()
    scaled_close(d_table.cpu().numpy(), O.encode_backward(x, gf, og, 0.5), O.encode_backward(x, np.abs(gf), og, 0.5),
                 1e-12 if dt == _lib.F64 else RTOL_GRAD, f"{name} n={n}")


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["tight", "loose", "modulo", "dense", "mixed", "masks"])
@pytest.mark.parametrize("n,sigma", [(1, 1e-3), (1025, 1e-4), (2049, 5e-2)])
def test_two_corner_sets(name, n, sigma):
    # x and x + eps in one cell (one entry for both) and apart (one entry each)
    needs_gpu()
    import torch
    F, rs, rt, T = GRIDS[name]
    L = len(rs)
    og = O.make_grid(L, F, rs, rt, T)
    lg = _lib.h4d_grid_init(L, F, rs, rt, T)
    rng, x = _inputs(n, n + len(name), False)
    table = synth.table_init(og.E, F, rng)
    eps = synth.perturbation(n, rng, sigma)
    gf = synth.upstream(n, L * F, rng)
    loss = torch.zeros(1, device="cuda")
    d_table = torch.full((og.E, F), float("nan"), device="cuda")
    wb = _lib.smoothness_workspace_bytes(lg, _lib.F32, n)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    _lib.hash4d_encode_backward_smooth(lg, _lib.F32, _dev(table), _dev(x), _dev(eps), n, _dev(gf), 0.5, 2.0, loss,
                                       d_table, ws, wb, _lib.QUERY_MAJOR | _lib.GRAD_OVERWRITE)
    torch.cuda.synchronize()
    xp = O.perturbed(x, eps)
    d = np.abs(O.encode(x, table, og) - O.encode(xp, table, og))
    s = O.encode(x, np.abs(table), og) + O.encode(xp, np.abs(table), og)
    g = 4.0 / n * (d + s)
    scale = O.encode_backward(x, g + 0.5 * np.abs(gf), og) + O.encode_backward(xp, g, og)
    ref = O.smoothness(x, eps, table, og, 2.0)[1] + O.encode_backward(x, gf, og, 0.5)
    scaled_close(d_table.cpu().numpy(), ref, scale, RTOL_GRAD, f"{name} n={n} sigma={sigma}")


@pytest.mark.gpu
def test_more_chunks_than_one_round():
    # 2^21 + 4001 queries: more chunks than the walk holds at a time
    needs_gpu()
    import torch
    og = O.make_grid(1, 1, [24], [6], 1 << 15)
    lg = _lib.h4d_grid_init(1, 1, [24], [6], 1 << 15)
    n = (1 << 21) + 4001
    rng = np.random.default_rng(5)
    x = synth.uniform_xyzt(n, rng)
    gf = synth.upstream(n, 1, rng)
    wb = _lib.hash4d_encode_backward_workspace_bytes(lg, n)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    d_table = torch.full((og.E, 1), float("nan"), device="cuda")
    _lib.hash4d_encode_backward(lg, _lib.F32, _dev(x), n, _dev(gf), 1.0, d_table, ws, wb, _lib.GRAD_OVERWRITE)
    torch.cuda.synchronize()
    scaled_close(d_table.cpu().numpy(), O.encode_backward(x, gf, og), O.encode_backward(x, np.abs(gf), og), RTOL_GRAD)


def _static_rule(L, F, rs, rt, T, n):
    """Bytes by which the static-workspace entry point has always decided: a mask and a
    word per (query, level), counts per chunk of 1024, a plan and partial tiles."""
    al = lambda b: (b + 255) // 256 * 256  # noqa: E731
    rows = [min((s + 1) ** 3 * (t + 1), T) for s, t in zip(rs, rt)]
    tiles = slot = 0
    for gb in (4, 8):
        mx, count = 131072 // (F * gb), 0
        for r in rows:
            sh = 8
            while (1 << sh) < mx and (1 << sh) < -(-r // 32):
                sh += 1
            count += (r + (1 << sh) - 1) >> sh
            slot = max(slot, min(1 << sh, r) * F * gb)
        tiles = max(tiles, count)
    pad, chunks, extra = (n + 3) // 4 * 4, (n + 1023) // 1024, min(96, max(8, tiles // 4))
    return (al(pad * L * 4) + al(pad * L * 8) + al(L * chunks * 128) + al((tiles + extra) * 16) + 256 + al(extra * 4)
            + 2 * extra * slot)


@pytest.mark.parametrize("case", [("paper", 16, 2, (16, 2048), (16, 150), 1 << 19),
                                  ("small", 4, 2, (4, 32), (4, 16), 1 << 12),
                                  ("hashed", 32, 2, (64, 2048), (16, 150), 1 << 19),
                                  ("one_level", 1, 4, (200, 200), (30, 30), 1 << 16),
                                  ("loose", 8, 2, (300, 2048), (16, 64), 1 << 13),
                                  ("modulo", 8, 8, (16, 512), (16, 64), 300_007),
                                  ("dense", 3, 8, (2, 8), (2, 8), 1 << 20)], ids=lambda c: c[0])
def test_static_workspace_takes_what_it_took(case):
    # hash4d_encode_backward_noalloc accepts a call iff its workspace fits 64 MiB: every
    # call that fits by the earlier rule still does, up to the largest of them
    _, L, F, sp, tm, T = case
    rs, rt = O.level_resolutions(*sp, L), O.level_resolutions(*tm, L)
    lg = _lib.h4d_grid_init(L, F, rs, rt, T)
    lo, hi = 1, 1 << 27
    while lo < hi:  # the largest n within the earlier rule
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if _static_rule(L, F, rs, rt, T, mid) <= 64 << 20 else (lo, mid - 1)
    for n in {1, 100, 4096, 60_000, lo // 3, lo - 1, lo}:
        if 1 <= n <= lo:
            assert _lib.hash4d_encode_backward_workspace_bytes(lg, n) <= 64 << 20, n


@pytest.mark.gpu
@pytest.mark.parametrize("F,names,ns", [(2, ("loose", "modulo", "dense"), (2049, 1, 4100)), (8, ("mixed", "masks"), (700, 300)),
                                        (1, ("loose_f1",), (5000,))], ids=["f2", "f8", "f1"])
@pytest.mark.parametrize("zero", [False, True], ids=["accumulate", "zero_grads"])
def test_batched_scatter_over_segments(F, names, ns, zero):
    # a scene's timestamps are one run of chunks; with ZERO_GRADS every gradient is written
    needs_gpu()
    import torch
    L = max(2, 8 // F)          # a decoder input of 8 or 16
    scenes, descs = [], []
    for i, (name, n) in enumerate(zip(names, ns)):
        f, rs, rt, T = GRIDS[name]
        rs, rt = (rs * L)[:L], (rt * L)[:L]
        og, lg = O.make_grid(L, F, rs, rt, T), _lib.h4d_grid_init(L, F, rs, rt, T)
        rng, x = _inputs(n, 90 + i, i == 1)
        x = np.clip(np.nan_to_num(x), 0, 1).astype(np.float32)
        times = [0.0, 1.0 / 3, 1.0][: 3 - i % 2]
        table = synth.table_init(og.E, F, rng)
        params = synth.decoder_params(L * F, rng)
        gd = synth.upstream(n * len(times), 10, rng).reshape(len(times), n, 10)
        init = float("nan") if zero else 0.0
        s = {"og": og, "x": x, "times": times, "table": table, "params": params, "gd": gd,
             "xyz": _dev(x), "table_d": _dev(table), "params_d": _dev(params), "gd_d": _dev(gd),
             "feat": torch.empty((len(times), L, n, F), device="cuda"),
             "delta": torch.empty((len(times), n, 10), device="cuda"),
             "d_table": torch.full((og.E, F), init, device="cuda"),
             "d_params": torch.full((params.size,), init, device="cuda")}
        scenes.append(s)
        descs.append(_lib.scene_desc(lg, n, s["xyz"], times, s["table_d"], s["params_d"], s["feat"], s["delta"],
                                     s["gd_d"], s["d_table"], s["d_params"]))
    flags = _lib.PLAN_GRAPH | (_lib.PLAN_ZERO_GRADS if zero else 0)
    plan = _lib.BatchedPlan(descs, _lib.mlp_shape(L * F), _lib.F32, 1.0, flags)
    plan.run()
    torch.cuda.synchronize()
    for i, s in enumerate(scenes):
        ref, scale = np.zeros((s["og"].E, F)), np.zeros((s["og"].E, F))
        for k, t in enumerate(s["times"]):
            xt = s["x"].copy()
            xt[:, 3] = np.float32(t)
            f_ref = O.encode(xt, s["table"], s["og"])
            ref += O.deform_backward(xt, s["table"], s["og"], s["params"], s["gd"][k])[0]
            sf, _ = mlp_backward_scale(s["params"], f_ref, s["gd"][k])
            scale += O.encode_backward(xt, sf, s["og"])
        scaled_close(s["d_table"].cpu().numpy(), ref, scale, RTOL_GRAD, f"scene {i}")
    plan.destroy()


# ---- workspace and passes ----
WS_GRIDS = {  # L, F, space, time, T
    "small_T": (16, 2, (16, 2048), (16, 150), 1 << 14),
    "paper": (16, 2, (16, 2048), (16, 150), 1 << 19),
    "loose": (8, 1, (300, 2048), (9, 20), 1 << 12),
    "many_levels": (32, 1, (4, 2048), (4, 64), 1 << 13),
    "one_level": (1, 2, (30, 30), (16, 16), 1 << 19),
    "masks": (1, 8, (512, 512), (40, 40), 1 << 21),
}


def _ws_grid(name):
    L, F, sp, tm, T = WS_GRIDS[name]
    return _lib.h4d_grid_init(L, F, O.level_resolutions(*sp, L), O.level_resolutions(*tm, L), T)


@pytest.mark.parametrize("name", WS_GRIDS)
def test_workspace_never_shrinks(name):
    # a workspace sized for the largest cloud serves every smaller one
    lg = _ws_grid(name)
    m = _lib.mlp_shape(lg.L * lg.F) if lg.L * lg.F in (8, 16, 32, 64) else None
    ns = sorted({1, 2, 5, 7, 511, 512, 513, 2047, 2048, 2049} | set(range(1000, 600_000, 499)) | {1 << 21, 6_000_000})
    for ws in (lambda n: _lib.hash4d_encode_backward_workspace_bytes(lg, n),
               lambda n: _lib.smoothness_workspace_bytes(lg, _lib.F32, n),
               lambda n: _lib.hash4d_deform_workspace_bytes(lg, m, _lib.F32, n) if m else 0):
        sizes = [ws(n) for n in ns]
        drops = [(a, b) for a, b, x, y in zip(ns, ns[1:], sizes, sizes[1:]) if y < x]
        assert not drops, drops[:3]


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["noalloc", "workspace"])
@pytest.mark.parametrize("overwrite", [False, True], ids=["accumulate", "overwrite"])
def test_scatter_in_several_passes(form, overwrite):
    # lists of all levels past the bytes at hand: shares of the levels one after the other,
    # every row and every non-finite value written once
    needs_gpu()
    import torch
    L, F, sp, tm, T = WS_GRIDS["many_levels"]
    rs, rt = O.level_resolutions(*sp, L), O.level_resolutions(*tm, L)
    og, lg = O.make_grid(L, F, rs, rt, T), _ws_grid("many_levels")
    n = 140_001
    rng, x = _inputs(n, 61, False)
    gf = synth.upstream(n, L * F, rng)
    base = synth.table_init(og.E, F, rng, scale=1e-3)
    d_table = _dev(np.full_like(base, np.nan) if overwrite else base)
    layout = _lib.QUERY_MAJOR | (_lib.GRAD_OVERWRITE if overwrite else 0)
    ref, scale = O.encode_backward(x, gf, og, 0.5), O.encode_backward(x, np.abs(gf), og, 0.5)
    wb = _lib.hash4d_encode_backward_workspace_bytes(lg, n)
    assert wb == 64 << 20   # what the static workspace holds, less than all lists take
    if form == "noalloc":
        _lib.hash4d_encode_backward_noalloc(lg, _lib.F32, _dev(x), n, _dev(gf), 0.5, d_table, layout)
    else:
        ws = torch.full((wb,), 0xA5, dtype=torch.uint8, device="cuda")
        bad = torch.zeros(1, dtype=torch.int32, device="cuda")
        gbad = gf.copy()
        gbad[777, 5], gbad[778, 30] = np.nan, np.inf
        d2 = d_table.clone()
        _lib.hash4d_encode_backward_checked(lg, _lib.F32, _dev(x), n, _dev(gbad), 0.5, d2, ws, wb, bad, layout)
        assert int(bad.item()) == int((~torch.isfinite(d2)).sum().item()) > 0
        _lib.hash4d_encode_backward(lg, _lib.F32, _dev(x), n, _dev(gf), 0.5, d_table, ws, wb, layout)
    torch.cuda.synchronize()
    if not overwrite:
        ref, scale = ref + base, scale + np.abs(base)
    scaled_close(d_table.cpu().numpy(), ref, scale, RTOL_GRAD, f"{form} n={n}")


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [_lib.F32, _lib.F64], ids=["f32", "f64"])
@pytest.mark.parametrize("pair", [False, True], ids=["one_set", "two_sets"])
@pytest.mark.parametrize("overwrite", [False, True], ids=["accumulate", "overwrite"])
def test_lists_beside_masks(dt, pair, overwrite):
    # a dense and a tight level with lists around two levels with more tiles than lists
    # have: each kernel skips the other's tiles, the second mask level has the second masks
    needs_gpu()
    import torch
    L, F, T, n = 5, 8, 1 << 21, 3000
    rs, rt = [512, 3, 600, 31, 24], [40, 4, 30, 7, 19]
    og, lg = O.make_grid(L, F, rs, rt, T), _lib.h4d_grid_init(L, F, rs, rt, T)
    assert lg.dense_list() == [False, True, False, True, True]
    rng, x = _inputs(n, 71, False)
    real = np.float64 if dt == _lib.F64 else np.float32
    gf = synth.upstream(n, L * F, rng)
    base = synth.table_init(og.E, F, rng, scale=1e-3)
    d_table = _dev(np.full(base.shape, np.nan, real) if overwrite else base.astype(real))
    layout = _lib.QUERY_MAJOR | (_lib.GRAD_OVERWRITE if overwrite else 0)
    ref, scale = O.encode_backward(x, gf, og, 0.5), O.encode_backward(x, np.abs(gf), og, 0.5)
    if pair:
        table, eps = synth.table_init(og.E, F, rng), synth.perturbation(n, rng, 1e-3)
        loss = torch.zeros(1, dtype=torch.float64 if dt == _lib.F64 else torch.float32, device="cuda")
        wb = _lib.smoothness_workspace_bytes(lg, dt, n)
        ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
        _lib.hash4d_encode_backward_smooth(lg, dt, _dev(table.astype(real)), _dev(x), _dev(eps), n,
                                           _dev(gf.astype(real)), 0.5, 2.0, loss, d_table, ws, wb, layout)
        xp = O.perturbed(x, eps)
        d = np.abs(O.encode(x, table, og) - O.encode(xp, table, og))
        s = 4.0 / n * (d + O.encode(x, np.abs(table), og) + O.encode(xp, np.abs(table), og))
        scale = O.encode_backward(x, s + 0.5 * np.abs(gf), og) + O.encode_backward(xp, s, og)
        ref = ref + O.smoothness(x, eps, table, og, 2.0)[1]
    else:
        wb = _lib.hash4d_encode_backward_workspace_bytes(lg, n)
        ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
        _lib.hash4d_encode_backward(lg, dt, _dev(x), n, _dev(gf.astype(real)), 0.5, d_table, ws, wb, layout)
    torch.cuda.synchronize()
    if not overwrite:
        ref, scale = ref + base, scale + np.abs(base)
    scaled_close(d_table.cpu().numpy(), ref, scale, 1e-12 if dt == _lib.F64 else RTOL_GRAD, f"pair={pair}")


@pytest.mark.parametrize("name", WS_GRIDS)
@pytest.mark.parametrize("n", [5, 100, 1000])
def test_workspace_of_few_queries(name, n):
    # the lists take what the queries can fill: 16 bytes per (query, level), twice that for
    # two corner sets or pairs that straddle tiles, and a head per tile
    lg = _ws_grid(name)
    tiles = 4 * 256 * lg.L + 512
    assert _lib.hash4d_encode_backward_workspace_bytes(lg, n) <= 32 * n * lg.L + tiles
    d = (4 * n * lg.L * lg.F + 255) // 256 * 256
    assert _lib.smoothness_workspace_bytes(lg, _lib.F32, n) - d <= 64 * n * lg.L + 2 * tiles


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["encode", "smooth", "encode_smooth", "deform"])
def test_workspace_of_the_former_size(entry):
    # the size reported before the scatter sorted pairs is still taken, one byte less is not
    needs_gpu()
    import torch
    L, F, sp, tm, T = WS_GRIDS["many_levels"]
    rs, rt = O.level_resolutions(*sp, L), O.level_resolutions(*tm, L)
    og, lg = O.make_grid(L, F, rs, rt, T), _ws_grid("many_levels")
    n = 9_001
    rng, x = _inputs(n, 83, False)
    gf, table = synth.upstream(n, L * F, rng), synth.table_init(og.E, F, rng)
    eps = synth.perturbation(n, rng, 1e-3)
    former = _static_rule(L, F, rs, rt, T, n)
    al = lambda b: (b + 255) // 256 * 256  # noqa: E731
    xd, loss, d_table = _dev(x), torch.zeros(1, device="cuda"), torch.zeros((og.E, F), device="cuda")
    xp = O.perturbed(x, eps)
    s = 4.0 / n * (np.abs(O.encode(x, table, og) - O.encode(xp, table, og)) + O.encode(x, np.abs(table), og)
                   + O.encode(xp, np.abs(table), og))
    if entry == "encode":
        assert _lib.hash4d_encode_backward_workspace_bytes(lg, n) > former
        wb, call = former, lambda ws, b: _lib.hash4d_encode_backward(lg, _lib.F32, xd, n, _dev(gf), 1.0, d_table, ws, b)
        ref, scale = O.encode_backward(x, gf, og), O.encode_backward(x, np.abs(gf), og)
    elif entry == "deform":
        m, params = _lib.mlp_shape(L * F), synth.decoder_params(L * F, rng)
        gd, feat, delta = synth.upstream(n, 10, rng), torch.empty((L, n, F), device="cuda"), torch.empty((n, 10), device="cuda")
        pd, d_params = _dev(params), torch.zeros(params.size, device="cuda")
        _lib.hash4d_deform_forward(lg, m, _lib.F32, _dev(table), pd, xd, n, feat, delta)
        rows = min(256, ((n + 15) // 16 + 7) // 8)      # decoder partials of eight tiles each
        wb = al(rows * params.size * 4) + al(4 * n * L * F) + former
        call = lambda ws, b: _lib.hash4d_deform_backward(lg, m, _lib.F32, pd, xd, n, feat, _dev(gd), 1.0, 1.0,  # noqa: E731
                                                         d_table, d_params, ws, b)
        ref = O.deform_backward(x, table, og, params, gd)[0]
        scale = O.encode_backward(x, mlp_backward_scale(params, O.encode(x, table, og), gd)[0], og)
    else:
        wb = al(4 * n * L * F) + former
        assert _lib.smoothness_workspace_bytes(lg, _lib.F32, n) > wb
        ref = O.smoothness(x, eps, table, og, 2.0)[1]
        scale = O.encode_backward(x, s, og) + O.encode_backward(xp, s, og)
        if entry == "smooth":
            call = lambda ws, b: _lib.smoothness_reg(lg, _lib.F32, _dev(table), xd, _dev(eps), n, 2.0, loss, d_table,  # noqa: E731
                                                     ws, b)
        else:
            call = lambda ws, b: _lib.hash4d_encode_backward_smooth(lg, _lib.F32, _dev(table), xd, _dev(eps), n,  # noqa: E731
                                                                    _dev(gf), 1.0, 2.0, loss, d_table, ws, b)
            ref, scale = ref + O.encode_backward(x, gf, og), scale + O.encode_backward(x, np.abs(gf), og)
    ws = torch.full((wb,), 0xA5, dtype=torch.uint8, device="cuda")
    with pytest.raises(_lib.H4DError, match="workspace"):
        call(ws, wb - 1)
    call(ws, wb)
    torch.cuda.synchronize()
    scaled_close(d_table.cpu().numpy(), ref, scale, RTOL_GRAD, entry)


@pytest.mark.gpu
@pytest.mark.parametrize("batches", [1, 2, 3, 63, 64, 65, 128])
def test_walk_ranges_of_whole_descriptions(batches):
    # eight tiles that every query reaches once: `batches` batches of 64 entries for each of
    # a tile's 16 wavefronts, up to the end of what a wavefront describes at a time
    needs_gpu()
    import torch
    og, lg = O.make_grid(1, 2, [1], [1], 16), _lib.h4d_grid_init(1, 2, [1], [1], 16)
    n = 64 * 16 * batches
    rng = np.random.default_rng(batches)
    x = synth.uniform_xyzt(n, rng)
    gf = synth.upstream(n, 2, rng)
    wb = _lib.hash4d_encode_backward_workspace_bytes(lg, n)
    ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
    d_table = torch.full((og.E, 2), float("nan"), device="cuda")
    _lib.hash4d_encode_backward(lg, _lib.F32, _dev(x), n, _dev(gf), 1.0, d_table, ws, wb, _lib.GRAD_OVERWRITE)
    torch.cuda.synchronize()
    scaled_close(d_table.cpu().numpy(), O.encode_backward(x, gf, og), O.encode_backward(x, np.abs(gf), og), RTOL_GRAD)


def test_batched_encode_grid_can_be_launched():
    # one workgroup of 256 threads per item up to the largest launch (below 2^32 threads),
    # whole rounds of the eight XCDs; a smaller grid where one is asked for
    grid = _lib.load()["_ZN3h4d17batch_encode_gridEii"]
    for items in (1, 7, 8, 9, 1000, (1 << 24) - 9, (1 << 24) - 8, 1 << 24, (1 << 24) + 1, (1 << 30) + 5, (1 << 31) - 1):
        g = grid(0, items)
        assert g % 8 == 0 and 0 < g * 256 < 1 << 32
        assert g == min((items + 7) // 8 * 8, (1 << 24) - 8)
        assert grid(1024, items) == min(1024, g)


@pytest.mark.gpu
def test_batched_plan_whose_lists_do_not_fit():
    # 9.6e9 (query, timestamp, level) triples: lists of 307 GB are more than the card has,
    # so the plan is made with masks (38 GB, and 38 GB of feature gradients); it is not run,
    # and its buffers are never touched
    needs_gpu()
    import torch
    L, n, times = 8, 240_000_000, [0.0, 0.25, 0.5, 0.75, 1.0]
    lg = _lib.h4d_grid_init(L, 1, [2047] * L, [3] * L, 1 << 11)
    one = torch.zeros(64, device="cuda")
    plan = _lib.BatchedPlan([_lib.scene_desc(lg, n, one, times, *[one] * 7)], _lib.mlp_shape(L), _lib.F32)
    info = plan.info()
    assert info.queries == n * len(times) and info.encode_grid * 256 < 1 << 32
    plan.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [_lib.F32, _lib.F64], ids=["f32", "f64"])
@pytest.mark.parametrize("form", ["one_set", "two_sets", "batched"])
@pytest.mark.parametrize("n,crowded", [(1, False), (3000, False), (2500, True)])
def test_dense_level_of_more_tiles_than_lists(form, dt, n, crowded):
    # 512 tiles of x-lines in FP32, 1024 in FP64: two or four tiles share a list
    if form == "batched" and dt == _lib.F64:
        pytest.skip("batched plans run F32 or BF16")
    needs_gpu()
    import torch
    L, F, rs, rt, T = 1, 8, [63], [4], 1 << 21
    og, lg = O.make_grid(L, F, rs, rt, T), _lib.h4d_grid_init(L, F, rs, rt, T)
    assert lg.dense_list() == [True]
    rng, x = _inputs(n, n + 3, crowded)
    real = np.float64 if dt == _lib.F64 else np.float32
    gf = synth.upstream(n, F, rng)
    d_table = _dev(np.full((og.E, F), np.nan, real))
    layout = _lib.QUERY_MAJOR | _lib.GRAD_OVERWRITE
    ref, scale = O.encode_backward(x, gf, og), O.encode_backward(x, np.abs(gf), og)
    if form == "one_set":
        wb = _lib.hash4d_encode_backward_workspace_bytes(lg, n)
        ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
        _lib.hash4d_encode_backward(lg, dt, _dev(x), n, _dev(gf.astype(real)), 1.0, d_table, ws, wb, layout)
    elif form == "two_sets":
        table, eps = synth.table_init(og.E, F, rng), synth.perturbation(n, rng, 1e-2)
        loss = torch.zeros(1, dtype=torch.float64 if dt == _lib.F64 else torch.float32, device="cuda")
        wb = _lib.smoothness_workspace_bytes(lg, dt, n)
        ws = torch.empty(wb, dtype=torch.uint8, device="cuda")
        _lib.hash4d_encode_backward_smooth(lg, dt, _dev(table.astype(real)), _dev(x), _dev(eps), n,
                                           _dev(gf.astype(real)), 1.0, 2.0, loss, d_table, ws, wb, layout)
        xp = O.perturbed(x, eps)
        s = 4.0 / n * (np.abs(O.encode(x, table, og) - O.encode(xp, table, og)) + O.encode(x, np.abs(table), og)
                       + O.encode(xp, np.abs(table), og))
        ref = ref + O.smoothness(x, eps, table, og, 2.0)[1]
        scale = scale + O.encode_backward(x, s, og) + O.encode_backward(xp, s, og)
    else:
        x = np.clip(np.nan_to_num(x), 0, 1).astype(np.float32)
        times = [0.25, 0.7]
        table, params = synth.table_init(og.E, F, rng), synth.decoder_params(F, rng)
        gd = synth.upstream(n * 2, 10, rng).reshape(2, n, 10)
        bufs = [_dev(x), _dev(table), _dev(params), torch.empty((2, L, n, F), device="cuda"),
                torch.empty((2, n, 10), device="cuda"), _dev(gd), torch.full((params.size,), float("nan"), device="cuda")]
        plan = _lib.BatchedPlan([_lib.scene_desc(lg, n, bufs[0], times, bufs[1], bufs[2], bufs[3], bufs[4], bufs[5],
                                                 d_table, bufs[6])], _lib.mlp_shape(F), _lib.F32, 1.0,
                                _lib.PLAN_ZERO_GRADS)
        plan.run()
        torch.cuda.synchronize()
        plan.destroy()
        ref, scale = np.zeros((og.E, F)), np.zeros((og.E, F))
        for k, t in enumerate(times):
            xt = x.copy()
            xt[:, 3] = np.float32(t)
            ref += O.deform_backward(xt, table, og, params, gd[k])[0]
            scale += O.encode_backward(xt, mlp_backward_scale(params, O.encode(xt, table, og), gd[k])[0], og)
    torch.cuda.synchronize()
    scaled_close(d_table.cpu().numpy(), ref, scale, 1e-12 if dt == _lib.F64 else RTOL_GRAD, f"{form} n={n}")
