"""The fp32 FFN kernels at the edges of their 32 x 32 tiles and 64-deep K
slices, against fp64 products. Tolerances: an fp32 sum of K products is within
gamma = K 2^-24 / (1 - K 2^-24) of the sum of the products' magnitudes in any
order (Higham, Accuracy and Stability, Sec. 3.1); the activation adds a few
ulp (E below)."""
import numpy as np
import pytest
import torch

E = 1e-5  # exp, divide and the products of the SwiGLU epilogues, relative


def _gamma(K):
    return (K + 2) * 2.0 ** -24 * 1.01


def _slots(rows, W):
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    return off, (np.arange(len(rows)) % W).astype(np.int32)


def _close(name, got, ref, bound):
    err = np.abs(got.double().cpu().numpy() - ref)
    assert np.all(err <= bound + 1e-30), f"{name}: {np.max(err - bound):.3g} over its bound"


# tile, slice and wavefront edges; widths of one; odd widths (rows of x, h
# and the weights then start at any multiple of 4 bytes)
SHAPES = [(1, 1, [1, 0, 3]), (31, 33, [63, 64, 0, 65]), (64, 32, [128, 1, 129]), (65, 127, [5, 200]),
          (128, 256, [45] * 6), (130, 96, [0, 0, 70])]


@pytest.mark.gpu
@pytest.mark.parametrize("d,F,rows", SHAPES)
def test_f32_ffn_matches_fp64(gpu, d, F, rows):
    from paper_2606_11867_amd import api
    print(f"\n[case] fp32 FFN d={d} F={F} rows={rows}", flush=True)
    rng = np.random.default_rng(d * 1000 + F)
    W = 2
    off, widx = _slots(rows, W)
    N, n_cap = int(off[-1]), int(off[-1]) + 7
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    x, h, dy, au, dau = f32(n_cap, d), f32(n_cap, F), f32(n_cap, d), f32(n_cap, 2 * F), f32(n_cap, 2 * F)
    gu, dn = f32(W, 2 * F, d), f32(W, d, F)
    dev = lambda a: torch.from_numpy(a).to(gpu)  # noqa: E731
    lib_off, lib_w = dev(off), dev(widx)
    hg, yg, aug = api.grouped_ffn_fwd(dev(x), lib_off, lib_w, dev(gu), dev(dn))
    daug, dxg = api.grouped_ffn_dgrad(dev(dy), dev(au), lib_off, lib_w, dev(gu), dev(dn))
    dwgu, dwdn = (torch.full(s, 0.5, device=gpu) for s in ((W + 1, 2 * F, d), (W + 1, d, F)))
    api.grouped_ffn_wgrad(dev(x), dev(h), dev(dy), dev(dau), lib_off, lib_w, dwgu, dwdn)
    torch.cuda.synchronize()
    D = np.float64
    rgu, rdn = np.full(dwgu.shape, 0.5), np.full(dwdn.shape, 0.5)
    bgu, bdn = np.full(dwgu.shape, 0.5), np.full(dwdn.shape, 0.5)  # magnitudes
    for j, w in enumerate(widx):
        r = slice(off[j], off[j + 1])
        X, Wgu, Wdn = x[r].astype(D), gu[w].astype(D), dn[w].astype(D)
        ref, mag = X @ Wgu.T, np.abs(X) @ np.abs(Wgu).T
        _close("A|U", aug[r], ref, _gamma(d) * mag)
        A, U = aug[r].double().cpu().numpy()[:, :F], aug[r].double().cpu().numpy()[:, F:]
        Href = A / (1 + np.exp(-A)) * U
        _close("H", hg[r], Href, E * np.abs(Href))
        Hs = hg[r].double().cpu().numpy()
        _close("Y", yg[r], Hs @ Wdn.T, _gamma(F) * (np.abs(Hs) @ np.abs(Wdn).T))
        dH, dHm = dy[r].astype(D) @ Wdn, np.abs(dy[r].astype(D)) @ np.abs(Wdn)
        a, u = au[r, :F].astype(D), au[r, F:].astype(D)
        s = 1 / (1 + np.exp(-a))
        ds = s + a * s * (1 - s)
        # the derivative is a sum that can cancel: its error is relative to its terms
        dsm = s + np.abs(a) * s * (1 - s)
        _close("dA", daug[r][:, :F], dH * u * ds, (_gamma(d) + E) * dHm * np.abs(u) * dsm)
        _close("dU", daug[r][:, F:], dH * a * s, (_gamma(d) + E) * dHm * np.abs(a) * s)
        G = daug[r].double().cpu().numpy()
        _close("dX", dxg[r], G @ Wgu, _gamma(2 * F) * (np.abs(G) @ np.abs(Wgu)))
        rgu[w] += dau[r].astype(D).T @ X
        bgu[w] += np.abs(dau[r].astype(D)).T @ np.abs(X)
        rdn[w] += dy[r].astype(D).T @ h[r].astype(D)
        bdn[w] += np.abs(dy[r].astype(D)).T @ np.abs(h[r].astype(D))
    _close("dW_gate_up", dwgu, rgu, _gamma(N + 1) * bgu)
    _close("dW_down", dwdn, rdn, _gamma(N + 1) * bdn)


@pytest.mark.gpu
def test_f32_ffn_many_slots_and_bad_weight_index(gpu):
    """More slots than one pass of the tile search covers; a slot with a
    weight index out of range leaves its rows as they were."""
    from paper_2606_11867_amd import _lib, api
    rng = np.random.default_rng(4)
    S, W, d, F = 700, 3, 20, 12
    rows = rng.integers(0, 4, S)
    rows[650] = 90
    off, widx = _slots(rows, W)
    widx[3], widx[650] = -1, W
    N = int(off[-1])
    x, gu = (rng.standard_normal(s).astype(np.float32) for s in ((N, d), (W, 2 * F, d)))
    dev = lambda a: torch.from_numpy(a).to(gpu)  # noqa: E731
    h = torch.full((N, F), 7.0, device=gpu)
    xd, od, wd, gd = dev(x), dev(off), dev(widx), dev(gu)
    print(f"\n[case] fp32 gate/up forward, {S} slots, {N} rows", flush=True)
    rc = _lib.load().foremoe_ffn_gate_up_fwd(xd.data_ptr(), _lib.F32, d, F, S, od.data_ptr(), wd.data_ptr(), W,
                                             gd.data_ptr(), N, h.data_ptr(), None, None, 0,
                                             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0
    for j, w in enumerate(widx):
        r = slice(off[j], off[j + 1])
        if not 0 <= w < W:
            assert bool((h[r] == 7.0).all())
            continue
        A, U = np.split(x[r].astype(np.float64) @ gu[w].astype(np.float64).T, 2, axis=1)
        m = np.abs(x[r].astype(np.float64)) @ np.abs(gu[w].astype(np.float64)).T
        mA, mU = np.split(m, 2, axis=1)
        ref = A / (1 + np.exp(-A)) * U
        # |silu'| < 1.1, |silu(A)| <= |A|
        _close("H", h[r], ref, _gamma(d) * (1.1 * mA * np.abs(U) + np.abs(A) * mU) * 1.1 + E * np.abs(ref) + 1e-6)


@pytest.mark.gpu
@pytest.mark.parametrize("d,F,parts", [(3, 1, 4), (33, 70, 2), (128, 40, 3), (65, 260, 16)])
def test_f32_wgrad_parts_are_the_whole(gpu, d, F, parts):
    """A part's tiles hold its own rows only (m = part + parts i): every part
    writes its rows, with the bits of the undivided call, and no others."""
    from paper_2606_11867_amd import api
    print(f"\n[case] fp32 weight gradients d={d} F={F} in {parts} parts", flush=True)
    rng = np.random.default_rng(d + F)
    rows, G = [70, 0, 5, 130], 3
    N = sum(rows)
    f32 = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(gpu)  # noqa: E731
    i32 = lambda a: torch.tensor(np.asarray(a, np.int32), device=gpu)  # noqa: E731
    rec = [dict(x_perm=f32(N, d), h=f32(N, F), dy_perm=f32(N, d), d_au=f32(N, 2 * F),
                slot_offset=i32(np.concatenate([[0], np.cumsum(rows)])), slot_gidx=i32([0, 1, 2, 0]))]
    whole = [f32(G, 2 * F, d), f32(G, d, F)]
    got = [t.clone() for t in whole]
    start = [t.clone() for t in whole]
    api.grouped_ffn_wgrad_steps(rec, *whole)
    for part in range(parts):
        api.grouped_ffn_wgrad_steps(rec, *got, part=part, parts=parts)
        torch.cuda.synchronize()
        for name, g, w, s in zip(("dW_gate_up", "dW_down"), got, whole, start):
            done = torch.arange(g.shape[1], device=gpu) % parts <= part
            assert torch.equal(g[:, done], w[:, done]) and torch.equal(g[:, ~done], s[:, ~done]), f"{name}, part {part}"
