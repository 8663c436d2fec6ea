"""The row GEMMs over every tile shape (256, 128 and 64 rows; whole and half
column tiles), as two launches and as one launch per direction, with and
without the workspace, against fp64 products of the same bf16 operands.

Tolerance: a bf16 output is within half an ulp (2^-8 relative) of its fp32
sum, which is within gamma = K 2^-24 of the magnitudes' sum (any order); the
second GEMM of a pair multiplies the first one's rounded rows as the GPU
wrote them."""
import numpy as np
import pytest
import torch

import row_units as R


def _dev(a, gpu, dtype=torch.bfloat16):
    return torch.from_numpy(np.ascontiguousarray(a)).to(gpu).to(dtype)


def _f64(t):
    return t.double().cpu().numpy()


def _close(name, got, ref, mag, K):
    err = np.abs(got - ref)
    bound = 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -23 * mag + 1e-6
    assert np.all(np.isfinite(got)), f"{name}: not finite"
    assert np.all(err <= bound), f"{name}: {np.max(err - bound):.3g} over its bound"


def _check(gpu, rows, d, F, W, use_ws, widx=None, misalign=0):
    from paper_2606_11867_amd import _lib, api
    lib = _lib.load()
    rng = np.random.default_rng(len(rows) * 7 + d + F)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    widx = (np.arange(len(rows)) % W if widx is None else np.asarray(widx)).astype(np.int32)
    N, S = int(off[-1]), len(rows)
    x, dy = (_dev(rng.standard_normal((N, d), dtype=np.float32), gpu) for _ in range(2))
    gu = _dev(rng.standard_normal((W, 2 * F, d), dtype=np.float32) * d ** -0.5, gpu)
    dn = _dev(rng.standard_normal((W, d, F), dtype=np.float32) * F ** -0.5, gpu)
    od, wd = _dev(off, gpu, torch.int32), _dev(widx, gpu, torch.int32)
    ws = api.ffn_workspace(gpu) if use_ws else None
    p = lambda t: t.data_ptr()  # noqa: E731
    wp, wn = (p(ws), ws.numel()) if use_ws else (None, 0)
    st = torch.cuda.current_stream().cuda_stream

    def rows_buf(cols, fill):  # guarded rows, optionally off the 128-byte line
        raw = torch.full((N * cols + 256,), fill, dtype=torch.bfloat16, device=gpu)
        return raw[misalign:misalign + N * cols].view(N, cols), raw

    outs = []
    for pair in (False, True):
        (h, hr), (y, yr), (au, ar) = rows_buf(F, 3.0), rows_buf(d, 3.0), rows_buf(2 * F, 3.0)
        (dau, dr), (dx, xr) = rows_buf(2 * F, 3.0), rows_buf(d, 3.0)
        for _ in range(2):  # twice: the counters must be back at zero
            if pair:
                rc = [lib.foremoe_grouped_ffn_fwd(p(x), 1, d, F, S, p(od), p(wd), W, p(gu), p(dn), N, p(h), p(y),
                                                  p(au), wp, wn, st),
                      lib.foremoe_grouped_ffn_dgrad(p(dy), p(au), 1, d, F, S, p(od), p(wd), W, p(gu), p(dn), N,
                                                    p(dau), p(dx), wp, wn, st)]
            else:
                rc = [lib.foremoe_ffn_gate_up_fwd(p(x), 1, d, F, S, p(od), p(wd), W, p(gu), N, p(h), p(au), wp, wn,
                                                  st),
                      lib.foremoe_ffn_down_fwd(p(h), 1, d, F, S, p(od), p(wd), W, p(dn), N, p(y), wp, wn, st),
                      lib.foremoe_ffn_down_dgrad(p(dy), p(au), 1, d, F, S, p(od), p(wd), W, p(dn), N, p(dau), wp, wn,
                                                 st),
                      lib.foremoe_ffn_gate_up_dgrad(p(dau), 1, d, F, S, p(od), p(wd), W, p(gu), N, p(dx), wp, wn,
                                                    st)]
            assert rc == [0] * len(rc)
        torch.cuda.synchronize()
        if use_ws:
            assert not bool(ws[:65536].any()), "counters not back at zero"
        for raw, t in ((hr, h), (yr, y), (ar, au), (dr, dau), (xr, dx)):  # nothing outside the rows
            assert bool((raw[:misalign] == 3.0).all()) and bool((raw[misalign + t.numel():] == 3.0).all())
        outs.append((h, y, au, dau, dx))
    # products that neither form cuts along K have the same bits in both (the
    # input gradients read the forward's A|U)
    G = torch.cuda.get_device_properties(gpu).multi_processor_count
    uncut = [all(fn(rows, d, F, phases=ph, G=G, ws=use_ws)[i].s == 1 for ph in (1 + i, 3))
             for fn in (R.forward, R.dgrad) for i in (0, 1)]
    for name, k, needs in (("H", 0, [0]), ("Y", 1, [0, 1]), ("A|U", 2, [0]), ("dA|dU", 3, [0, 2]),
                           ("dX", 4, [0, 2, 3])):
        if all(uncut[i] for i in needs):
            assert torch.equal(outs[0][k], outs[1][k]), f"{name}: one launch and two differ"
    gu64, dn64 = _f64(gu), _f64(dn)
    for pair, (h, y, au, dau, dx) in enumerate(outs):
        for j, w in enumerate(widx):
            r = slice(off[j], off[j + 1])
            if rows[j] == 0:
                continue
            if not 0 <= w < W:
                assert all(bool((t[r] == 3.0).all()) for t in (h, y, au, dau, dx))
                continue
            tag = f"pair={bool(pair)} slot {j} ({rows[j]} rows)"
            X, G, D = _f64(x[r]), gu64[w], dn64[w]
            AU = _f64(au[r])
            _close(tag + " A|U", AU, X @ G.T, np.abs(X) @ np.abs(G).T, d)
            A, U = np.split(X @ G.T, 2, axis=1)  # H comes from the unrounded sums
            mA, mU = np.split(np.abs(X) @ np.abs(G).T, 2, axis=1)
            s = 1 / (1 + np.exp(-A))
            H = _f64(h[r])
            _close(tag + " H", H, A * s * U, 1.2 * (mA * np.abs(U) + np.abs(A) * mU), d + 16)
            _close(tag + " Y", _f64(y[r]), H @ D.T, np.abs(H) @ np.abs(D).T, F)
            A, U = np.split(AU, 2, axis=1)
            s = 1 / (1 + np.exp(-A))
            DY, DAU = _f64(dy[r]), _f64(dau[r])
            dH, mH = DY @ D, np.abs(DY) @ np.abs(D)
            ds = s + A * s * (1 - s)
            _close(tag + " dA", DAU[:, :F], dH * U * ds, mH * np.abs(U) * (s + np.abs(A) * s * (1 - s)), d + 16)
            _close(tag + " dU", DAU[:, F:], dH * A * s, mH * np.abs(A) * s, d + 16)
            _close(tag + " dX", _f64(dx[r]), DAU @ G, np.abs(DAU) @ np.abs(G), 2 * F)


# rows at the edges of the three tile heights; widths that end in a column
# tile of 128, fewer and more than 12 column tiles (row groups of 8)
LAYOUTS = {
    "edges": ([1, 63, 64, 65, 0, 127, 128, 129, 255, 256, 257, 0, 320, 321, 384, 385], 256, 128),
    "odd-width": ([5, 200, 700, 40, 0, 90], 384, 640),
    "thin-only": ([3, 0, 17, 64], 1024, 256),
    "row-groups": ([2304, 40, 300], 3328, 1664),
    "one-round": ([3000, 1500, 100, 60, 900], 1152, 896),
    # both products of both directions in more than a round of units, with
    # every tile height; more than a round with row groups
    "rounds": ([1300, 900, 500] + [10 + 2 * i for i in range(52)], 1280, 1280),
    "row-group-rounds": ([2304, 300] + [30] * 12, 3328, 1664),
}


@pytest.mark.parametrize("name", ["rounds", "row-group-rounds"])
def test_layouts_are_more_than_a_round(name):
    """On 256 CUs (host arithmetic)."""
    rows, d, F = LAYOUTS[name]
    grouped = 0
    for fn in (R.forward, R.dgrad):
        u0, u1, t = fn(rows, d, F, G=256)
        assert t.full and t.thin and (t.short or name != "rounds")
        for u in (u0, u1):
            if name == "rounds" or u.nt >= 12:
                assert u.total > 256 and u.total % 256, u
            grouped += u.nt >= 12
    assert grouped == (3 if name == "row-group-rounds" else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("use_ws", [True, False])
@pytest.mark.parametrize("name", list(LAYOUTS))
def test_row_tiles(gpu, name, use_ws):
    rows, d, F = LAYOUTS[name]
    print(f"\n[case] row tiles {name}: rows {rows}, d={d}, F={F}, workspace {use_ws}", flush=True)
    _check(gpu, rows, d, F, 3, use_ws)


@pytest.mark.gpu
def test_row_tiles_many_slots(gpu):
    """More slots than one wavefront's table pass, with bad weight indices."""
    rows = [int(v) for v in np.random.default_rng(3).integers(0, 90, 300)]
    rows[7], rows[299] = 500, 300
    widx = np.arange(300) % 3
    widx[5], widx[7] = -1, 3
    print(f"\n[case] row tiles, 300 slots, {sum(rows)} rows", flush=True)
    _check(gpu, rows, 256, 128, 3, True, widx=widx)


@pytest.mark.gpu
def test_row_tiles_rows_off_the_line(gpu):
    """Handed-over rows that do not start on a 128-byte line: two launches."""
    print("\n[case] row tiles, rows 16 bytes off the line", flush=True)
    _check(gpu, [300, 70, 30], 256, 128, 2, True, misalign=8)


@pytest.mark.gpu
def test_round_of_halves_and_small_tiles_is_not_cut_along_k(gpu):
    """One round of 256-row tiles (in halves) and of smaller ones that would
    be more than 7/8 of the CUs as halves throughout: no K pieces, so the
    workspace changes no bit."""
    from paper_2606_11867_amd import api
    rows, d, F = [300, 40, 26, 17, 200, 64, 1, 90, 5], 2048, 768  # 60 tiles of the gate/up product, 12 of 256 rows
    if torch.cuda.get_device_properties(gpu).multi_processor_count != 256:
        pytest.skip("the layout is worked out for 256 CUs")
    print(f"\n[case] mixed round, rows {rows}, d={d}, F={F}", flush=True)
    g = torch.Generator(device=gpu).manual_seed(3)
    bf = lambda *s, scale=1.0: torch.randn(*s, generator=g, device=gpu).mul_(scale).bfloat16()  # noqa: E731
    W, N = len(rows), sum(rows)
    x, dy = bf(N, d), bf(N, d)
    gu, dn = bf(W, 2 * F, d, scale=d ** -0.5), bf(W, d, F, scale=F ** -0.5)
    off = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32, device=gpu)
    widx = torch.arange(W, dtype=torch.int32, device=gpu)
    runs = []
    for ws in (api.ffn_workspace(gpu), None):
        h, y, au = api.grouped_ffn_fwd(x, off, widx, gu, dn, ws=ws)
        runs.append((h, y, au))
    torch.cuda.synchronize()
    for name, a, b in zip(("H", "Y", "A|U"), *runs):
        assert torch.equal(a, b), name


@pytest.mark.gpu
@pytest.mark.parametrize("left_over", [1000, 2 ** 32 - 16])
def test_counters_that_were_not_zero(gpu, left_over):
    """A queue counter that another call left behind: the launch of both
    products ends (its waits are bounded, and no counter value is taken for a
    unit), leaves every counter at zero, and the next call is right again."""
    from paper_2606_11867_amd import api
    d, F, rows = 512, 256, [700, 40, 300]
    print(f"\n[case] queue counter at {left_over}, rows {rows}", flush=True)
    g = torch.Generator(device=gpu).manual_seed(5)
    bf = lambda *s: torch.randn(*s, generator=g, device=gpu).mul_(0.05).bfloat16()  # noqa: E731
    x, gu, dn = bf(sum(rows), d), bf(3, 2 * F, d), bf(3, d, F)
    off = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32, device=gpu)
    widx = torch.arange(3, dtype=torch.int32, device=gpu)
    ws = api.ffn_workspace(gpu)
    want = api.grouped_ffn_fwd(x, off, widx, gu, dn, ws=ws)
    counters = ws[:65536].view(torch.int32)
    counters[1024] = left_over if left_over < 2 ** 31 else left_over - 2 ** 32  # first product, first queue
    api.grouped_ffn_fwd(x, off, widx, gu, dn, ws=ws)
    torch.cuda.synchronize()
    assert not bool(counters.any()), "counters not back at zero"
    got = api.grouped_ffn_fwd(x, off, widx, gu, dn, ws=ws)
    torch.cuda.synchronize()
    for name, a, b in zip(("H", "Y", "A|U"), got, want):
        assert torch.equal(a, b), name


@pytest.mark.gpu
def test_nan_next_to_a_tile_stays_out(gpu):
    """NaN and infinities in what the half-empty last column tiles of an odd
    width read and must not store (the next weight row's first columns), and
    in the rows of other slots."""
    from paper_2606_11867_amd import api
    rows, d, F, W = [40, 100, 300, 17], 384, 384, 2
    print(f"\n[case] NaN beside the tiles, rows {rows}, d={d}, F={F}", flush=True)
    g = torch.Generator(device=gpu).manual_seed(9)
    bf = lambda *s, scale=1.0: torch.randn(*s, generator=g, device=gpu).mul_(scale).bfloat16()  # noqa: E731
    N = sum(rows)
    x, dy, au = bf(N, d), bf(N, d), bf(N, 2 * F)
    gu, dn = bf(W, 2 * F, d, scale=d ** -0.5), bf(W, d, F, scale=F ** -0.5)
    off = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32, device=gpu)
    widx = torch.tensor([0, 1, 0, 1], dtype=torch.int32, device=gpu)
    for ws in (api.ffn_workspace(gpu), None):
        _, y0, _ = api.grouped_ffn_fwd(x, off, widx, gu, dn, ws=ws)
        dau0, dx0 = api.grouped_ffn_dgrad(dy, au, off, widx, gu, dn, ws=ws)
        # input gradients: the first 128 columns of every weight row
        gu1, dn1 = gu.clone(), dn.clone()
        gu1[:, :, :128], dn1[:, :, :128] = float("nan"), float("inf")
        dau, _ = api.grouped_ffn_dgrad(dy, au, off, widx, gu, dn1, ws=ws)
        _, dx = api.grouped_ffn_dgrad(dy, au, off, widx, gu1, dn, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(dau[:, 128:F], dau0[:, 128:F]) and torch.equal(dau[:, F + 128:], dau0[:, F + 128:])
        assert not bool(dau[:, :128].isfinite().all())
        assert torch.equal(dx[:, 128:], dx0[:, 128:]) and bool(dx[:, :128].isnan().all())
        # rows of the slots before and after slot 1
        x1, dy1 = x.clone(), dy.clone()
        other = torch.ones(N, dtype=torch.bool, device=gpu)
        other[rows[0]:rows[0] + rows[1]] = False
        x1[other], dy1[other] = float("nan"), float("inf")
        _, y, _ = api.grouped_ffn_fwd(x1, off, widx, gu, dn, ws=ws)
        _, dx = api.grouped_ffn_dgrad(dy1, au, off, widx, gu, dn, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(y[~other], y0[~other]) and torch.equal(dx[~other], dx0[~other])


@pytest.mark.gpu
def test_launches_of_both_products_side_by_side(gpu):
    """Two launches of both products on two streams with a workspace each, and
    a weight gradient on a third: the workgroups of each are partly resident
    while others wait. Every result is that of the calls one after another."""
    from paper_2606_11867_amd import api
    d, F, W = 1024, 512, 4
    print("\n[case] launches of both products on two streams, weight gradients on a third", flush=True)
    g = torch.Generator(device=gpu).manual_seed(4)
    bf = lambda *s, scale=1.0: torch.randn(*s, generator=g, device=gpu).mul_(scale).bfloat16()  # noqa: E731
    gu, dn = bf(W, 2 * F, d, scale=d ** -0.5), bf(W, d, F, scale=F ** -0.5)
    sets = []
    for rows in ([4000, 3000, 70, 1500], [100, 5000, 2500, 40]):
        N = sum(rows)
        sets.append(dict(off=torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32, device=gpu), x=bf(N, d),
                         dy=bf(N, d), au=bf(N, 2 * F), ws=api.ffn_workspace(gpu)))
    widx = torch.arange(W, dtype=torch.int32, device=gpu)
    wops = (sets[0]["x"], bf(sum([4000, 3000, 70, 1500]), F), sets[0]["dy"], sets[0]["au"], sets[0]["off"], widx)
    wws = api.wgrad_workspace(d, F, gpu)
    dw = lambda: [torch.zeros(s, device=gpu) for s in ((W, 2 * F, d), (W, d, F))]  # noqa: E731

    def ffn(s):
        out = []
        for _ in range(4):
            out = [*api.grouped_ffn_fwd(s["x"], s["off"], widx, gu, dn, ws=s["ws"]),
                   *api.grouped_ffn_dgrad(s["dy"], s["au"], s["off"], widx, gu, dn, ws=s["ws"])]
        return out

    def wgrad(out):
        for _ in range(4):
            api.grouped_ffn_wgrad(*wops, *out, ws=wws)
        return out

    want = [ffn(s) for s in sets] + [wgrad(dw())]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(gpu) for _ in range(3)]
    got_dw = dw()
    torch.cuda.synchronize()
    got = []
    for st, fn, arg in zip(streams, (ffn, ffn, wgrad), (*sets, got_dw)):
        with torch.cuda.stream(st):
            got.append(fn(arg))
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(got, want)):
        for j, (t, r) in enumerate(zip(a, b)):
            assert torch.equal(t, r), f"stream {i}, output {j}"
    for s in sets:
        assert not bool(s["ws"][:65536].any()), "counters not back at zero"
