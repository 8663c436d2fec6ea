"""Weight gradients on widths that are odd multiples of 128 (256-wide tiles
with half-empty last ones, or 128-wide tiles), with many groups and with
groups spread over many micro-steps, against fp64 sums of the same bf16
operands. Tolerance: an fp32 sum of K products in any order is within
K 2^-24 of the sum of the products' magnitudes (the pieces of a split group
are added in fp32 too)."""
import numpy as np
import pytest
import torch

# d, F, rows of every micro-step's slots, gradient groups
CASES = {
    "odd-large": (640, 384, [[700, 0, 130, 65], [1, 300, 0, 511]], 5),     # 256-wide tiles, half empty
    "odd-few-rows": (640, 384, [[70, 0, 33, 65]], 3),                      # 128-wide tiles
    "odd-one-side": (1152, 1024, [[64, 190, 7]], 3),                       # 256-wide, one dimension odd
    "many-groups": (256, 256, [[(7 * i) % 83 for i in range(100)]], 100),  # more groups than a wavefront
    "many-steps": (256, 256, [[40, 200, 3, 64]] * 16, 4),                  # long chains of slots
}


@pytest.mark.gpu
@pytest.mark.parametrize("ws_kind", ["none", "counters", "split"])
@pytest.mark.parametrize("name", list(CASES))
def test_wgrad_tiles(gpu, name, ws_kind):
    from paper_2606_11867_amd import api
    d, F, steps, G = CASES[name]
    print(f"\n[case] weight gradients {name}: d={d} F={F} steps={len(steps)} workspace {ws_kind}", flush=True)
    rng = np.random.default_rng(len(name))
    bf = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(gpu).to(torch.bfloat16)  # noqa: E731
    i32 = lambda a: torch.tensor(np.asarray(a, np.int32), device=gpu)  # noqa: E731
    recs, ref = [], {"gu": np.full((G, 2 * F, d), 0.25), "dn": np.full((G, d, F), 0.25)}
    mag = {k: v.copy() for k, v in ref.items()}
    for m, rows in enumerate(steps):
        off = np.concatenate([[0], np.cumsum(rows)])
        gidx = (np.arange(len(rows)) * 3 + m) % G
        n = int(off[-1]) + 5
        r = dict(x_perm=bf(n, d), h=bf(n, F), dy_perm=bf(n, d), d_au=bf(n, 2 * F))
        f64 = {k: t.double().cpu().numpy() for k, t in r.items()}
        for j, g in enumerate(gidx):
            s = slice(off[j], off[j + 1])
            for key, a, b in (("gu", f64["d_au"][s], f64["x_perm"][s]), ("dn", f64["dy_perm"][s], f64["h"][s])):
                ref[key][g] += a.T @ b
                mag[key][g] += np.abs(a).T @ np.abs(b)
        recs.append(dict(r, slot_offset=i32(off), slot_gidx=i32(gidx)))
    ws = {"none": None, "counters": torch.zeros(256, dtype=torch.uint8, device=gpu),
          "split": api.wgrad_workspace(d, F, gpu)}[ws_kind]
    K = sum(sum(r) for r in steps) + 2
    for parts in (1, 2):
        gu, dn = (torch.full(ref[k].shape, 0.25, device=gpu) for k in ("gu", "dn"))
        for part in range(parts):
            api.grouped_ffn_wgrad_steps(recs, gu, dn, ws=ws, part=part, parts=parts)
        torch.cuda.synchronize()
        for key, got in (("gu", gu), ("dn", dn)):
            err = np.abs(got.double().cpu().numpy() - ref[key])
            bound = K * 2.0 ** -24 * mag[key]
            assert np.all(err <= bound), f"{key} parts={parts}: {np.max(err - bound):.3g} over its bound"


@pytest.mark.gpu
def test_nan_next_to_a_tile_stays_out(gpu):
    """NaN and infinities in the operand columns that a half-empty last tile
    of an odd width reads and must not store (the next row's first ones), and
    in the rows of another group."""
    from paper_2606_11867_amd import api
    d, F, rows, G = 640, 384, [700, 130, 300], 3
    print(f"\n[case] NaN beside the weight-gradient tiles, rows {rows}, d={d}, F={F}", flush=True)
    g = torch.Generator(device=gpu).manual_seed(2)
    bf = lambda *s: torch.randn(*s, generator=g, device=gpu).bfloat16()  # noqa: E731
    N = sum(rows)
    ops = [bf(N, d), bf(N, F), bf(N, d), bf(N, 2 * F)]  # x, h, dy, d_au
    off = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int32, device=gpu)
    gidx = torch.arange(G, dtype=torch.int32, device=gpu)

    def run(ops, ws):
        dw = [torch.zeros(s, device=gpu) for s in ((G, 2 * F, d), (G, d, F))]
        api.grouped_ffn_wgrad(*ops, off, gidx, *dw, ws=ws)
        torch.cuda.synchronize()
        return dw

    for ws in (api.wgrad_workspace(d, F, gpu), None):
        want = run(ops, ws)
        bad = [t.clone() for t in ops]
        for t, v in zip(bad, (float("nan"), float("inf"), float("-inf"), float("nan"))):
            t[:, :128] = v
        for name, a, b in zip(("dW_gate_up", "dW_down"), run(bad, ws), want):
            assert torch.equal(a[:, 128:, 128:], b[:, 128:, 128:]), name
            assert not bool(a[:, :128].isfinite().any()) and not bool(a[:, :, :128].isfinite().any()), name
        bad = [t.clone() for t in ops]
        for t in bad:
            t[:700] = float("nan")  # group 0
        for name, a, b in zip(("dW_gate_up", "dW_down"), run(bad, ws), want):
            assert torch.equal(a[1:], b[1:]) and bool(a[0].isnan().all()), name
