"""Row GEMMs, the last, partial round of output tiles: 256-row tiles that
would leave the chip less than half busy are cut along N into half-width
tiles, and with the optional workspace the (half) tiles of such a round are cut
along K into up to 4 pieces whose fp32 partial sums the last piece to finish
adds in piece order (grouped SwiGLU FFN of App. A; the cuts only change where
and in which fp32 order the Step-4 products are summed).

Row layouts are chosen so that the cuts really happen: what each case is named
after is asserted on 256 CUs from the library's own arithmetic (row_units).
Checked, for each GEMM as a launch of its own and for both of a direction in
one, with and without workspace: sampled rows of every slot against the fp64
oracle, two runs bit for bit equal, forms that cut nothing along K bit for bit
equal to each other and the others within the tolerance, and the counters left
at zero.
"""
import numpy as np
import pytest
import torch

import oracle.foremoe_oracle as O
import row_units as R
from gpu_helpers import check_close, to_np
from workload import bf16_round

pytestmark = pytest.mark.gpu

D, W = 2048, 3


def sampled(off, rng, per_slot=5):
    rows, sub, widx = [], [0], []
    for j in range(len(off) - 1):
        lo, hi = int(off[j]), int(off[j + 1])
        if hi <= lo:
            continue
        pick = np.unique(np.concatenate([[lo, hi - 1], rng.integers(lo, hi, size=per_slot)]))
        rows.extend(pick.tolist())
        sub.append(sub[-1] + len(pick))
        widx.append(j % W)
    return np.array(rows), np.array(sub), np.array(widx)


def layouts(d, F, rows, grid):
    """{(GEMM, form): Phase} of the four GEMMs in the forms they are run in:
    "pair" (both of a direction in one launch, with workspace), "single" (a
    launch each, with workspace) and "no workspace"."""
    out = {}
    for names, fn in ((("gate_up_fwd", "down_fwd"), R.forward), (("down_dgrad", "gate_up_dgrad"), R.dgrad)):
        for i, name in enumerate(names):
            out[name, "pair"] = fn(rows, d, F, G=grid)[i]
            out[name, "single"] = fn(rows, d, F, phases=1 + i, G=grid)[i]
            out[name, "no workspace"] = fn(rows, d, F, phases=1 + i, G=grid, ws=False)[i]
    return out


def run_forms(gpu, d, F, rows, seed):
    """Inputs (host), slot offsets and {form: outputs of two runs}."""
    from paper_2606_11867_amd import _lib, api
    lib = _lib.load()
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    N, S = int(off[-1]), len(rows)
    x = bf16_round(rng.standard_normal((N, d), dtype=np.float32))
    dy = bf16_round(rng.standard_normal((N, d), dtype=np.float32))
    gu = bf16_round((rng.standard_normal((W, 2 * F, d)) / np.sqrt(d)).astype(np.float32))
    dn = bf16_round((rng.standard_normal((W, d, F)) / np.sqrt(F)).astype(np.float32))
    # saved [A | U] for the input gradient: seeded inputs of their own (the
    # forward's are checked against the oracle separately)
    au_in = bf16_round((2.0 * rng.standard_normal((N, 2 * F))).astype(np.float32))
    bf = torch.bfloat16
    dev = lambda a: torch.from_numpy(a).to(gpu).to(bf)  # noqa: E731
    xd, dyd, gud, dnd, aud = dev(x), dev(dy), dev(gu), dev(dn), dev(au_in)
    so = torch.from_numpy(off).to(gpu)
    wi = torch.from_numpy((np.arange(S) % W).astype(np.int32)).to(gpu)
    ws = api.ffn_workspace(gpu)
    st = torch.cuda.current_stream(gpu).cuda_stream
    p = lambda t: t.data_ptr()  # noqa: E731

    def single(w_):
        e = lambda c: torch.empty((N, c), dtype=bf, device=gpu)  # noqa: E731
        h, y, au, d_au, dx = e(F), e(d), e(2 * F), e(2 * F), e(d)
        wp, wn = (p(w_), w_.numel()) if w_ is not None else (None, 0)
        common = _lib.BF16, d, F, S, p(so), p(wi), W
        assert [lib.foremoe_ffn_gate_up_fwd(p(xd), *common, p(gud), N, p(h), p(au), wp, wn, st),
                lib.foremoe_ffn_down_fwd(p(h), *common, p(dnd), N, p(y), wp, wn, st),
                lib.foremoe_ffn_down_dgrad(p(dyd), p(aud), *common, p(dnd), N, p(d_au), wp, wn, st),
                lib.foremoe_ffn_gate_up_dgrad(p(d_au), *common, p(gud), N, p(dx), wp, wn, st)] == [0] * 4
        return dict(h=h, y=y, au=au, d_au=d_au, dx=dx)

    def pair(w_):
        h, y, au = api.grouped_ffn_fwd(xd, so, wi, gud, dnd, ws=w_)
        d_au, dx = api.grouped_ffn_dgrad(dyd, aud, so, wi, gud, dnd, ws=w_)
        return dict(h=h, y=y, au=au, d_au=d_au, dx=dx)

    out = {}
    for form, fn, w_ in (("pair", pair, ws), ("single", single, ws), ("no workspace", single, None)):
        out[form] = [fn(w_), fn(w_)]
        torch.cuda.synchronize()
        assert not ws[:65536].any().item(), f"{form}: counters not back at zero"
    return dict(x=x, dy=dy, gu=gu, dn=dn, au=au_in), off, out


def check_forms(lay, out):
    # which GEMMs' sums an output depends on
    needs = dict(h=["gate_up_fwd"], au=["gate_up_fwd"], y=["gate_up_fwd", "down_fwd"], d_au=["down_dgrad"],
                 dx=["down_dgrad", "gate_up_dgrad"])
    ref = out["no workspace"][0]
    for form, (a, b) in out.items():
        for k in a:
            assert torch.equal(a[k], b[k]), f"{k} ({form}): not deterministic"
            if all(lay[g, form].s == 1 for g in needs[k]):
                assert torch.equal(a[k], ref[k]), f"{k} ({form}): not cut along K, and other bits"
            else:
                check_close(f"{k} ({form}) cut along K vs not", to_np(a[k]), to_np(ref[k]))


def check_oracle(inp, out, r, sub, sw, F, gpu):
    rt = torch.from_numpy(r).to(gpu)
    f = O.ffn_forward(inp["x"][r].astype(np.float64), sub, sw, inp["gu"], inp["dn"])
    g = O.ffn_dgrad(inp["dy"][r].astype(np.float64), inp["au"][r, :F], inp["au"][r, F:], sub, sw, inp["gu"],
                    inp["dn"])
    for form, (run, _) in out.items():
        check_close(f"H ({form})", to_np(run["h"][rt]), f["H"])
        check_close(f"Y ({form})", to_np(run["y"][rt]), f["Y"])
        check_close(f"A ({form})", to_np(run["au"][rt][:, :F]), f["A"])
        check_close(f"U ({form})", to_np(run["au"][rt][:, F:]), f["U"])
        check_close(f"dA ({form})", to_np(run["d_au"][rt][:, :F]), g["dA"])
        check_close(f"dU ({form})", to_np(run["d_au"][rt][:, F:]), g["dU"])
        check_close(f"dX ({form})", to_np(run["dx"][rt]), g["dX"])


# d, F, rows of each slot, and what each GEMM in each form has to be cut into
# on 256 CUs: (halves, pieces along K, whether whole rounds come before,
# whether 256-row tiles are among the cut ones, whether smaller ones are)
CASES = {
    "halves": (2048, 256, [5000, 3000], {("gate_up_fwd", "pair"): (2, 1, False, True, False),
                                         ("gate_up_fwd", "no workspace"): (2, 1, False, True, False)}),
    "halves-2-pieces": (2048, 256, [3000, 2000], {("gate_up_fwd", "pair"): (2, 2, False, True, False)}),
    "halves-3-pieces": (3072, 256, [3000, 2000], {("down_dgrad", "pair"): (2, 3, False, True, False)}),
    "halves-and-short-4-pieces": (4096, 256, [3000, 1800], {("down_dgrad", "pair"): (2, 4, False, True, True)}),
    # a last column tile of 128 columns, whose second half has none
    "odd-width-2-pieces": (2048, 384, [2000, 1500], {("down_dgrad", "pair"): (2, 2, False, True, False),
                                                     ("gate_up_fwd", "pair"): (2, 2, False, True, False)}),
    "odd-width-4-pieces": (4096, 384, [2000, 1500], {("down_dgrad", "single"): (2, 4, False, True, False)}),
    "small-2-pieces": (1024, 512, [40] * 8, {("gate_up_fwd", "pair"): (1, 2, False, False, True)}),
    "small-3-pieces": (1536, 512, [40, 100] * 5, {("gate_up_fwd", "pair"): (1, 3, False, False, True)}),
    "small-4-pieces": (2048, 512, [40, 100] * 3, {("gate_up_fwd", "pair"): (1, 4, False, False, True)}),
    "rounds+small-4-pieces": (4096, 1024, [6000, 2300, 90], {
        ("gate_up_fwd", "single"): (1, 4, True, False, True), ("gate_up_dgrad", "pair"): (1, 4, True, False, True),
        ("gate_up_fwd", "pair"): (1, 1, True, False, False)}),
    "rounds+halves-2-pieces": (2048, 1024, [9000, 20, 70], {
        ("gate_up_fwd", "single"): (2, 2, True, True, True), ("gate_up_dgrad", "pair"): (2, 2, True, True, True),
        ("gate_up_fwd", "pair"): (1, 1, True, False, False)}),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tail_split_parity_and_determinism(gpu, name):
    d, F, rows, want = CASES[name]
    grid = torch.cuda.get_device_properties(gpu).multi_processor_count
    lay = layouts(d, F, rows, grid)
    print(f"\n[case] {name}: d={d} F={F} rows {rows}, {grid} CUs", flush=True)
    if grid == 256:
        for k, v in want.items():
            u = lay[k]
            assert (u.h, u.s, u.plain > 0, u.full_cut > 0, u.small_cut > 0) == v, f"{k}: {u}"
    inp, off, out = run_forms(gpu, d, F, rows, 5)
    check_forms(lay, out)
    check_oracle(inp, out, *sampled(off, np.random.default_rng(6)), F, gpu)


# (F, rows): d = 2048, so both plain-store GEMMs (down forward, K = F, and
# gate/up dgrad, K = 2F) have 8 columns of tiles. 66 row tiles of 256 (528
# tiles: two whole rounds and 16 tiles cut into 32 halves); 11 row tiles (88
# tiles, all halves); F = 2048 and 7 row tiles (56 tiles of 32 and 64 k-steps:
# halves without a workspace, halves in 2 K pieces with one)
@pytest.mark.parametrize("F,rows", [(768, [8960, 7168, 768]), (768, [2000, 700]), (2048, [1000, 700])],
                         ids=["rounds+halves", "all-halves", "long-k"])
def test_n_split_last_round(gpu, F, rows):
    grid = torch.cuda.get_device_properties(gpu).multi_processor_count
    lay = layouts(D, F, rows, grid)
    print(f"\n[case] F={F} rows {rows}, {grid} CUs", flush=True)
    if grid == 256:
        for g in ("down_fwd", "gate_up_dgrad"):
            for form in ("single", "no workspace"):
                u = lay[g, form]
                assert u.h == 2 and u.full_cut > 0 and (u.plain > 0) == (sum(rows) > 10000), f"{g} {form}: {u}"
                assert u.s == (2 if F == 2048 and form == "single" else 1), f"{g} {form}: {u}"
    inp, off, out = run_forms(gpu, D, F, rows, 17)
    check_forms(lay, out)
    # every row against the oracle when it is quick, else sampled rows
    N = int(off[-1])
    if N <= 4000:
        pick = np.arange(N), off, np.arange(len(rows)) % W
    else:
        pick = sampled(off, np.random.default_rng(18))
    check_oracle(inp, out, *pick, F, gpu)


def test_invalid_weight_index_slot_is_skipped(gpu):
    """A slot whose weight index is outside [0, W) is skipped by every row
    GEMM: its rows of every output keep what they held, and no arrival
    counter is left set, also when the last round is cut into halves and K
    pieces (here in 2 pieces for the gate/up forward and the down dgrad); the
    other slots' rows match the oracle."""
    from paper_2606_11867_amd import _lib, api
    F, rows, widx = 256, [3000, 2000, 700], [0, -1, W]
    grid = torch.cuda.get_device_properties(gpu).multi_processor_count
    if grid == 256:
        for g in ("gate_up_fwd", "down_dgrad"):
            u = layouts(D, F, rows, grid)[g, "pair"]
            assert (u.h, u.s, u.full_cut > 0) == (2, 2, True), f"{g}: {u}"
    rng = np.random.default_rng(23)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    N = int(off[-1])
    x = bf16_round(rng.standard_normal((N, D)).astype(np.float32))
    dy = bf16_round(rng.standard_normal((N, D)).astype(np.float32))
    gu = bf16_round((rng.standard_normal((W, 2 * F, D)) / np.sqrt(D)).astype(np.float32))
    dn = bf16_round((rng.standard_normal((W, D, F)) / np.sqrt(F)).astype(np.float32))
    au_in = bf16_round((2.0 * rng.standard_normal((N, 2 * F))).astype(np.float32))
    bf = torch.bfloat16
    dev = lambda a: torch.from_numpy(a).to(gpu).to(bf)  # noqa: E731
    xd, dyd, gud, dnd, aud = dev(x), dev(dy), dev(gu), dev(dn), dev(au_in)
    so = torch.from_numpy(off).to(gpu)
    wi = torch.from_numpy(np.array(widx, dtype=np.int32)).to(gpu)
    ws = api.ffn_workspace(gpu)
    sentinel = 7.0
    h, y, au = (torch.full((N, c), sentinel, dtype=bf, device=gpu) for c in (F, D, 2 * F))
    d_au, dx = (torch.full((N, c), sentinel, dtype=bf, device=gpu) for c in (2 * F, D))
    lib = _lib.load()
    st = torch.cuda.current_stream(gpu).cuda_stream
    print(f"\n[case] slots {rows} with weight indices {widx} (W={W}), F={F}", flush=True)
    assert lib.foremoe_grouped_ffn_fwd(xd.data_ptr(), _lib.BF16, D, F, len(rows), so.data_ptr(), wi.data_ptr(), W,
                                       gud.data_ptr(), dnd.data_ptr(), N, h.data_ptr(), y.data_ptr(), au.data_ptr(),
                                       ws.data_ptr(), ws.numel(), st) == 0
    assert lib.foremoe_grouped_ffn_dgrad(dyd.data_ptr(), aud.data_ptr(), _lib.BF16, D, F, len(rows), so.data_ptr(),
                                         wi.data_ptr(), W, gud.data_ptr(), dnd.data_ptr(), N, d_au.data_ptr(),
                                         dx.data_ptr(), ws.data_ptr(), ws.numel(), st) == 0
    torch.cuda.synchronize()
    assert not ws[:65536].any().item(), "counters not back at zero"
    skipped = slice(int(off[1]), N)  # slots 1 and 2
    for name, t in (("H", h), ("Y", y), ("A|U", au), ("dA|dU", d_au), ("dX", dx)):
        assert bool((t[skipped] == sentinel).all()), f"{name}: rows of a skipped slot were written"
    n0 = int(off[1])
    sub, sw = np.array([0, n0]), np.array([0])
    f = O.ffn_forward(x[:n0].astype(np.float64), sub, sw, gu, dn)
    g = O.ffn_dgrad(dy[:n0].astype(np.float64), au_in[:n0, :F], au_in[:n0, F:], sub, sw, gu, dn)
    check_close("H (slot 0)", to_np(h[:n0]), f["H"])
    check_close("Y (slot 0)", to_np(y[:n0]), f["Y"])
    check_close("dA (slot 0)", to_np(d_au[:n0, :F]), g["dA"])
    check_close("dX (slot 0)", to_np(dx[:n0]), g["dX"])
