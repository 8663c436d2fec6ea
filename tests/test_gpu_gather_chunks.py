"""combine, permute_bwd and combine_bwd at the edges of a wavefront's column
chunk (128 vectors of 16 bytes) and of a workgroup's four chunks, with rows
dropped, against fp64. Tolerance: an fp32 sum of K products is within
(K + 1) 2^-24 of the magnitudes' sum, and a bf16 result (8 significant bits)
within half an ulp, at most 2^-8 of it."""
import numpy as np
import pytest
import torch


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("bf16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("T,K,d", [(1, 1, 8), (5, 3, 1016), (3, 64, 1024), (7, 8, 1032), (2, 5, 4112)])
def test_gather_chunks(gpu, T, K, d, dtype, out):
    from paper_2606_11867_amd import api
    dt, od = (dict(f32=torch.float32, bf16=torch.bfloat16)[v] for v in (dtype, out))
    print(f"\n[case] gathers T={T} K={K} d={d} {dtype} -> {out}", flush=True)
    rng = np.random.default_rng(T * 100 + K)
    n = max(1, T * K // 2)  # rows; the other pairs are not local
    p2r = np.full(T * K, -1, np.int32)
    p2r[rng.permutation(T * K)[:n]] = rng.permutation(n)
    p2r[0] = n + 3  # past the buffer: dropped
    yp = torch.from_numpy(rng.standard_normal((n, d), dtype=np.float32)).to(gpu).to(dt)
    dy = torch.from_numpy(rng.standard_normal((T, d), dtype=np.float32)).to(gpu).to(dt)
    gates = torch.from_numpy(rng.random((T, K), dtype=np.float32)).to(gpu)
    pd = torch.from_numpy(p2r).to(gpu)
    y = api.combine(yp, pd, gates, out_dtype=od)
    dx = api.permute_bwd(yp, pd, T, K, out_dtype=od)
    dyp, dg = api.combine_bwd(dy, yp, pd, gates)
    torch.cuda.synchronize()
    Y, D, G = (t.double().cpu().numpy() for t in (yp, dy, gates))
    ry, my, rx, mx = (np.zeros((T, d)) for _ in range(4))
    eps = 2.0 ** -8 if od is torch.bfloat16 else 2.0 ** -23
    epsp = 2.0 ** -8 if dt is torch.bfloat16 else 2.0 ** -23
    for p, r in enumerate(p2r):
        t, k = divmod(p, K)
        if not 0 <= r < n:
            assert dg[t, k].item() == 0
            continue
        ry[t] += G[t, k] * Y[r]
        my[t] += np.abs(G[t, k] * Y[r])
        rx[t] += Y[r]
        mx[t] += np.abs(Y[r])
        got = dyp[r].double().cpu().numpy()
        assert np.all(np.abs(got - G[t, k] * D[t]) <= epsp * np.abs(G[t, k] * D[t]))
        assert abs(dg[t, k].item() - D[t] @ Y[r]) <= (d + 2) * 2.0 ** -24 * (np.abs(D[t]) @ np.abs(Y[r]))
    for got, ref, mag in ((y, ry, my), (dx, rx, mx)):
        err = np.abs(got.double().cpu().numpy() - ref)
        assert np.all(err <= eps * np.abs(ref) + (K + 2) * 2.0 ** -23 * mag)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [8, 264])
def test_combine_past_the_launch_limit(gpu, d):
    """2^26 wavefronts and more, one per token: as many threads as a launch
    may not have. Narrow rows and wider ones; slices of the result against
    torch (one pair per token, so the product is rounded once)."""
    from paper_2606_11867_amd import api
    T, n = 2 ** 26 + 5, 1000
    print(f"\n[case] combine T={T} d={d}", flush=True)
    g = torch.Generator(device=gpu).manual_seed(d)
    yp = torch.randn(n, d, generator=g, device=gpu).bfloat16()
    p2r = torch.randint(-1, n + 2, (T,), generator=g, device=gpu, dtype=torch.int32)
    gates = torch.rand(T, 1, generator=g, device=gpu)
    for name, y, scale in (("combine", api.combine(yp, p2r, gates, out_dtype=torch.bfloat16), gates),
                           ("permute_bwd", api.permute_bwd(yp, p2r, T, 1, out_dtype=torch.bfloat16), None)):
        torch.cuda.synchronize()
        for t0 in [0, 2 ** 24 - 7, 2 ** 25, T - 2 ** 16]:
            s = slice(t0, min(t0 + 2 ** 16, T))
            r = p2r[s].long()
            ok = (r >= 0) & (r < n)
            ref = yp[r.clamp(0, n - 1)].float() * (scale[s] if scale is not None else 1.0)
            ref[~ok] = 0
            assert torch.equal(y[s], ref.bfloat16()), f"{name}: tokens from {t0}"
        del y
