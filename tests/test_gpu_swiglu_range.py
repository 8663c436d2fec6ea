"""The bf16 SwiGLU epilogues at gate values where the sigmoid is a subnormal
fp32 number, against fp64. Tolerance: half an ulp of the bf16 result (2^-8
relative) and E for the fp32 exponential, divide and products: an argument of
90 rounds to 2^-18, so the exponential is within 2^-17 of itself."""
import numpy as np
import pytest
import torch

E = 2.0 ** -16


def _close(name, got, ref, mag=None):
    got = got.double().cpu().numpy()
    mag = np.abs(ref) if mag is None else mag
    bad = np.abs(got - ref) > 2.0 ** -8 * np.abs(ref) + E * mag
    assert not bad.any(), f"{name}: {got[bad][:4]} for {ref[bad][:4]}"


@pytest.mark.gpu
@pytest.mark.parametrize("use_ws", [True, False])
def test_swiglu_with_subnormal_sigmoid(gpu, use_ws):
    from paper_2606_11867_amd import api
    d, F = 128, 128
    A = np.arange(-88.5, -80.0, 0.5)  # bf16 numbers; e^-A is still finite
    A = np.concatenate([A, [-87.5, -30.0, -1.0, 0.0, 1.0, 30.0, 88.5]])
    N, u = len(A), 3.0
    print(f"\n[case] SwiGLU, gate values {A.min()} .. {A.max()}, workspace {use_ws}", flush=True)
    bf = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(gpu).to(torch.bfloat16)  # noqa: E731
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=gpu)  # noqa: E731
    # x = (A, u, 0, ...), so that every gate column is A and every up column u
    x, gu = np.zeros((N, d)), np.zeros((1, 2 * F, d))
    x[:, 0], x[:, 1], gu[0, :F, 0], gu[0, F:, 1] = A, u, 1, 1
    # one-hot down weights: dH is dy
    dn = np.eye(d, F)[None]
    dy = np.full((N, d), -2.0)
    ws = api.ffn_workspace(gpu) if use_ws else None
    h, _, au = api.grouped_ffn_fwd(bf(x), i32([0, N]), i32([0]), bf(gu), bf(dn), ws=ws)
    dau, _ = api.grouped_ffn_dgrad(bf(dy), au, i32([0, N]), i32([0]), bf(gu), bf(dn), ws=ws)
    torch.cuda.synchronize()
    a = np.repeat(A[:, None], F, axis=1)
    s = 1 / (1 + np.exp(-a))
    _close("H", h, a * s * u)
    _close("dU", dau[:, F:], -2.0 * a * s)
    terms = s + np.abs(a) * s * (1 - s)  # the derivative is a sum that can cancel
    _close("dA", dau[:, :F], -2.0 * u * (s + a * s * (1 - s)), 2.0 * u * terms)
