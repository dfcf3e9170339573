"""GPU parity of favorsharp_attention_backward against the oracle's attention_backward (non-causal and causal).

Tolerance: the kernels accumulate in fp32, the oracle in fp64; the gradients are sums of products of the same
quantities as the forward pass plus one more contraction, so they are held to the forward bar per (b, h): relative
Frobenius error <= 1e-4 times a factor 3 for the extra chain of contractions (f32 inputs) and the same for bf16
inputs on the general-shape kernels (the oracle sees the rounded inputs; all arithmetic of that path is fp32).  The
bf16 MFMA gradient kernels (bf16 rows, d = dv = 64, M = 256) round their operands, features, states and G1 rows to
bf16 and are held to the bf16 bar of the forward pass, 2e-2, whatever dtype the gradients are stored in.
Next to the Frobenius bound every gradient row is bounded: |dg_i| <= 4 tol max_j |g_ref,j| (a few wrong rows at a
slot or chunk boundary of a long tensor would pass the Frobenius bound alone)."""
import numpy as np
import pytest

from oracle import favorsharp_oracle as orc
from paper_2302_00787_amd import synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fs():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2302_00787_amd import binding
    binding.lib()
    return binding


def _theta_block(variant, Q, K, scale):
    vecs = []
    for h in range(Q.shape[1]):
        d = Q.shape[-1]
        th = orc.fit(variant, scale * Q[:, h].reshape(-1, d).astype(np.float64), scale * K[:, h].reshape(-1, d).astype(np.float64))
        vecs.append(util.theta_vec_from_oracle(th))
    return np.stack(vecs)


def _assert_grads(got, ref, tol, where, floor=0.0):
    """Frobenius and per-row bounds for (dQ, dK, dV) of one (b, h).  A gradient that is zero by construction (a
    single key: Y = V_0 whatever Q and K are) is measured against `floor`, a small multiple of the scale of the
    output gradient, instead of against 0."""
    errs = [util.gradient_errors(g, r, floor) for g, r in zip(got, ref)]
    assert max(e[0] for e in errs) <= tol, (where, "frobenius", errs)
    assert max(e[1] for e in errs) <= 4 * tol, (where, "row", errs)
    return max(e[0] for e in errs), max(e[1] for e in errs)


def _check_backward(fs, Q, K, V, dY, Omega, scale, variant, dtype, tol, grad_dtype=None, causal=False):
    import torch
    B, H, Lq, d = Q.shape
    theta = _theta_block(variant, Q, K, scale)
    gQ, gK, gV = fs.attention_backward(torch.from_numpy(theta).cuda(), util.to_device(Q, dtype), util.to_device(K, dtype),
                                       util.to_device(V, dtype), util.to_device(dY, dtype), scale,
                                       torch.from_numpy(Omega).cuda(), causal=causal, grad_dtype=grad_dtype)
    torch.cuda.synchronize()
    gQ, gK, gV = util.to_host(gQ), util.to_host(gK), util.to_host(gV)
    assert np.isfinite(gQ).all() and np.isfinite(gK).all() and np.isfinite(gV).all()
    worst = 0.0
    for b in range(B):
        for h in range(H):
            th = util.oracle_theta_from_vec(theta[h], d)
            rq, rk, rv = orc.attention_backward(th, Omega[h], Q[b, h], K[b, h], V[b, h], dY[b, h], scale, causal)
            floor = max(0.5 * tol, 1e-3) * float(np.linalg.norm(dY[b, h]))   # scale for a gradient that is zero by construction
            fro, _ = _assert_grads((gQ[b, h], gK[b, h], gV[b, h]), (rq, rk, rv), tol, (b, h), floor)
            worst = max(worst, fro)
    return worst


@pytest.mark.parametrize("variant", ["sderf", "aderf", "saderf", "gerf"])
def test_backward_f32_small_ragged_different_lengths(fs, variant):
    rng = np.random.default_rng(61)
    B, H, Lq, Lk, d, dv, M = 2, 2, 70, 45, 12, 20, 50      # row starts must be 16-byte aligned: d, dv multiples of 4
    Q = (rng.standard_normal((B, H, Lq, d)) * np.linspace(0.5, 1.2, d) + 0.1).astype(np.float32)
    K = (rng.standard_normal((B, H, Lk, d)) * np.linspace(1.1, 0.6, d) - 0.05).astype(np.float32)
    V = rng.standard_normal((B, H, Lk, dv)).astype(np.float32)
    dY = rng.standard_normal((B, H, Lq, dv)).astype(np.float32)
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, variant, "f32", 3e-4)


@pytest.mark.parametrize("variant,L,d,M", [("saderf", 1300, 16, 40), ("aderf", 1100, 20, 130), ("saderf", 200, 68, 257),
                                           ("aderf", 210, 100, 60), ("saderf", 145, 128, 512)])
@pytest.mark.parametrize("causal", [False, True])
def test_backward_general_path_dense_quadratic_forms(fs, variant, L, d, M, causal):
    """A dense C where it is split over the waves: fewer, as many and more groups of sixteen coordinates than waves (row
    terms: four waves; gradient walks: four with M <= 64, else eight); 1100 and 1300 tokens are nine and eleven causal
    segments, whose prefix is formed eight at a time.  The bar of this file for fp32."""
    rng = np.random.default_rng(73 + d)
    Q, K = ((0.6 * rng.standard_normal((1, 1, L, d))).astype(np.float32) for _ in range(2))
    V, dY = (rng.standard_normal((1, 1, L, d)).astype(np.float32) for _ in range(2))
    Om = rng.standard_normal((1, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, variant, "f32", 3e-4, causal=causal)


@pytest.mark.parametrize("d,dv,M,B,L", [(8, 16, 250, 128, 500), (30, 30, 130, 64, 512), (64, 64, 150, 64, 300),       # four tiles of features per wave
                                        (16, 16, 70, 128, 512), (32, 20, 100, 128, 300), (48, 64, 120, 128, 300),     # two
                                        (66, 66, 40, 200, 300), (80, 96, 70, 128, 300), (128, 128, 100, 128, 300),     # two, rows of up to 96 and 128
                                        (128, 8, 17, 300, 1100), (16, 128, 33, 130, 260),
                                        (16, 16, 16, 300, 50), (64, 64, 20, 300, 40), (8, 64, 32, 300, 33), (24, 24, 64, 40, 300),   # causal walks with
                                        (36, 64, 33, 3, 150), (12, 60, 64, 2, 140), (128, 100, 40, 5, 70)])                         # few features
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_general_states_of_many_waves(fs, d, dv, M, B, L, causal, dtype):
    """Calls large enough for a wave of the state kernel to take two or four tiles of features, with remainders of tiles and of
    segments, and calls on either side of the rules that choose the causal kernels: attention and its gradients of the first, a middle and the last sequence against float64 on the same inputs.  The
    bars of this file: 1e-4 for the output, three times that for gradients."""
    import torch
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(d + M + L)

    def rows(n, scale=1.0):
        x = scale * torch.randn((B, 1, L, (n + 7) // 8 * 8), generator=gen, device="cuda")
        return x.to(dt)[..., :n]
    Q, K, V, dY = rows(d, 0.7), rows(d, 0.7), rows(dv), rows(dv)
    Om = torch.randn((1, M, d), generator=gen, device="cuda")
    rng = np.random.default_rng(d)
    theta = util.theta_vec_from_oracle(orc.fit("saderf", 0.5 * rng.standard_normal((400, d)), 0.4 * rng.standard_normal((400, d))))
    th, s = util.oracle_theta_from_vec(theta, d), d ** -0.25
    td = torch.from_numpy(theta[None]).cuda()

    def out(n):
        return torch.full((B, 1, L, (n + 7) // 8 * 8), float("nan"), device="cuda")[..., :n]
    Y = fs.attention(td, Q, K, V, s, Om, causal=causal, out=out(dv))
    grads = fs.attention_backward(td, Q, K, V, dY, s, Om, causal=causal, grads=(out(d), out(d), out(dv)))
    om = Om[0].double()
    A, B1, B2, C2 = (torch.from_numpy(np.asarray(x, dtype=np.float64)).cuda() for x in (th.A, th.B1, th.B2, th.C2))
    for b in (0, B // 2, B - 1):
        q, k, v = (x[b, 0].double().requires_grad_(True) for x in (Q, K, V))
        bias = (om * om) @ A
        E1, E2 = s * q @ (om @ B1).T + bias, s * k @ (om @ B2).T + bias + s * s * ((k @ C2) * k).sum(1, keepdim=True)
        W = torch.exp(E1 - E1.detach().max(1, keepdim=True).values) @ torch.exp(E2 - E2.detach().max()).T
        if causal:
            W = torch.tril(W)
        ref = (W @ v) / W.sum(1, keepdim=True)
        gref = torch.autograd.grad((ref * dY[b, 0].double()).sum(), (q, k, v))
        err = float((Y[b, 0].double() - ref.detach()).norm() / ref.detach().norm())
        assert err <= 1e-4, (b, err)
        for g, r, name in zip(grads, gref, ("dQ", "dK", "dV")):
            fro, row = util.gradient_errors(g[b, 0].double().cpu().numpy(), r.cpu().numpy())
            assert fro <= 3e-4 and row <= 1.2e-3, (b, name, fro, row)


@pytest.mark.parametrize("d,dv,M,L,B", [(20, 28, 129, 31, 3), (32, 44, 256, 65, 3), (64, 60, 140, 40, 3), (36, 64, 257, 97, 3),
                                        (60, 36, 512, 130, 3), (32, 20, 65, 70, 3), (128, 124, 70, 33, 3), (100, 128, 130, 64, 3),
                                        (96, 68, 300, 100, 3), (128, 80, 511, 160, 3), (20, 28, 257, 100, 16000),
                                        (20, 28, 129, 63, 3), (32, 44, 256, 81, 300), (64, 60, 140, 17, 3), (60, 76, 200, 50, 3), (32, 20, 65, 49, 3),
                                        (128, 124, 70, 55, 3), (100, 128, 130, 33, 3), (24, 40, 200, 17, 3), (64, 60, 140, 16, 3), (32, 44, 256, 48, 300)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_general_causal_calls_on_bf16_matrix_instructions(fs, d, dv, M, L, B, dtype):
    """Causal calls whose fp32 products run on bf16 pieces: remainders of tokens, coordinates, value columns (one and two blocks of
    them, with the normaliser in either) and features (one and two launches; 16000 sequences: in two parts, as partial rows take
    at most 256 MB)."""
    test_general_states_of_many_waves(fs, d, dv, M, B, L, True, dtype)


@pytest.mark.parametrize("below", [96, 110, 121])
@pytest.mark.parametrize("d,M,dtype", [(32, 160, "f32"), (64, 300, "f32"), (48, 100, "bf16"), (128, 300, "bf16")])
def test_general_causal_rows_whose_keys_lie_far_below_the_largest(fs, d, M, dtype, below):
    """The first 40 keys have all their features 2^-`below` times those of the others (a coordinate of their own in C2 that no
    projection sees), down to 2^-125 of the largest: with one shift per sequence fp32 holds them to the rounding of their exponents,
    2^-18 for numbers between 64 and 128.  Four of those (projection, row term, sum, shift) are 1.1e-5 of a feature; outputs of the
    first rows divide two sums of them, gradients multiply another two."""
    import torch
    L, n, s = 100, 40, d ** -0.25
    gen = torch.Generator(device="cuda").manual_seed(d + M + below)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = (f * torch.randn((1, 1, L, d), generator=gen, device="cuda") for f in (0.1, 0.1, 1.0, 1.0))
    Q[..., 0] = K[..., 0] = 0.0
    K[:, :, :n, 0] = 1.0
    Q, K, V, dY = (x.to(dt) for x in (Q, K, V, dY))
    Om = torch.randn((1, M, d), generator=gen, device="cuda")
    B, C2 = np.eye(d), np.zeros((d, d))
    B[0, 0], C2[0, 0] = 0.0, -below * np.log(2.0) / s ** 2
    th = orc.Theta(logD=0.0, A=np.zeros(d), B1=B, B2=B, C1=-0.5 * np.eye(d), C2=C2)
    td = torch.from_numpy(util.theta_vec_from_oracle(th)[None]).cuda()
    Y = fs.attention(td, Q, K, V, s, Om, causal=True, out_dtype=torch.float32)
    grads = fs.attention_backward(td, Q, K, V, dY, s, Om, causal=True, grad_dtype=torch.float32)
    q, k, v = (x[0, 0].double().requires_grad_(True) for x in (Q, K, V))
    om, c2 = Om[0].double(), float(td[0, 8 + d + 3 * d * d])
    om[:, 0] = 0.0
    W = torch.tril(torch.exp(s * q @ om.T) @ torch.exp(s * k @ om.T + s * s * c2 * k[:, :1] ** 2).T)
    ref = (W @ v) / W.sum(1, keepdim=True)
    gref = torch.autograd.grad((ref * dY[0, 0].double()).sum(), (q, k, v))
    errs = [float((a[0, 0, :n].double() - r[:n]).norm() / r[:n].norm()) for a, r in zip((Y, *grads), (ref.detach(), *gref))]
    print(d, M, dtype, below, " ".join("%.2e" % e for e in errs))
    assert errs[0] <= 2.2e-5 and max(errs[1:]) <= 4.4e-5, errs


@pytest.mark.parametrize("d,M,dtype", [(32, 160, "f32"), (48, 100, "bf16"), (128, 300, "bf16")])
def test_general_causal_rows_that_see_no_key_are_zero_and_counted(fs, d, M, dtype):
    """Keys 2^-170 below the largest: none of their features is a number of fp32.  Rows that see only them get zeros, outputs and
    gradients, and are counted; the others are as without those keys."""
    import torch
    L, n, s = 100, 40, d ** -0.25
    gen = torch.Generator(device="cuda").manual_seed(d + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = (f * torch.randn((2, 1, L, d), generator=gen, device="cuda") for f in (0.1, 0.1, 1.0, 1.0))
    Q[..., 0] = K[..., 0] = 0.0
    K[:, :, :n, 0] = 1.0
    Q, K, V, dY = (x.to(dt) for x in (Q, K, V, dY))
    Om = torch.randn((1, M, d), generator=gen, device="cuda")
    B, C2 = np.eye(d), np.zeros((d, d))
    B[0, 0], C2[0, 0] = 0.0, -170.0 * np.log(2.0) / s ** 2
    td = torch.from_numpy(util.theta_vec_from_oracle(orc.Theta(logD=0.0, A=np.zeros(d), B1=B, B2=B, C1=-0.5 * np.eye(d), C2=C2))[None]).cuda()
    ws = torch.empty(fs.attention_backward_workspace_bytes(2, 1, L, L, d, d, M, True, 1, 1), dtype=torch.uint8, device="cuda")
    Y = fs.attention(td, Q, K, V, s, Om, causal=True, workspace=ws)
    assert fs.attention_flushed_rows(ws) == 2 * n
    grads = fs.attention_backward(td, Q, K, V, dY, s, Om, causal=True, workspace=ws)
    assert fs.attention_flushed_rows(ws) == 2 * n
    assert all(bool((x[:, :, :n] == 0).all()) and bool(torch.isfinite(x).all()) for x in (Y, *grads))
    Qr, Kr, Vr, dYr = (x[:, :, n:] for x in (Q, K, V, dY))
    tail = (fs.attention(td, Qr, Kr, Vr, s, Om, causal=True), *fs.attention_backward(td, Qr, Kr, Vr, dYr, s, Om, causal=True))
    # (sums of other chunks: fp32 rounding, and that of the outputs' type)
    tol = 1e-5 if dtype == "f32" else 4e-3
    for x, y in zip((Y, *grads), tail):
        assert float((x[:, :, n:].double() - y.double()).norm()) <= tol * float(y.double().norm())


@pytest.mark.parametrize("tg,og", [("H", "H"), ("BH", "1"), ("1", "BH"), ("BH", "H")])
@pytest.mark.parametrize("variant", ["sderf", "saderf", "aderf"])
@pytest.mark.parametrize("d,M,dtype", [(64, 256, "f32"), (28, 300, "f32"), (128, 300, "bf16"), (64, 100, "bf16")])
def test_general_causal_calls_with_parameters_per_head_and_sequence(fs, d, M, dtype, variant, tg, og):
    """Parameter sets and omegas of their own for heads and sequences, in every combination, isotropic and dense families, one launch
    and two: attention and gradients of every sequence against float64, at this file's bars."""
    import torch
    B, H, L, s = 2, 3, 90, d ** -0.25
    gen = torch.Generator(device="cuda").manual_seed(d + M)
    rng = np.random.default_rng(d)
    count = {"1": 1, "H": H, "BH": B * H}
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = ((f * torch.randn((B, H, L, d), generator=gen, device="cuda")).to(dt) for f in (0.7, 0.7, 1.0, 1.0))
    Om = torch.randn((count[og], M, d), generator=gen, device="cuda")
    ths = [orc.fit(variant, (0.3 + 0.1 * i) * rng.standard_normal((4 * d, d)), 0.4 * rng.standard_normal((4 * d, d))) for i in range(count[tg])]
    td = torch.from_numpy(np.stack([util.theta_vec_from_oracle(t) for t in ths])).cuda()
    Y = fs.attention(td, Q, K, V, s, Om, causal=True, out_dtype=torch.float32)
    grads = fs.attention_backward(td, Q, K, V, dY, s, Om, causal=True, grad_dtype=torch.float32)
    for b in range(B):
        for h in range(H):
            at = {"1": 0, "H": h, "BH": b * H + h}
            th, om = util.oracle_theta_from_vec(td[at[tg]].cpu().numpy(), d), Om[at[og]].double()
            A, B1, B2, C2 = (torch.from_numpy(np.asarray(x, dtype=np.float64)).cuda() for x in (th.A, th.B1, th.B2, th.C2))
            q, k, v = (x[b, h].double().requires_grad_(True) for x in (Q, K, V))
            bias = (om * om) @ A
            E1, E2 = s * q @ (om @ B1).T + bias, s * k @ (om @ B2).T + bias + s * s * ((k @ C2) * k).sum(1, keepdim=True)
            W = torch.tril(torch.exp(E1 - E1.detach().max(1, keepdim=True).values) @ torch.exp(E2 - E2.detach().max()).T)
            ref = (W @ v) / W.sum(1, keepdim=True)
            gref = torch.autograd.grad((ref * dY[b, h].double()).sum(), (q, k, v))
            assert float((Y[b, h].double() - ref.detach()).norm() / ref.detach().norm()) <= 1e-4, (b, h)
            for g, r, name in zip(grads, gref, ("dQ", "dK", "dV")):
                fro, row = util.gradient_errors(g[b, h].double().cpu().numpy(), r.cpu().numpy())
                assert fro <= 3e-4 and row <= 1.2e-3, (b, h, name, fro, row)


@pytest.mark.parametrize("kv,kd", [(-120, 0), (-110, 20), (0, -118), (-60, -60), (105, 0), (0, 100), (60, 40)])
@pytest.mark.parametrize("d,M,dtype", [(32, 160, "f32"), (64, 300, "f32"), (48, 100, "bf16"), (128, 300, "bf16")])
def test_general_causal_values_of_any_size(fs, d, M, dtype, kv, kd):
    """V and dY of one sequence near 2^kv and 2^kd, of its neighbours near one (the last: its first 40 rows of V and last 40 of dY
    2^-80 of the others): outputs and gradients as near to float64 as fp32 sums are, each sequence by itself."""
    import torch
    L, n, s = 100, 40, d ** -0.25
    gen = torch.Generator(device="cuda").manual_seed(d + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = (f * torch.randn((3, 1, L, d), generator=gen, device="cuda") for f in (0.5, 0.5, 1.0, 1.0))
    V[1] *= 2.0 ** kv
    dY[1] *= 2.0 ** kd
    V[2, :, :n] *= 2.0 ** -80
    dY[2, :, -n:] *= 2.0 ** -80
    Q, K, V, dY = (x.to(dt) for x in (Q, K, V, dY))
    Om = torch.randn((1, M, d), generator=gen, device="cuda")
    td = torch.from_numpy(util.theta_vec_from_oracle(orc.fit_posrf(d))[None]).cuda()
    Y = fs.attention(td, Q, K, V, s, Om, causal=True, out_dtype=torch.float32)
    grads = fs.attention_backward(td, Q, K, V, dY, s, Om, causal=True, grad_dtype=torch.float32)
    om = Om[0].double()
    for b in range(3):
        q, k, v = (x[b, 0].double().requires_grad_(True) for x in (Q, K, V))
        W = torch.tril(torch.exp(s * q @ om.T) @ torch.exp(s * k @ om.T - 0.5 * s * s * (k * k).sum(1, keepdim=True)).T)
        ref = (W @ v) / W.sum(1, keepdim=True)
        gref = torch.autograd.grad((ref * dY[b, 0].double()).sum(), (q, k, v))
        for x, r, name in zip((Y, *grads), (ref.detach(), *gref), "YQKV"):
            for part in ((slice(0, n), slice(n, L - n), slice(L - n, L)) if b == 2 and name in "YV" else (slice(0, L),)):
                assert float((x[b, 0, part].double() - r[part]).norm() / r[part].norm()) <= 1.2e-5, (b, name, part)


@pytest.mark.parametrize("values,lefts", [((-100, 20), (0, 0)), ((-60, 60), (60, 0)), ((-20, 100), (0, 0)), ((0, 0), (0, -105)),
                                          ((0, 0), (20, -90)), ((0, 60), (60, -60)), ((-90, 30), (30, -80))])
@pytest.mark.parametrize("d,M,dtype", [(32, 160, "f32"), (64, 300, "f32"), (48, 100, "bf16"), (128, 300, "bf16")])
def test_general_causal_rows_of_every_size_in_one_sequence(fs, d, M, dtype, values, lefts):
    """The first 40 rows of V near 2^values[0], the others near 2^values[1]; dY near 2^lefts[0] but for its last 40 rows, 2^lefts[1];
    with an infinity among the last, which none of the first rows sees.  Rows of both ends as near to float64 as fp32 sums are."""
    import torch
    L, n, s = 100, 40, d ** -0.25
    gen = torch.Generator(device="cuda").manual_seed(d + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = (f * torch.randn((1, 1, L, d), generator=gen, device="cuda") for f in (0.5, 0.5, 1.0, 1.0))
    V[:, :, :n] *= 2.0 ** values[0]
    V[:, :, n:] *= 2.0 ** values[1]
    dY[:, :, :-n] *= 2.0 ** lefts[0]
    dY[:, :, -n:] *= 2.0 ** lefts[1]
    Q, K, V, dY = (x.to(dt) for x in (Q, K, V, dY))
    Om = torch.randn((1, M, d), generator=gen, device="cuda")
    td = torch.from_numpy(util.theta_vec_from_oracle(orc.fit_posrf(d))[None]).cuda()
    om = Om[0].double()
    q, k, v = (x[0, 0].double().requires_grad_(True) for x in (Q, K, V))
    W = torch.tril(torch.exp(s * q @ om.T) @ torch.exp(s * k @ om.T - 0.5 * s * s * (k * k).sum(1, keepdim=True)).T)
    ref = (W @ v) / W.sum(1, keepdim=True)
    gref = torch.autograd.grad((ref * dY[0, 0].double()).sum(), (q, k, v))
    for infinite in (False, True):
        if infinite:
            V = V.clone()
            V[:, :, -1, 0] = float("inf")
        got = (fs.attention(td, Q, K, V, s, Om, causal=True, out_dtype=torch.float32),
               *fs.attention_backward(td, Q, K, V, dY, s, Om, causal=True, grad_dtype=torch.float32))
        for x, r, name in zip(got, (ref.detach(), *gref), "YQKV"):
            if infinite and name == "K":
                continue
            for part in (slice(0, n), slice(n, L - n), slice(L - n, L))[:1 if infinite else 3]:
                assert float((x[0, 0, part].double() - r[part]).norm() / r[part].norm()) <= 1.2e-5, (infinite, name, part)


@pytest.mark.parametrize("row", [42, 58])
@pytest.mark.parametrize("d,M,dtype", [(32, 160, "f32"), (64, 300, "f32"), (48, 100, "bf16"), (128, 300, "bf16")])
def test_general_causal_rows_that_are_not_finite_stay_in_their_tile(fs, d, M, dtype, row):
    """A row of V that is not finite leaves the outputs and the gradients of Q as they are in all tiles of sixteen rows before
    its own, one of dY or Q the gradients of K and V in those behind it: masked scores are zeros, but zeros times such a number are
    not."""
    import torch
    L, s, tile = 100, d ** -0.25, row // 16 * 16
    gen = torch.Generator(device="cuda").manual_seed(d + M)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = ((f * torch.randn((1, 1, L, d), generator=gen, device="cuda")).to(dt) for f in (0.5, 0.5, 1.0, 1.0))
    Om = torch.randn((1, M, d), generator=gen, device="cuda")
    td = torch.from_numpy(util.theta_vec_from_oracle(orc.fit_posrf(d))[None]).cuda()

    def call(*args):
        return (fs.attention(td, *args[:3], s, Om, causal=True), *fs.attention_backward(td, *args, s, Om, causal=True))
    Y, dQ, dK, dV = call(Q, K, V, dY)
    for value in (float("inf"), float("nan")):
        V2, dY2 = V.clone(), dY.clone()
        V2[:, :, row, 3] = dY2[:, :, row, 3] = value
        got = call(Q, K, V2, dY)
        assert torch.equal(got[0][:, :, :tile], Y[:, :, :tile]) and torch.equal(got[1][:, :, :tile], dQ[:, :, :tile])
        assert not bool(torch.isfinite(got[0][:, :, row:, 3]).any())
        assert torch.equal(got[0][..., :3], Y[..., :3]) and torch.equal(got[0][..., 4:], Y[..., 4:])
        got = call(Q, K, V, dY2)
        assert torch.equal(got[0], Y)
        assert torch.equal(got[2][:, :, tile + 16:], dK[:, :, tile + 16:]) and torch.equal(got[3][:, :, tile + 16:], dV[:, :, tile + 16:])
        assert not bool(torch.isfinite(got[3][:, :, :row + 1, 3]).any())
    Q2 = Q.clone()
    Q2[:, :, row] = float("nan")
    got = call(Q2, K, V, dY)
    assert torch.equal(got[0][:, :, :tile], Y[:, :, :tile]) and torch.equal(got[0][:, :, tile + 16:], Y[:, :, tile + 16:])
    assert torch.equal(got[2][:, :, tile + 16:], dK[:, :, tile + 16:]) and torch.equal(got[3][:, :, tile + 16:], dV[:, :, tile + 16:])


@pytest.mark.parametrize("d,M,causal", [(8, 40, False), (16, 16, False), (18, 40, False), (32, 70, False), (36, 40, False), (64, 33, False),
                                        (80, 40, False), (128, 40, False), (16, 40, True), (64, 130, True), (18, 40, True), (24, 520, True)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward_general_path_weights_of_every_row_sum_to_one(fs, d, M, causal, dtype):
    """The rows of K_hat over their normalisers sum to one, so sum_j dV_j = sum_i dY_i, but only as far as the features that the
    gradient sums are those whose sum the normaliser is: with exponents of 2e5 a projection that is rounded in another order is
    off by up to 2e-3.  All terms are positive: 2^-24 for each of at most 2 (L + M) additions in a row, and for the exponents' own
    few roundings of the keys (below 16: 1e-6)."""
    import torch
    rng = np.random.default_rng(90 + d + M)
    L = 300
    Om = rng.standard_normal((1, M, d)).astype(np.float32)
    Q = rng.standard_normal((1, 1, L, d))
    Q *= 2e5 / (np.log2(np.e) * np.abs(Q[0, 0] @ Om[0].T.astype(np.float64)).max(1)[None, None, :, None])
    K = 0.1 * rng.standard_normal((1, 1, L, d))
    V = rng.standard_normal((1, 1, L, d))
    dY = 0.5 + rng.random((1, 1, L, d))
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    width = (d + 7) // 8 * 8               # rows start at multiples of 16 bytes

    def dev(x, t=dt):
        y = torch.zeros((1, 1, L, width), dtype=t, device="cuda")
        y[..., :d] = torch.from_numpy(x).to(t)
        return y[..., :d]
    th = orc.Theta(logD=0.0, A=np.zeros(d), B1=np.eye(d), B2=np.eye(d), C1=-0.5 * np.eye(d), C2=-0.5 * np.eye(d))
    theta = torch.from_numpy(util.theta_vec_from_oracle(th)[None]).cuda()
    dYd = dev(dY)
    grads = tuple(dev(np.zeros((1, 1, L, d)), torch.float32) for _ in range(3))
    fs.attention_backward(theta, dev(Q), dev(K), dev(V), dYd, 1.0, torch.from_numpy(Om).cuda(), causal=causal, grads=grads)
    got, want = grads[2][0, 0].double().sum(0), dYd[0, 0].double().sum(0)
    rel = float(((got - want).abs() / want).max())
    assert rel <= 2 * (L + M) * 2.0 ** -24 + 1e-6, rel


@pytest.mark.parametrize("L,M,d,dv", [(1, 1, 4, 4), (33, 16, 8, 4), (64, 200, 128, 128)])
def test_backward_degenerate_and_maximum_sizes(fs, L, M, d, dv):
    rng = np.random.default_rng(62)
    Q = (0.7 * rng.standard_normal((1, 1, L, d))).astype(np.float32)
    K = (0.7 * rng.standard_normal((1, 1, L, d))).astype(np.float32)
    V = rng.standard_normal((1, 1, L, dv)).astype(np.float32)
    dY = rng.standard_normal((1, 1, L, dv)).astype(np.float32)
    Om = rng.standard_normal((1, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, "sderf" if L > 1 else "posrf", "f32", 3e-4)


def test_backward_c3_shape_bf16_inputs(fs):
    """The non-causal bf16 workload at its real d, M and statistics, shortened so the oracle finishes in seconds.
    This shape runs on the bf16 MFMA kernels (bf16 operands, fp32 accumulation): the bar is the bf16 one, 2e-2, for
    fp32 and for bf16 gradients.  The length is not a multiple of the tile sizes (ragged tails in every kernel)."""
    w = synth.make("c3", B=2, H=2, L=712)
    rng = np.random.default_rng(63)
    dY = synth.round_to_bf16(rng.standard_normal(w["V"].shape).astype(np.float32))
    import torch
    worst = _check_backward(fs, w["Q"], w["K"], w["V"], dY, w["Omega"], w["qk_scale"], "sderf", "bf16", 2e-2,
                            grad_dtype=torch.float32)
    assert worst > 0.0
    _check_backward(fs, w["Q"], w["K"], w["V"], dY, w["Omega"], w["qk_scale"], "sderf", "bf16", 2e-2)


@pytest.mark.parametrize("variant", ["aderf", "saderf", "gerf"])
def test_backward_bf16_path_other_families_and_lengths(fs, variant):
    """Dense C (ADERF: row terms from the precomputed table, dense derivative of the row term), diagonal C (SADERF)
    and the scalar family on the bf16 kernels, with different numbers of queries and keys."""
    import torch
    rng = np.random.default_rng(65)
    B, H, Lq, Lk, d, M = 1, 2, 200, 333, 64, 256
    sc = np.linspace(0.6, 1.1, d)
    Q = synth.round_to_bf16((rng.standard_normal((B, H, Lq, d)) * sc + 0.05).astype(np.float32))
    K = synth.round_to_bf16((rng.standard_normal((B, H, Lk, d)) * sc[::-1] - 0.05).astype(np.float32))
    V = synth.round_to_bf16(rng.standard_normal((B, H, Lk, d)).astype(np.float32))
    dY = synth.round_to_bf16(rng.standard_normal((B, H, Lq, d)).astype(np.float32))
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, variant, "bf16", 2e-2, grad_dtype=torch.float32)


@pytest.mark.parametrize("variant,B,H,Lq,Lk,f32", [("sderf", 1, 2, 128, 128, True), ("aderf", 1, 2, 100, 120, True),
                                                   ("saderf", 2, 2, 64, 190, False), ("gerf", 48, 8, 300, 200, False),
                                                   ("aderf", 64, 8, 70, 333, True), ("posrf", 1, 3, 1, 190, True)])
def test_backward_bf16_path_whole_sequences_per_workgroup(fs, variant, B, H, Lq, Lk, f32):
    """Non-causal calls with many sequences (B*H >= 384) or short ones (at most four chunks of queries and keys
    together) run the whole backward pass of a sequence in one workgroup, both states staying on chip: equal and
    different numbers of queries and keys, ragged tails, isotropic and dense key-side quadratic forms, fp32 output
    gradients into fp32 gradients and bf16 into bf16 (every seventh batch entry against the oracle)."""
    import torch
    rng = np.random.default_rng(67 + Lq + Lk)
    d, M = 64, 256
    sc = np.linspace(0.6, 1.1, d)
    Q = synth.round_to_bf16((rng.standard_normal((B, H, Lq, d)) * sc + 0.05).astype(np.float32))
    K = synth.round_to_bf16((rng.standard_normal((B, H, Lk, d)) * sc[::-1] - 0.05).astype(np.float32))
    V = synth.round_to_bf16(rng.standard_normal((B, H, Lk, d)).astype(np.float32))
    dY = rng.standard_normal((B, H, Lq, d)).astype(np.float32)
    if not f32:
        dY = synth.round_to_bf16(dY)
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    scale = d ** -0.25
    theta = _theta_block(variant, Q[::7], K[::7], scale)
    gQ, gK, gV = fs.attention_backward(torch.from_numpy(theta).cuda(), util.to_device(Q, "bf16"), util.to_device(K, "bf16"),
                                       util.to_device(V, "bf16"), util.to_device(dY, "f32" if f32 else "bf16"), scale,
                                       torch.from_numpy(Om).cuda(), causal=False,
                                       grad_dtype=torch.float32 if f32 else torch.bfloat16)
    torch.cuda.synchronize()
    gQ, gK, gV = util.to_host(gQ), util.to_host(gK), util.to_host(gV)
    assert np.isfinite(gQ).all() and np.isfinite(gK).all() and np.isfinite(gV).all()
    worst = (0.0, 0.0)
    for b in range(0, B, 7):
        for h in range(H):
            th = util.oracle_theta_from_vec(theta[h], d)
            ref = orc.attention_backward(th, Om[h], Q[b, h], K[b, h], V[b, h], dY[b, h], scale, False)
            floor = 1e-2 * float(np.linalg.norm(dY[b, h]))
            e = _assert_grads((gQ[b, h], gK[b, h], gV[b, h]), ref, 2e-2, (b, h), floor)
            worst = (max(worst[0], e[0]), max(worst[1], e[1]))
    print(f"backward, whole sequences, B={B} H={H} Lq={Lq} Lk={Lk} {variant}: worst frobenius {worst[0]:.2e}, "
          f"worst row {worst[1]:.2e}")


@pytest.mark.parametrize("variant", ["gerf", "saderf"])
@pytest.mark.parametrize("H,Lq,Lk,f32", [(1, 1, 400, False), (3, 15, 700, True), (20, 129, 1000, False), (2, 2049, 1039, False),   # one row tile per wave
                                         (33, 1999, 130, False), (70, 100, 1121, True), (65, 1041, 1025, False),                # two: queries, keys, both
                                         (50, 1100, 1030, False), (104, 515, 520, False), (150, 3990, 3970, False),   # 2 or 5 parts in one pass, 3 in two
                                         (64, 1000, 1500, False), (64, 1200, 1700, False),              # slots of 4 and of 5 chunks of queries, 6 and 7 of keys
                                         (385, 800, 780, False)])                                                               # longest whole, then rows
def test_backward_bf16_path_row_tiles(fs, variant, H, Lq, Lk, f32):
    """The row-split gradient kernels in each of their row-tile widths, with remainders of tiles, steps and workgroups.
    Reference: float64 chain rule on the same bf16 inputs and the kernels' bf16 projection matrices."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(H + Lq + Lk)
    Q, K, V, dY = (torch.randn((1, H, L, 64), generator=gen, device="cuda") for L in (Lq, Lk, Lk, Lq))
    Q, K, V = (x.bfloat16() for x in (Q, K, V))
    dY = dY if f32 else dY.bfloat16()
    Om = torch.randn((1, 256, 64), generator=gen, device="cuda")
    rng = np.random.default_rng(7)
    vec = util.theta_vec_from_oracle(orc.fit(variant, 0.35 * rng.standard_normal((400, 64)), 0.4 * rng.standard_normal((400, 64))))
    th, s = util.oracle_theta_from_vec(vec, 64), 64 ** -0.25
    grads = tuple(torch.full((1, H, L, 64), float("nan"), dtype=dY.dtype, device="cuda") for L in (Lq, Lk, Lk))
    got = fs.attention_backward(torch.from_numpy(vec[None]).cuda(), Q, K, V, dY, s, Om, grads=grads)
    log2e = float(np.log2(np.e))
    W1, W2 = ((log2e * s * (Om[0] @ torch.from_numpy(Bm).float().cuda())).bfloat16().double() / log2e for Bm in (th.B1, th.B2))
    bias = (Om[0].double() ** 2) @ torch.from_numpy(th.A).cuda()
    C2 = s * s * torch.from_numpy(th.C2).cuda()
    for h in sorted({0, H // 2, H - 1}):
        q, k, v = (x[0, h].double().requires_grad_(True) for x in (Q, K, V))
        E1, E2 = q @ W1.T + bias, k @ W2.T + bias + ((k @ C2) * k).sum(1, keepdim=True)
        P = torch.exp(E1 - E1.detach().max(1, keepdim=True).values)
        S = torch.exp(E2 - E2.detach().max())
        Y = (P @ (S.T @ v)) / (P @ S.sum(0))[:, None]
        ref = torch.autograd.grad((Y * dY[0, h].double()).sum(), (q, k, v))
        # (one key: the gradients of Q and K vanish by construction; their rounding is measured against dY and V)
        floor = 1e-3 * float(dY[0, h].double().norm() * V[0, h].double().norm(dim=1).max())
        for g, r, name in zip(got, ref, ("dQ", "dK", "dV")):
            fro, row = util.gradient_errors(g[0, h].double().cpu().numpy(), r.cpu().numpy(), floor)
            assert fro <= 2e-2 and row <= 8e-2, (h, name, fro, row)


def test_backward_whole_sequences_per_workgroup_is_bitwise_reproducible(fs):
    """The one-workgroup backward pass reuses one LDS region for six loops and a transposition, ordered by workgroup
    barriers only, and reads back rows of G1 that the same workgroup wrote to memory: a missing barrier would show up
    as run-to-run differences (512 sequences of 200 rows, five repetitions, other work in between), and the forward
    call of the same shape must be reproducible too."""
    import torch
    torch.manual_seed(5)
    B, H, L, d, M = 64, 8, 200, 64, 256
    Q, K, V, dY = (torch.randn(B, H, L, d, device="cuda").to(torch.bfloat16) for _ in range(4))
    Om = torch.randn(H, M, d, device="cuda")
    s = d ** -0.25
    theta = fs.fit_params("aderf", Q, K, s, groups=H)
    first = [g.clone() for g in fs.attention_backward(theta, Q, K, V, dY, s, Om, causal=False)]
    y0 = fs.attention(theta, Q, K, V, s, Om, causal=False).clone()
    assert all(torch.isfinite(g.float()).all().item() for g in first)
    for rep in range(5):
        scratch = torch.randn(1 << 22, device="cuda").sum().item()
        again = fs.attention_backward(theta, Q, K, V, dY, s, Om, causal=False)
        for a, b in zip(first, again):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (rep, scratch)
        assert torch.equal(y0.view(torch.int16), fs.attention(theta, Q, K, V, s, Om, causal=False).view(torch.int16))


def test_backward_value_gradients_sum_to_output_gradients_at_full_c3_size(fs):
    """At the full size of the non-causal workload the oracle cannot run; what holds at any size: the attention
    weights of a row sum to one, so sum_j dV_j = sum_i dY_i per (b, h); and sampled rows of dV against the oracle's
    weights W^T dY restricted to a subset of the queries' contribution is not available, so only the invariant is
    checked here."""
    import torch
    w = synth.make("c3")
    rng = np.random.default_rng(64)
    dY = synth.round_to_bf16(rng.standard_normal(w["V"].shape).astype(np.float32))
    theta = _theta_block("sderf", w["Q"][:1], w["K"][:1], w["qk_scale"])
    gQ, gK, gV = fs.attention_backward(torch.from_numpy(theta).cuda(), util.to_device(w["Q"], "bf16"),
                                       util.to_device(w["K"], "bf16"), util.to_device(w["V"], "bf16"),
                                       util.to_device(dY, "bf16"), w["qk_scale"], torch.from_numpy(w["Omega"]).cuda(),
                                       grad_dtype=torch.float32)
    torch.cuda.synchronize()
    gV = util.to_host(gV).astype(np.float64)
    assert np.isfinite(util.to_host(gQ)).all() and np.isfinite(util.to_host(gK)).all()
    want = dY.astype(np.float64).sum(axis=2)
    got = gV.sum(axis=2)
    scale = np.abs(dY).astype(np.float64).sum(axis=2).max()
    # bf16 kernels: every dV row carries a relative rounding error of about 2^-9; the column sums of 4096 of them
    # against the sum of absolute values
    assert np.abs(got - want).max() <= 1e-3 * scale


@pytest.mark.parametrize("variant", ["sderf", "aderf", "saderf", "gerf"])
def test_backward_causal_f32_small_ragged(fs, variant):
    """Causal variant: several segments, several 32-row steps per segment and a ragged tail."""
    rng = np.random.default_rng(71)
    B, H, L, d, dv, M = 2, 2, 333, 12, 20, 50
    Q = (rng.standard_normal((B, H, L, d)) * np.linspace(0.5, 1.2, d) + 0.1).astype(np.float32)
    K = (rng.standard_normal((B, H, L, d)) * np.linspace(1.1, 0.6, d) - 0.05).astype(np.float32)
    V = rng.standard_normal((B, H, L, dv)).astype(np.float32)
    dY = rng.standard_normal((B, H, L, dv)).astype(np.float32)
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, variant, "f32", 3e-4, causal=True)


@pytest.mark.parametrize("L,M,d,dv", [(1, 1, 4, 4), (33, 16, 8, 4), (64, 200, 128, 128)])
def test_backward_causal_degenerate_and_maximum_sizes(fs, L, M, d, dv):
    rng = np.random.default_rng(72)
    Q = (0.7 * rng.standard_normal((1, 1, L, d))).astype(np.float32)
    K = (0.7 * rng.standard_normal((1, 1, L, d))).astype(np.float32)
    V = rng.standard_normal((1, 1, L, dv)).astype(np.float32)
    dY = rng.standard_normal((1, 1, L, dv)).astype(np.float32)
    Om = rng.standard_normal((1, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, "sderf" if L > 1 else "posrf", "f32", 3e-4, causal=True)


def test_backward_causal_c4_shape_bf16_inputs(fs):
    """The causal bf16 workload at its real d, M and statistics, shortened so the oracle finishes in seconds: bf16
    MFMA kernels, bar 2e-2.  Several slots per sequence, several chunks per slot and a ragged tail."""
    import torch
    w = synth.make("c4", B=1, H=2, L=1216)
    rng = np.random.default_rng(73)
    dY = synth.round_to_bf16(rng.standard_normal(w["V"].shape).astype(np.float32))
    _check_backward(fs, w["Q"], w["K"], w["V"], dY, w["Omega"], w["qk_scale"], "sderf", "bf16", 2e-2,
                    grad_dtype=torch.float32, causal=True)
    _check_backward(fs, w["Q"], w["K"], w["V"], dY, w["Omega"], w["qk_scale"], "sderf", "bf16", 2e-2, causal=True)


@pytest.mark.parametrize("variant,L", [("aderf", 333), ("saderf", 64), ("gerf", 100)])
def test_backward_causal_bf16_path_other_families_and_lengths(fs, variant, L):
    import torch
    rng = np.random.default_rng(75)
    B, H, d, M = 1, 2, 64, 256
    sc = np.linspace(0.6, 1.1, d)
    Q = synth.round_to_bf16((rng.standard_normal((B, H, L, d)) * sc + 0.05).astype(np.float32))
    K = synth.round_to_bf16((rng.standard_normal((B, H, L, d)) * sc[::-1] - 0.05).astype(np.float32))
    V = synth.round_to_bf16(rng.standard_normal((B, H, L, d)).astype(np.float32))
    dY = synth.round_to_bf16(rng.standard_normal((B, H, L, d)).astype(np.float32))
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    _check_backward(fs, Q, K, V, dY, Om, d ** -0.25, variant, "bf16", 2e-2, grad_dtype=torch.float32, causal=True)


@pytest.mark.parametrize("variant,L", [("sderf", 200), ("aderf", 128), ("gerf", 333)])
def test_backward_causal_one_slot_per_sequence(fs, variant, L):
    """Causal calls with 256 sequences or more give every sequence one slot: no prefix and no suffix states exist, the
    walks start from a block of zeros and only the key shift of each sequence is computed beforehand (the workspace
    is filled with NaN bit patterns first: nothing that was not written may be read; every fifth batch entry against
    the oracle)."""
    import torch
    rng = np.random.default_rng(79 + L)
    B, H, d, M = 32, 8, 64, 256
    sc = np.linspace(0.6, 1.1, d)
    Q = synth.round_to_bf16((rng.standard_normal((B, H, L, d)) * sc + 0.05).astype(np.float32))
    K = synth.round_to_bf16((rng.standard_normal((B, H, L, d)) * sc[::-1] - 0.05).astype(np.float32))
    V = synth.round_to_bf16(rng.standard_normal((B, H, L, d)).astype(np.float32))
    dY = synth.round_to_bf16(rng.standard_normal((B, H, L, d)).astype(np.float32))
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    scale = d ** -0.25
    theta = _theta_block(variant, Q[::5], K[::5], scale)
    ws = torch.full((fs.attention_backward_workspace_bytes(B, H, L, L, d, d, M, True, H, H),), 0xFF, dtype=torch.uint8,
                    device="cuda")
    grads = fs.attention_backward(torch.from_numpy(theta).cuda(), util.to_device(Q, "bf16"), util.to_device(K, "bf16"),
                                  util.to_device(V, "bf16"), util.to_device(dY, "bf16"), scale, torch.from_numpy(Om).cuda(),
                                  causal=True, grad_dtype=torch.float32, workspace=ws)
    assert fs.attention_flushed_rows(ws) == 0
    gQ, gK, gV = (util.to_host(g) for g in grads)
    assert np.isfinite(gQ).all() and np.isfinite(gK).all() and np.isfinite(gV).all()
    worst = (0.0, 0.0)
    for b in range(0, B, 5):
        for h in range(H):
            th = util.oracle_theta_from_vec(theta[h], d)
            ref = orc.attention_backward(th, Om[h], Q[b, h], K[b, h], V[b, h], dY[b, h], scale, True)
            e = _assert_grads((gQ[b, h], gK[b, h], gV[b, h]), ref, 2e-2, (b, h))
            worst = (max(worst[0], e[0]), max(worst[1], e[1]))
    print(f"backward, causal, 256 sequences of {L} {variant}: worst frobenius {worst[0]:.2e}, worst row {worst[1]:.2e}")


@pytest.mark.parametrize("causal", [False, True])
def test_backward_bf16_path_single_token(fs, causal):
    """One query and one key: Y = V_0 whatever Q and K are, so dQ = dK = 0 and dV = dY.  On the bf16 kernels the zero
    is a cancellation of terms of size |dY| |V| that were rounded to bf16 on the way, so it is held to 2e-2 of that
    size; dV to the bf16 bar."""
    import torch
    rng = np.random.default_rng(76)
    d, M = 64, 256
    Q, K, V, dY = (synth.round_to_bf16(rng.standard_normal((1, 2, 1, d)).astype(np.float32)) for _ in range(4))
    Om = rng.standard_normal((2, M, d)).astype(np.float32)
    theta = np.stack([util.theta_vec_from_oracle(orc.fit_posrf(d))] * 2)
    gQ, gK, gV = fs.attention_backward(torch.from_numpy(theta).cuda(), util.to_device(Q, "bf16"), util.to_device(K, "bf16"),
                                       util.to_device(V, "bf16"), util.to_device(dY, "bf16"), d ** -0.25,
                                       torch.from_numpy(Om).cuda(), causal=causal, grad_dtype=torch.float32)
    torch.cuda.synchronize()
    gQ, gK, gV = util.to_host(gQ), util.to_host(gK), util.to_host(gV)
    for h in range(2):
        size = float(np.linalg.norm(dY[0, h]) * np.linalg.norm(V[0, h]))
        assert np.linalg.norm(gQ[0, h]) <= 2e-2 * size and np.linalg.norm(gK[0, h]) <= 2e-2 * size
        assert np.linalg.norm(gV[0, h] - dY[0, h]) <= 2e-2 * np.linalg.norm(dY[0, h])


@pytest.mark.parametrize("causal", [False, True])
def test_backward_bf16_path_strided_inputs_and_shared_parameters(fs, causal):
    """Q, K, V packed as [B, L, H, 3, d] and dY as [B, L, H, d] (row strides 3 H d and H d), one parameter set and
    one omega for all heads, two batches: strides, batch offsets and parameter groups on the bf16 kernels."""
    import torch
    w = synth.make("c4", B=2, H=2, L=448, seed=83)
    Q, K, V, s, d = w["Q"], w["K"], w["V"], w["qk_scale"], w["d"]
    Om = w["Omega"][:1]
    rng = np.random.default_rng(84)
    dY = synth.round_to_bf16(rng.standard_normal(V.shape).astype(np.float32))
    X = np.concatenate([s * Q[b, h] for b in range(2) for h in range(2)]).astype(np.float64)
    Yk = np.concatenate([s * K[b, h] for b in range(2) for h in range(2)]).astype(np.float64)
    vec = util.theta_vec_from_oracle(orc.fit_sderf(X, Yk))
    th = util.oracle_theta_from_vec(vec, d)
    qkv = torch.empty((2, 448, 2, 3, d), dtype=torch.bfloat16, device="cuda")
    for i, a in enumerate((Q, K, V)):
        qkv[:, :, :, i] = util.to_device(a, "bf16").permute(0, 2, 1, 3)
    Qd, Kd, Vd = (qkv[:, :, :, i].permute(0, 2, 1, 3) for i in range(3))
    dYd = util.to_device(dY, "bf16").permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    gQ, gK, gV = fs.attention_backward(torch.from_numpy(vec[None]).cuda(), Qd, Kd, Vd, dYd, s, torch.from_numpy(Om).cuda(),
                                       causal=causal, grad_dtype=torch.float32)
    torch.cuda.synchronize()
    gQ, gK, gV = util.to_host(gQ), util.to_host(gK), util.to_host(gV)
    for b in range(2):
        for h in range(2):
            rq, rk, rv = orc.attention_backward(th, Om[0], Q[b, h], K[b, h], V[b, h], dY[b, h], s, causal)
            _assert_grads((gQ[b, h], gK[b, h], gV[b, h]), (rq, rk, rv), 2e-2, (b, h))


@pytest.mark.parametrize("name", ["c3", "c4"])
def test_backward_bf16_path_is_bitwise_reproducible(fs, name):
    """No atomics, every LDS region ordered by workgroup barriers: repeated calls at the benchmark's full size must
    agree bit for bit; a race in a producer / consumer hand-over or between the walks of a call would show up here."""
    import torch
    w = synth.make(name)
    s, causal = w["qk_scale"], bool(w["causal"])
    Qd, Kd, Vd = (util.to_device(w[k], "bf16") for k in ("Q", "K", "V"))
    rng = np.random.default_rng(85)
    dYd = util.to_device(synth.round_to_bf16(rng.standard_normal(w["V"].shape).astype(np.float32)), "bf16")
    Om = torch.from_numpy(w["Omega"]).cuda()
    theta = fs.fit_params("sderf", Qd, Kd, s, groups=w["H"])
    first = [g.clone() for g in fs.attention_backward(theta, Qd, Kd, Vd, dYd, s, Om, causal=causal)]
    for rep in range(4):
        scratch = torch.randn(1 << 22, device="cuda").sum().item()      # unrelated work in between
        again = fs.attention_backward(theta, Qd, Kd, Vd, dYd, s, Om, causal=causal)
        torch.cuda.synchronize()
        for a, b in zip(first, again):
            assert torch.equal(a, b), (name, rep)
    assert all(torch.isfinite(g.float()).all().item() for g in first)


@pytest.mark.parametrize("name", ["c3", "c4"])
def test_backward_full_size_against_the_oracle_on_two_heads(fs, name):
    """The bf16 workloads at their full size, in the launch configuration the benchmark times (c4: 32 sequences of
    16384 tokens, eight slots of 32 chunks each); the oracle evaluates two whole (b, h) sequences (first and last)
    and every gradient row of them is compared."""
    import torch
    w = synth.make(name)
    B, H, L, d = w["B"], w["H"], w["L"], w["d"]
    s, causal = w["qk_scale"], bool(w["causal"])
    rng = np.random.default_rng(86)
    dY = synth.round_to_bf16(rng.standard_normal(w["V"].shape).astype(np.float32))
    Qd, Kd, Vd, dYd = (util.to_device(a, "bf16") for a in (w["Q"], w["K"], w["V"], dY))
    Om = torch.from_numpy(w["Omega"]).cuda()
    theta = fs.fit_params("sderf", Qd, Kd, s, groups=H)
    gQ, gK, gV = fs.attention_backward(theta, Qd, Kd, Vd, dYd, s, Om, causal=causal, grad_dtype=torch.float32)
    torch.cuda.synchronize()
    th_host = util.to_host(theta).astype(np.float32)
    for b, h in [(0, 0), (B - 1, H - 1)]:
        th = util.oracle_theta_from_vec(th_host[h], d)
        rq, rk, rv = orc.attention_backward(th, w["Omega"][h], w["Q"][b, h], w["K"][b, h], w["V"][b, h], dY[b, h], s, causal)
        fro, row = _assert_grads(tuple(util.to_host(g[b, h]) for g in (gQ, gK, gV)), (rq, rk, rv), 2e-2, (b, h))
        print(f"{name} backward full size (b={b}, h={h}): worst relative Frobenius error {fro:.2e}, worst row error {row:.2e}")


@pytest.mark.parametrize("causal", [False, True])
def test_forward_and_backward_bf16_path_one_parameter_set_per_sequence(fs, causal):
    """groups = omega_groups = B*H: every (b, h) sequence has its own fitted parameters and its own omega."""
    import torch
    w = synth.make("c4", B=2, H=2, L=320, seed=87)
    Q, K, V, s, d, M = w["Q"], w["K"], w["V"], w["qk_scale"], w["d"], w["M"]
    rng = np.random.default_rng(88)
    dY = synth.round_to_bf16(rng.standard_normal(V.shape).astype(np.float32))
    Om = rng.standard_normal((4, M, d)).astype(np.float32)
    ths = [orc.fit_sderf(s * Q[b, h].astype(np.float64), s * K[b, h].astype(np.float64)) for b in range(2) for h in range(2)]
    theta = torch.from_numpy(np.stack([util.theta_vec_from_oracle(t) for t in ths])).cuda()
    Qd, Kd, Vd, dYd = (util.to_device(a, "bf16") for a in (Q, K, V, dY))
    Y = util.to_host(fs.attention(theta, Qd, Kd, Vd, s, torch.from_numpy(Om).cuda(), causal=causal, out_dtype=torch.float32))
    gQ, gK, gV = (util.to_host(g) for g in fs.attention_backward(theta, Qd, Kd, Vd, dYd, s, torch.from_numpy(Om).cuda(),
                                                                  causal=causal, grad_dtype=torch.float32))
    for b in range(2):
        for h in range(2):
            g = 2 * b + h
            th = util.oracle_theta_from_vec(util.theta_vec_from_oracle(ths[g]), d)
            ref = orc.attention(th, Om[g], Q[b, h], K[b, h], V[b, h], s, causal)
            fro, row = util.attention_errors(Y[b, h], ref, V[b, h].astype(np.float64))
            assert fro <= 2e-2 and row <= 8e-2, (b, h, fro, row)
            rq, rk, rv = orc.attention_backward(th, Om[g], Q[b, h], K[b, h], V[b, h], dY[b, h], s, causal)
            _assert_grads((gQ[b, h], gK[b, h], gV[b, h]), (rq, rk, rv), 2e-2, (b, h))


@pytest.mark.parametrize("causal", [False, True])
def test_backward_gradient_tensors_with_huge_row_strides(fs, causal):
    """Gradient tensors whose row stride does not fit the 32-bit offsets of the bf16 kernels (2^23 elements and
    more): the call must take the general-shape kernels instead of wrapping offsets, and stay correct."""
    import torch
    w = synth.make("c4", B=1, H=1, L=40, seed=93)
    Q, K, V, s, d = w["Q"], w["K"], w["V"], w["qk_scale"], w["d"]
    rng = np.random.default_rng(94)
    dY = synth.round_to_bf16(rng.standard_normal(V.shape).astype(np.float32))
    vec = util.theta_vec_from_oracle(orc.fit_sderf(s * Q[0, 0].astype(np.float64), s * K[0, 0].astype(np.float64)))
    th = util.oracle_theta_from_vec(vec, d)
    big = 1 << 23
    wide = [torch.zeros((1, 1, 40, big), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    gK = wide[0][..., :d]
    dYd = wide[1][..., :d]
    dYd.copy_(util.to_device(dY, "bf16"))
    gQ = torch.empty((1, 1, 40, d), dtype=torch.bfloat16, device="cuda")
    gV = torch.empty((1, 1, 40, d), dtype=torch.bfloat16, device="cuda")
    fs.attention_backward(torch.from_numpy(vec[None]).cuda(), util.to_device(Q, "bf16"), util.to_device(K, "bf16"),
                          util.to_device(V, "bf16"), dYd, s, torch.from_numpy(w["Omega"]).cuda(), causal=causal,
                          grads=(gQ, gK, gV))
    torch.cuda.synchronize()
    ref = orc.attention_backward(th, w["Omega"][0], Q[0, 0], K[0, 0], V[0, 0], dY[0, 0], s, causal)
    _assert_grads(tuple(util.to_host(g[0, 0]) for g in (gQ, gK, gV)), ref, 2e-2, "huge strides")
    assert float(wide[0][..., d:d + 64].abs().max()) == 0.0          # nothing written beside the rows


@pytest.mark.parametrize("causal,L", [(False, 300), (True, 300), (False, 120)])
def test_backward_counts_rows_with_a_zero_normaliser_and_drops_their_terms(fs, causal, L):
    """Denominator guard in the backward pass (bf16 gradient kernels): a query row whose features all flush (40
    times the data's length: its Cauchy-Schwarz shift is more than 2^126 above every actual feature) has the
    normaliser 0, so its G1 row is 0: it gets a zero dQ row and adds nothing to dK and dV, which is what the oracle
    computes when that row of dY is zero.  The counter in the workspace's first word must report exactly these
    rows, and 0 again after a call without them (120 rows: the kernel that takes a whole sequence per workgroup)."""
    import torch
    w = synth.make("c4", B=1, H=2, L=L, seed=29)
    Q0, K, V, s, d, Om = w["Q"], w["K"], w["V"], w["qk_scale"], w["d"], w["Omega"]
    rows = [2, 64, min(200, L - 20), L - 1]
    Q = Q0.copy()
    Q[:, :, rows] *= 40.0
    Q = synth.round_to_bf16(Q)
    rng = np.random.default_rng(30)
    dY = synth.round_to_bf16(rng.standard_normal(V.shape).astype(np.float32))
    dY_seen = dY.copy()
    dY_seen[:, :, rows] = 0.0
    vec = util.theta_vec_from_oracle(orc.fit_posrf(d))
    th = util.oracle_theta_from_vec(vec, d)
    thd, Omd = torch.from_numpy(vec[None]).cuda(), torch.from_numpy(Om).cuda()
    nbytes = fs.attention_backward_workspace_bytes(1, 2, L, L, d, d, Om.shape[1], causal, 1, Om.shape[0])
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    Kd, Vd, dYd = (util.to_device(t, "bf16") for t in (K, V, dY))
    grads = fs.attention_backward(thd, util.to_device(Q, "bf16"), Kd, Vd, dYd, s, Omd, causal=causal, workspace=ws)
    assert fs.attention_flushed_rows(ws) == 2 * len(rows)
    gQ, gK, gV = (util.to_host(g) for g in grads)
    assert np.isfinite(gQ).all() and np.isfinite(gK).all() and np.isfinite(gV).all()
    assert (gQ[:, :, rows] == 0).all()
    for h in range(2):
        ref = orc.attention_backward(th, Om[h], Q[0, h], K[0, h], V[0, h], dY_seen[0, h], s, causal)
        _assert_grads((gQ[0, h], gK[0, h], gV[0, h]), ref, 2e-2, h)
    fs.attention_backward(thd, util.to_device(Q0, "bf16"), Kd, Vd, dYd, s, Omd, causal=causal, workspace=ws)
    assert fs.attention_flushed_rows(ws) == 0


@pytest.mark.parametrize("causal", [False, True])
def test_backward_bf16_kernels_take_an_fp32_output_gradient(fs, causal):
    """dY in fp32 next to bf16 Q, K, V (a caller that asked for an fp32 Y): the bf16 gradient kernels read it as it is
    (it stays fp32 until the G1 rows are rounded), so the result must agree with the oracle on the UNROUNDED dY to the
    bf16 bar, and must not be the result for the bf16-rounded dY bit for bit."""
    import torch
    w = synth.make("c4", B=1, H=2, L=333, seed=97)
    Q, K, V, s, d, Om = w["Q"], w["K"], w["V"], w["qk_scale"], w["d"], w["Omega"]
    rng = np.random.default_rng(98)
    dY = rng.standard_normal(V.shape).astype(np.float32)
    theta = _theta_block("sderf", Q, K, s)
    thd, Omd = torch.from_numpy(theta).cuda(), torch.from_numpy(Om).cuda()
    Qd, Kd, Vd = (util.to_device(t, "bf16") for t in (Q, K, V))
    got = fs.attention_backward(thd, Qd, Kd, Vd, util.to_device(dY, "f32"), s, Omd, causal=causal, grad_dtype=torch.float32)
    got = [util.to_host(g) for g in got]
    rounded = fs.attention_backward(thd, Qd, Kd, Vd, util.to_device(synth.round_to_bf16(dY), "bf16"), s, Omd, causal=causal,
                                    grad_dtype=torch.float32)
    assert any(not np.array_equal(a, util.to_host(b)) for a, b in zip(got, rounded))
    for h in range(2):
        th = util.oracle_theta_from_vec(theta[h], d)
        ref = orc.attention_backward(th, Om[h], Q[0, h], K[0, h], V[0, h], dY[0, h], s, causal)
        _assert_grads(tuple(g[0, h] for g in got), ref, 2e-2, h)


@pytest.mark.parametrize("name,over,variant", [("c3", dict(B=2, H=2, L=712), "sderf"), ("c4", dict(B=1, H=2, L=1216), "aderf"),
                                               ("c3", dict(B=2, H=2, L=128), "aderf"), ("c4", dict(B=32, H=8, L=100), "sderf"),
                                               ("c5", dict(B=1, H=2, L=96), "sderf")])
def test_backward_on_prepared_constants_gives_the_same_bits(fs, name, over, variant):
    """favorsharp_attention_backward_prepared against favorsharp_attention_backward: the projection constants are the
    same numbers, so the gradients agree bit for bit (separate kernels, the one-workgroup form, the causal form with
    and without slots; parameter sets with a dense C2 still compute their key row terms per call; the d = 128 shape
    runs on kernels that keep no constants and must simply ignore the buffer)."""
    import torch
    w = synth.make(name, **over)
    s, causal = w["qk_scale"], bool(w["causal"])
    Qd, Kd, Vd = (util.to_device(w[k], "bf16") for k in ("Q", "K", "V"))
    dY = torch.randn(Vd.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).to(torch.bfloat16)
    Om = torch.from_numpy(w["Omega"]).cuda()
    theta = fs.fit_params(variant, Qd, Kd, s, groups=w["H"])
    prepared = fs.attention_prepare(theta, Om, w["B"], w["H"], s)
    want = fs.attention_backward(theta, Qd, Kd, Vd, dY, s, Om, causal=causal)
    got = fs.attention_backward(theta, Qd, Kd, Vd, dY, s, Om, causal=causal, prepared=prepared)
    torch.cuda.synchronize()
    for a, b in zip(want, got):
        assert torch.isfinite(a.float()).all().item()
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (name, variant)


@pytest.mark.parametrize("name,over,prepared", [("c3", dict(B=2, H=2, L=712), False), ("c4", dict(B=1, H=2, L=1216), True),
                                                ("c3", dict(B=2, H=2, L=128), True), ("c4", dict(B=32, H=8, L=100), False),
                                                ("c1", {}, False)])
def test_backward_call_replays_from_a_hip_graph(fs, name, over, prepared):
    """The backward entry points only enqueue kernels on the caller's stream (no synchronisation, no allocation, no
    memset nodes): captured in a HIP graph and replayed three times, with eager work and synchronisations in between,
    every replay reproduces the eager gradients bit for bit (separate non-causal kernels, the causal kernels with
    slots, the one-workgroup form, the causal form with one slot per sequence, the general-shape kernels)."""
    import torch
    w = synth.make(name, **over)
    dt = w.get("dtype", "f32")
    Q, K, V = (util.to_device(w[k], dt) for k in "QKV")
    dY = torch.randn(V.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(7)).to(V.dtype)
    Om, s, causal = torch.from_numpy(w["Omega"]).cuda(), w["qk_scale"], bool(w["causal"])
    theta = fs.fit_params("aderf" if name == "c3" else "sderf", Q, K, s, groups=w["H"])
    B, H, L, d = Q.shape
    ws = torch.empty(fs.attention_backward_workspace_bytes(B, H, L, L, d, V.shape[-1], Om.shape[-2], causal, H, H),
                     dtype=torch.uint8, device="cuda")
    grads = tuple(torch.empty_like(t) for t in (Q, K, V))
    prep = fs.attention_prepare(theta, Om, B, H, s) if prepared else None

    def call():
        fs.attention_backward(theta, Q, K, V, dY, s, Om, causal=causal, workspace=ws, grads=grads, prepared=prep)

    call()
    torch.cuda.synchronize()
    ref = [g.clone() for g in grads]
    assert all(torch.isfinite(g.float()).all().item() for g in ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):           # warm-up on a side stream, as graph capture asks for
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for rep in range(3):
        for g in grads:
            g.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for g, r in zip(grads, ref):
            assert torch.equal(g, r), (name, rep)
        _ = torch.randn(1 << 20, device="cuda").sum().item()


@pytest.mark.parametrize("d,M,dtype", [(64, 256, "f32"), (128, 300, "bf16")])
def test_general_causal_calls_replay_on_other_values(fs, d, M, dtype):
    """Attention and gradients captured once and replayed on inputs of other sizes (the powers of two that values and dY are divided by
    are found by every replay): the bits of eager calls on the same inputs."""
    import torch
    L, s = 300, d ** -0.25
    gen = torch.Generator(device="cuda").manual_seed(d)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dY = ((f * torch.randn((1, 2, L, d), generator=gen, device="cuda")).to(dt) for f in (0.5, 0.5, 1.0, 1.0))
    Om = torch.randn((2, M, d), generator=gen, device="cuda")
    theta = fs.fit_params("saderf", Q, K, s, groups=2)
    ws = torch.empty(fs.attention_backward_workspace_bytes(1, 2, L, L, d, d, M, True, 2, 2), dtype=torch.uint8, device="cuda")
    Y, grads = torch.empty_like(V), tuple(torch.empty_like(x) for x in (Q, K, V))

    def call():
        fs.attention(theta, Q, K, V, s, Om, causal=True, workspace=ws, out=Y)
        fs.attention_backward(theta, Q, K, V, dY, s, Om, causal=True, workspace=ws, grads=grads)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for kv, kd in ((0, 0), (60, -50), (-100, 0), (0, 30)):
        V.copy_(V.float() * 2.0 ** kv)
        dY.copy_(dY.float() * 2.0 ** kd)
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in (Y, *grads)]
        call()
        torch.cuda.synchronize()
        assert all(torch.isfinite(x.float()).all().item() and torch.equal(x, y) for x, y in zip(got, (Y, *grads))), (kv, kd)
        V.copy_(V.float() * 2.0 ** -kv)
        dY.copy_(dY.float() * 2.0 ** -kd)


def test_backward_error_paths(fs):
    import torch
    Q = torch.zeros((1, 1, 8, 8), device="cuda")
    K = torch.zeros((1, 1, 12, 8), device="cuda")
    th = torch.from_numpy(util.theta_vec_from_oracle(orc.fit_posrf(8))[None]).cuda()
    Om = torch.zeros((1, 4, 8), device="cuda")
    with pytest.raises(fs.FavorSharpError) as err:          # causal needs as many queries as keys
        fs.attention_backward(th, Q, K, K, Q, 1.0, Om, causal=True)
    assert err.value.status in (2, 4)       # unsupported (the workspace query already says so with 0 bytes)


@pytest.mark.parametrize("variant", ["sderf", "saderf"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("L,d,dv,M", [
    (1, 8, 8, 1),              # one row, one feature: everything but element 0 of each tile is padding
    (33, 32, 16, 32),          # one row past a tile; exactly one block of features (the second of a pair is absent)
    (65, 40, 128, 33),         # one feature past a block; the widest values (a state of 144 columns)
    (96, 128, 96, 100),        # the widest rows; values whose normaliser column opens a new tile of 16; three of four blocks full
])
def test_backward_causal_general_path_at_tile_edges(fs, L, d, dv, M, dtype, variant):
    rng = np.random.default_rng(7 * L + d)
    B, H = 1, 2
    Q, K = ((0.6 * rng.standard_normal((B, H, L, d))).astype(np.float32) for _ in range(2))
    V, dY = (rng.standard_normal((B, H, L, dv)).astype(np.float32) for _ in range(2))
    Om = rng.standard_normal((H, M, d)).astype(np.float32)
    if dtype == "bf16":
        Q, K, V, dY = (synth.round_to_bf16(x) for x in (Q, K, V, dY))
    # parameters are fitted to more rows than the call has, so that their statistics have full rank
    fit_rows = np.concatenate([Q, (0.6 * rng.standard_normal((B, H, 4 * d, d))).astype(np.float32)], axis=2)
    import torch
    scale = d ** -0.25
    theta = _theta_block(variant, fit_rows, fit_rows[:, :, ::-1], scale)
    grads = fs.attention_backward(torch.from_numpy(theta).cuda(), *(util.to_device(x, dtype) for x in (Q, K, V, dY)), scale,
                                  torch.from_numpy(Om).cuda(), causal=True, grad_dtype=torch.float32)
    grads = [util.to_host(g) for g in grads]
    for h in range(H):
        th = util.oracle_theta_from_vec(theta[h], d)
        ref = orc.attention_backward(th, Om[h], Q[0, h], K[0, h], V[0, h], dY[0, h], scale, True)
        # the bar of this file (3e-4); gradients that are zero by construction (one row) against the scale of dY
        _assert_grads([g[0, h] for g in grads], ref, 3e-4, (h, L, d, dv, M), 1e-3 * float(np.linalg.norm(dY[0, h])))
