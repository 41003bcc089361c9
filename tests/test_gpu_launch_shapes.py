"""The kernels on both sides of the sizes and alignments at which their launch
shape changes: against the oracle, or bit for bit against the same call in the
shape that the oracle tests cover."""

import numpy as np
import pytest

import oracle
from tests import _harness as H

pytestmark = pytest.mark.gpu


def _cuda(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _loss_inputs(rng, lens):
    T = int(np.sum(lens))
    off = np.r_[0, np.cumsum(lens)].astype(np.int32)
    logp = (-rng.random(T) * 5.0).astype(np.float32)
    lp_old = (logp + rng.uniform(-0.4, 0.4, T)).astype(np.float32)
    lp_roll = (lp_old + rng.uniform(-3.0, 3.0, T)).astype(np.float32)
    lp_ref = (logp + rng.uniform(-0.5, 0.5, T)).astype(np.float32)
    adv = rng.choice([-1.0, 1.0, 0.5], T).astype(np.float32)
    mask = (rng.random(len(lens)) < 0.6).astype(np.uint8)
    mask[0] = 1
    return logp, lp_old, lp_roll, lp_ref, adv, off, mask


@pytest.mark.parametrize("kl,ratio", [("none", "step_geomean"), ("k3", "step_product")])
@pytest.mark.parametrize("S,length", [
    (1, 3),        # one wave with a step
    (32, 40),      # the last size on one workgroup
    (33, 40),      # the first on several, the second workgroup's waves mostly idle
    (48, 257),     # a lane's second batch of tokens holds one token
    (20, 47), (20, 50),  # one workgroup: a lane's tokens one by one, in batches
    (70, 47), (70, 50),  # several
    (3000, 1),     # as many workgroups as 3000 tokens have room for
    (20000, 1),    # fewer workgroups than the steps ask for (the workspace's room)
    (700, 256),
])
def test_step_ratio_launch_shapes(S, length, kl, ratio):
    """Coefficients bit for bit those of the one-workgroup launch, the loss the
    same fp64 sum in another order, and both the oracle's."""
    import paper_2509_23866_amd as dart

    rng = np.random.default_rng(S * 1000 + length)
    lens = np.full(S, length) if length == 1 else rng.integers(max(1, length - 2), length + 1, S)
    lens[-1] = length
    logp, lp_old, lp_roll, lp_ref, adv, off, mask = _loss_inputs(rng, lens)
    eps_low, eps_high, C = H.f32(0.2), H.f32(0.28), H.f32(2.0)
    ref = oracle.tis_loss_ex(logp.astype(np.float64), lp_old, lp_roll, adv, off, mask, eps_low,
                             eps_high, C, lp_ref=lp_ref, kl=kl, beta=0.05, agg="step_mean",
                             ratio=ratio)
    args = [_cuda(a) for a in (logp, lp_old, lp_roll, adv, off, mask)]
    got = {}
    for ws in ("auto", None):
        got[ws] = dart.dart_tis_loss_fwd_ex(*args, eps_low, eps_high, C, logp_ref=_cuda(lp_ref),
                                            kl=kl, beta=0.05, aggregation="step_mean",
                                            ratio=ratio, workspace=ws)
    (la, ca, sa), (lb, cb, sb) = got["auto"], got[None]
    assert np.array_equal(ca.cpu().numpy().view(np.uint32), cb.cpu().numpy().view(np.uint32))
    assert abs(la.item() - lb.item()) <= 1e-12 * max(abs(lb.item()), 1e-300)
    assert np.allclose(sa.cpu().numpy(), sb.cpu().numpy(), rtol=1e-6, atol=0)
    ok = ~ref["boundary"]
    g = ca.cpu().numpy().astype(np.float64)
    floor = 1e-6 * np.abs(ref["g"]).max()
    assert np.all((np.abs(g - ref["g"]) <= 1e-4 * np.abs(ref["g"]) + floor)[ok])
    if ok.all():
        assert abs(la.item() - ref["L"]) <= H.LOSS_RTOL * max(abs(ref["L"]), 1e-30)


@pytest.mark.parametrize("G,T", [(1, 2048), (2, 9000), (3, 40000), (1, 70000)])
def test_grpo_advantage_several_workgroups_a_group(G, T):
    """1, 2, 6 and 16 workgroups a group; trajectories shorter than a run of 64
    tokens among them."""
    import paper_2509_23866_amd as dart

    rng = np.random.default_rng(T)
    n_traj = 7 * G
    cut = lambda n, k: np.r_[0, np.sort(rng.choice(np.arange(1, n), k - 1, False)), n].astype(np.int32)  # noqa: E731
    S = 5 * n_traj
    off, traj = cut(T, S), cut(S, n_traj)
    grp = (np.arange(G + 1) * 7).astype(np.int32)
    reward = rng.random(n_traj).astype(np.float32)
    A, mean, std = oracle.grpo_advantage(reward, traj, grp, off)[:3]
    adv = _cuda(np.full(T, np.nan, np.float32))
    adv, gm, gs = dart.dart_grpo_advantage(_cuda(reward), _cuda(traj), _cuda(grp), _cuda(off), T=T,
                                           adv=adv)
    # one rounding to fp32 of a value formed in fp64 on both sides
    assert np.all(np.abs(adv.cpu().numpy() - A) <= 2.0 ** -23 * np.abs(A))
    assert np.allclose(gm.cpu().numpy(), mean, rtol=2.0 ** -23, atol=0)
    assert np.allclose(gs.cpu().numpy(), std, rtol=2.0 ** -23, atol=0)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,pad", [(1, 2), (7, 1), (50, 3), (2049, 0), (4099, 9)])
def test_gradient_rows_aligned_unlike_the_logits(dtype, V, pad):
    """Every alignment of the logits against every alignment of the gradient
    gives the bits of the call on 16-byte aligned rows, reads nothing outside
    the rows (NaN there) and writes nothing outside them."""
    import torch

    import paper_2509_23866_amd as dart

    T = 9
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    per = 8 if dtype == "bf16" else 4
    g = torch.Generator(device="cuda").manual_seed(V)
    z = (torch.randn(T, V, generator=g, device="cuda") * 3).to(dt)
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    wide = -(-V // per) * per

    def rows(offset, ld, fill):
        buf = torch.full((offset + T * ld + per,), fill, dtype=dt, device="cuda")
        return buf, buf[offset:offset + T * ld].view(T, ld)[:, :V]

    _, za = rows(0, wide, float("nan"))
    za.copy_(z)
    logp, ent, lse = dart.dart_tok_stats(za, y)
    coef = torch.randn(T, generator=g, device="cuda") * 0.1
    coef[3] = 0.0
    _, want = rows(0, wide, 7.0)
    for skip in (False, True):
        dart.dart_tis_grad(za, y, logp, lse, coef, dlogits=want, skip_zero_rows=skip)
        for a in range(per):
            for b in range(per):
                _, zi = rows(a, V + pad, float("nan"))
                zi.copy_(z)
                buf, out = rows(b, V + (pad + a) % 3, 7.0)
                dart.dart_tis_grad(zi, y, logp, lse, coef, dlogits=out, skip_zero_rows=skip)
                assert torch.equal(out, want), (a, b, skip)
                out.fill_(7.0)
                assert bool((buf == 7.0).all()), (a, b, skip)


SKIP, BF16 = 1, 4


@pytest.mark.parametrize("flags", [0, BF16, SKIP, SKIP | BF16])
@pytest.mark.parametrize("T,d,V,rows,cols,parts", [
    (40, 72, 4095, 40, 4095, 1),     # one column short of two parts
    (40, 72, 4096, 40, 4096, 2),
    (300, 136, 9001, 300, 9001, 4),  # the last part ends inside a slice
    (300, 136, 9001, 300, 8300, 4),  # the second block has fewer slices than parts
    (300, 136, 9001, 100, 9001, 4),  # several row blocks on one set of parts
])
def test_lmhead_backward_dh_in_parts(T, d, V, rows, cols, parts, flags):
    """dhidden summed in parts: against the oracle and the exact product of the
    GPU's own bf16 dlogits, within the bounds of the one-run sum (which a smaller
    workspace takes); bf16 gradients are the fp32 ones rounded; garbage in the
    workspace does not matter."""
    import torch

    import paper_2509_23866_amd as dart
    from tests import test_gpu_lmhead_grad as G

    h, w, y, g = G._problem(T, d, V)
    rlogp, _, rlse = oracle.lmhead_token_stats(h, w, y)
    dz64, dh64, dw64 = oracle.lmhead_grads(h, w, y, rlse, rlogp, g)
    h64, w64 = oracle.bf16_bits_to_f64(h), oracle.bf16_bits_to_f64(w)
    hd, wd, yd, gd = G._dev_bf16(h), G._dev_bf16(w), _cuda(y), _cuda(g)
    logp, _, lse = dart.dart_lmhead_tok_stats(hd, wd, yd)
    dzo = G._own_dz(hd, wd, yd, lse, logp, gd)
    need = dart.dart_lmhead_backward_ex_workspace_bytes(T, d, V, rows, cols, flags)
    full = dart.dart_lmhead_backward_split_workspace_bytes(T, d, V, rows, cols, flags)
    up = -(-need // 256) * 256
    assert full == (need if parts == 1 else up + parts * min(rows, T) * d * 4)

    def run(nbytes, f):
        ws = torch.full((nbytes,), 0x7F, dtype=torch.uint8, device="cuda")
        return dart.dart_lmhead_backward_ex(hd, wd, yd, lse, logp, gd, chunk_rows=rows,
                                            chunk_cols=cols, flags=f, workspace=ws)

    bf = bool(flags & BF16)
    for nbytes in (full, full - 1) if parts > 1 else (full,):
        dh, dw = run(nbytes, flags)
        G._check_grad(dh, dh64, dzo @ w64, np.abs(dz64) @ np.abs(w64), "dhidden", bf16=bf)
        G._check_grad(dw, dw64, dzo.T @ h64, np.abs(dz64).T @ np.abs(h64), "dweight", bf16=bf)
        if flags & SKIP:
            assert bool((dh[torch.from_numpy(g == 0.0).cuda()] == 0).all())
    auto = dart.dart_lmhead_backward_ex(hd, wd, yd, lse, logp, gd, chunk_rows=rows,
                                        chunk_cols=cols, flags=flags)
    a, b = run(full, flags)
    assert torch.equal(auto[0], a) and torch.equal(auto[1], b)
    if bf:
        wide = dart.dart_lmhead_backward_split_workspace_bytes(T, d, V, rows, cols, flags & SKIP)
        assert torch.equal(a, run(wide, flags & SKIP)[0].to(torch.bfloat16))


@pytest.mark.parametrize("T,d,V", [
    (64, 64, 1000),       # one 64-row tile, one K slice
    (65, 128, 257),       # two 64-row tiles, two slices, one column past a tile
    (200, 200, 33000),    # 128-row tiles: 130 a row of tiles
    (256, 320, 40001),    # 128-row tiles, five slices
    (500, 72, 60000),     # 256-row tiles
    (600, 72, 60000),     # 256-row tiles and a last 128-row one
    (640, 136, 60000),    # the last one full
])
def test_lmhead_tile_rows(T, d, V):
    """Every tile height: the statistics against the oracle, and dlogits bit for
    bit those of calls on 64 rows at a time (the K sums run in the same order)."""
    import torch

    import paper_2509_23866_amd as dart
    from tests import test_gpu_lmhead_grad as G

    h, w, y, g = G._problem(T, d, V)
    rlogp, rH, rlse = oracle.lmhead_token_stats(h, w, y)
    hd, wd, yd, gd = G._dev_bf16(h), G._dev_bf16(w), _cuda(y), _cuda(g)
    logp, ent, lse = dart.dart_lmhead_tok_stats(hd, wd, yd)
    for got, ref in ((logp, rlogp), (ent, rH), (lse, rlse)):
        assert np.abs(got.cpu().numpy() - ref).max() <= 2e-4
    ld = (V + 7) // 8 * 8
    out = torch.full((T, ld), 5.0, dtype=torch.bfloat16, device="cuda")
    dart.dart_lmhead_dlogits(hd, wd, yd, lse, logp, gd, dlogits=out[:, :V])
    assert bool((out[:, V:] == 5.0).all())
    for a in range(0, T, 64):
        b = min(T, a + 64)
        part = torch.empty((b - a, ld), dtype=torch.bfloat16, device="cuda")
        dart.dart_lmhead_dlogits(hd[a:b], wd, yd[a:b], lse[a:b], logp[a:b], gd[a:b],
                                 dlogits=part[:, :V])
        assert torch.equal(out[a:b, :V], part[:, :V]), (a, b)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,vecs,extra", [
    (5, 512, 0), (5, 512, 3),        # 128 threads: one full iteration, no tail and a tail
    (5, 513, 0),                     # 256 threads, an iteration of 513 of 1024 vectors
    (5, 2048, 7), (256, 2049, 0),    # 256 and 768 threads
    (257, 2049, 1), (257, 8192, 0),  # 512 threads
    (257, 8193, 5), (600, 8193, 0),  # 768 threads
    (7, 1, 0), (7, 0, 3),            # one vector a row, none
])
def test_token_statistics_by_row_length(T, vecs, extra, dtype):
    """Every workgroup size of the statistics pass at both ends of its range of
    rows, at a 16-byte aligned and a misaligned row start, with the target in
    the row's head, first and last vector, last full iteration and tail."""
    import torch

    import paper_2509_23866_amd as dart

    per = 8 if dtype == "bf16" else 4
    V = vecs * per + extra % per
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(V + T)
    for shift in (0, 1):
        ld = -(-V // per) * per + (per if shift else 0)
        buf = torch.full((T * ld + 2 * per,), float("nan"), dtype=dt, device="cuda")
        z = buf[shift:shift + T * ld].view(T, ld)[:, :V]
        z.copy_((torch.randn(T, V, generator=g, device="cuda") * 3).to(dt))
        y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
        for i, col in enumerate((0, V - 1, V // 2, max(0, (vecs - 1) * per), V - extra % per - 1)):
            y[i % T] = min(V - 1, max(0, col))
        z[torch.arange(T, device="cuda"), y.long()] += 4
        z[0, : V // 3] = float("-inf")
        if V // 3 and int(y[0]) < V // 3:
            y[0] = V - 1
        zh = z.contiguous().cpu()
        host = zh.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else zh.numpy()
        logp, H_, lse = oracle.token_stats(host, y.cpu().numpy())
        got = dart.dart_tok_stats(z, y)
        for name, a, b in zip(("logp", "entropy", "lse"), got, (logp, H_, lse)):
            err = np.abs(a.cpu().numpy() - b).max()
            # a few fp32 roundings of values up to ~20
            assert err <= 1.5e-5, (name, shift, err)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,shift", [(1, 0), (9, 1), (2049, 3), (20000, 0)])
def test_gradient_of_rows_with_a_zero_coefficient(V, shift, dtype):
    """Rows whose coefficient is zero are written unread: the bits of
    -g exp(z - lse), a zero of -g's sign (the target: of g's), with the logits
    replaced by NaN; where lse is not finite, what the formula gives (NaN from
    NaN or -inf), and plain zeros under the skip flag."""
    import torch

    import paper_2509_23866_amd as dart

    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    per = 8 if dtype == "bf16" else 4
    T, ld = 12, V + per + shift
    g = torch.Generator(device="cuda").manual_seed(V)
    base = torch.zeros(shift + T * ld, dtype=dt, device="cuda")
    z = base[shift:].view(T, ld)[:, :V]
    z.copy_((torch.randn(T, V, generator=g, device="cuda") * 3).to(dt))
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    logp, _, lse = dart.dart_tok_stats(z, y)
    coef = torch.randn(T, generator=g, device="cuda") * 0.1
    full = dart.dart_tis_grad(z, y, logp, lse, coef)
    coef[[1, 4]], coef[[2, 7]] = 0.0, -0.0
    zero = [1, 2, 4, 7]
    z[zero] = float("nan")  # never read
    bits = torch.int16 if dtype == "bf16" else torch.int32
    for it in (1.0, 0.5):
        dz = dart.dart_tis_grad(z, y, logp, lse, coef, inv_temp=it)
        want = torch.zeros(T, V, device="cuda")
        want[[1, 4]] = -0.0
        want[[2, 7], y[[2, 7]].long()] = -0.0
        want[[1, 4], y[[1, 4]].long()] = 0.0
        # a target with all the mass (V = 1): g (-expm1(0)) turns the sign
        sure = [t for t in zero if float(logp[t]) == 0.0]
        want[sure, y[sure].long()] *= -1.0
        assert torch.equal(dz[zero].view(bits), want[zero].to(dt).view(bits))
        rest = [t for t in range(T) if t not in zero]
        if it == 1.0:
            assert torch.equal(dz[rest], full[rest])
    bad = lse.clone()
    bad[1], bad[2], bad[4] = float("nan"), float("-inf"), float("inf")
    z[zero] = 1.0
    dz = dart.dart_tis_grad(z, y, logp, bad, coef)
    keep = torch.ones(T, V, dtype=torch.bool, device="cuda")
    keep[torch.arange(T, device="cuda"), y.long()] = False
    assert bool(dz[1][keep[1]].isnan().all()) and bool(dz[2][keep[2]].isnan().all())
    assert bool((dz[4] == 0).all()) and bool((dz[7] == 0).all())
    skipped = dart.dart_tis_grad(z, y, logp, bad, coef, skip_zero_rows=True)
    assert bool((skipped[zero].view(bits) == 0).all())


@pytest.mark.parametrize("flags", [0, BF16])
@pytest.mark.parametrize("rows,cols,kept", [(700, 143000, "some"), (700, 100000, "some"),
                                            (512, 143000, "some"), (700, 143000, "none"),
                                            (700, 143000, "nan")])
def test_lmhead_backward_leaves_zero_rows_out(rows, cols, kept, flags):
    """A large call without the skip flag leaves rows with a zero coefficient out
    where its workspace has the room: against the exact products of the GPU's own
    bf16 dlogits (64-bit, by torch), and against the call on a smaller workspace,
    which forms every row; a zero row with a NaN in it still gives its NaNs."""
    import torch

    import paper_2509_23866_amd as dart

    T, d, V = 700, 1024, 143000
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    h = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn(V, d, generator=g, device="cuda") * 3 / d ** 0.5).to(torch.bfloat16)
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    coef = torch.randn(T, generator=g, device="cuda") * 1e-2
    zero = torch.rand(T, generator=g, device="cuda") < 0.2
    zero[100:260] = True
    if kept == "none":
        zero[:] = True
    coef[zero] = 0.0
    if kept == "nan":
        h[150, 7] = float("nan")
    logp, _, lse = dart.dart_lmhead_tok_stats(h, w, y)
    need = dart.dart_lmhead_backward_ex_workspace_bytes(T, d, V, rows, cols, flags)
    full = dart.dart_lmhead_backward_split_workspace_bytes(T, d, V, rows, cols, flags)
    assert full >= need + T * (6 * d + 20)

    def run(nbytes):
        ws = torch.full((nbytes,), 0x7F, dtype=torch.uint8, device="cuda")
        return dart.dart_lmhead_backward_ex(h, w, y, lse, logp, coef, chunk_rows=rows,
                                            chunk_cols=cols, flags=flags, workspace=ws)

    (dh, dw), (dh0, dw0) = run(full), run(need)
    if kept == "nan":
        for a, b in ((dh, dh0), (dw, dw0)):
            assert torch.equal(a.isnan(), b.isnan()) and bool(a.isnan().any())
        return
    assert bool((dh[zero] == 0).all())
    buf = torch.empty((T, V), dtype=torch.bfloat16, device="cuda")
    dz = dart.dart_lmhead_dlogits(h, w, y, lse, logp, coef, dlogits=buf).double()
    h64, w64 = h.double(), w.double()
    A, U = 2.0 ** -13, 2.0 ** -8  # fp32 sums over |terms|; the bf16 output's rounding
    for got, dense, ref, bound in ((dh, dh0, dz @ w64, dz.abs() @ w64.abs()),
                                   (dw, dw0, dz.t() @ h64, dz.abs().t() @ h64.abs())):
        tol = A * bound + (U * ref.abs() if flags & BF16 else 0)
        assert bool(((got.double() - ref).abs() <= tol + 1e-30).all())
        assert bool(((dense.double() - ref).abs() <= tol + 1e-30).all())


@pytest.mark.parametrize("S", [1, 16, 17, 48, 49, 64, 65, 80, 81, 128, 256, 257])
@pytest.mark.parametrize("rho", [0.3, 0.8])
def test_selection_by_number_of_steps(S, rho):
    """Step means and mask exactly the oracle's, ties between whole steps
    included, on both sides of the one-launch, four-way-rank and direct-rank
    limits; and the selection and loss in one call bit for bit the two calls'."""
    import torch

    import paper_2509_23866_amd as dart

    rng = np.random.default_rng(S)
    lens = rng.choice([1, 2, 7, 40], S)
    T = int(lens.sum())
    ent = rng.choice([0.0, 0.5, 1.25, 3.0], T).astype(np.float32)
    off = np.r_[0, np.cumsum(lens)].astype(np.int32)
    Hs, Hs32 = oracle.step_entropy(ent.astype(np.float64), off)
    mask, k = oracle.step_mask(Hs32, rho)
    sh, m, nk = dart.dart_step_select(_cuda(ent), _cuda(off), rho)
    assert np.array_equal(sh.cpu().numpy().view(np.uint32) & 0x7FFFFFFF,
                          Hs32.view(np.uint32) & 0x7FFFFFFF)
    assert np.array_equal(m.cpu().numpy(), mask) and int(nk.item()) == k
    logp, lp_old, lp_roll, _, adv, _, _ = _loss_inputs(rng, lens)
    x = [_cuda(a) for a in (logp, lp_old, lp_roll, adv, off)]
    got = dart.dart_select_tis_loss_fwd(_cuda(ent), *x, rho, 0.2, 0.28, 2.0)
    loss, coef, stats = dart.dart_tis_loss_fwd(*x, m, 0.2, 0.28, 2.0)
    assert torch.equal(got[0], sh) and torch.equal(got[1], m) and torch.equal(got[2], nk)
    assert torch.equal(got[4].view(torch.int32), coef.view(torch.int32))
    assert abs(got[3].item() - loss.item()) <= 1e-12 * max(abs(loss.item()), 1e-300)
    assert torch.allclose(got[5], stats, rtol=1e-6, atol=0)


@pytest.mark.parametrize("V", [2048, 8000, 32003])
def test_lse_close_to_its_rounding(V):
    """lse lies in [8, 16) here, where float32 values are u = 2^-20 apart: its own
    rounding is uniform, u / sqrt(12) = 2.75e-7 in the root mean square. What the
    sums and the row's finish add is held to 2e-7, in quadrature 3.4e-7 in all
    (a finish by one log2f of the whole sum reaches 3.5e-7 to 4.3e-7)."""
    import torch

    import paper_2509_23866_amd as dart

    rng = np.random.default_rng(V)
    T = 4096
    z = _cuda((2.0 * rng.standard_normal((T, V), dtype=np.float32)))
    y = _cuda(rng.integers(0, V, T).astype(np.int32))
    lse = dart.dart_tok_stats(z, y)[2].double()
    ref = torch.cat([torch.logsumexp(z[a:a + 512].double(), 1) for a in range(0, T, 512)])
    assert 8 < float(ref.min()) and float(ref.max()) < 16
    assert float((lse - ref).square().mean().sqrt()) < 3.4e-7


def _same_bits(a, b):
    import torch

    return all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(a, b))


@pytest.mark.parametrize("V", [60000, 59963])  # a last tile of 96 columns and of 59
@pytest.mark.parametrize("inv_temp", [1.0, 1.3])
def test_lmhead_statistics_of_equal_rows(V, inv_temp):
    """Equal rows have the same bits wherever they stand, in the 256-row tiles or
    the last short one of a call, and in calls of every tile height: 64 different
    rows, repeated."""
    import torch

    import paper_2509_23866_amd as dart

    d, n = 72, 64
    g = torch.Generator(device="cuda").manual_seed(V)
    h = torch.randn(n, d, generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn(V, d, generator=g, device="cuda") * 3 / d ** 0.5).to(torch.bfloat16)
    y = torch.randint(V, (n,), generator=g, device="cuda", dtype=torch.int32)
    y[:4] = torch.tensor([0, 63, 64, V - 1], dtype=torch.int32)
    want = None
    # 64- and 128-row tiles; 256-row ones; with a last tile of 88 rows; with a full one
    for T in (64, 128, 500, 600, 640):
        i = torch.arange(T, device="cuda") % n
        got = dart.dart_lmhead_tok_stats_ex(h[i], w, y[i], inv_temp)
        want = want or [x.clone() for x in got]
        assert _same_bits(got, [x[i] for x in want]), T


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("vecs", [512, 2048, 2049, 8000, 8193])
def test_token_statistics_do_not_depend_on_the_number_of_rows(vecs, dtype):
    """A row has the same bits in a call of one row, of some hundred, and of more
    logits than are loaded cacheably (64 MB)."""
    import torch

    import paper_2509_23866_amd as dart

    per = 8 if dtype == "bf16" else 4
    V, dt = vecs * per + 1, torch.bfloat16 if dtype == "bf16" else torch.float32
    T = (64 << 20) // (vecs * 16) + 300
    g = torch.Generator(device="cuda").manual_seed(vecs)
    z = (torch.randn(T, V + per - 1, generator=g, device="cuda") * 3).to(dt)[:, :V]
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    want = [x[:300] for x in dart.dart_tok_stats(z, y)]
    for n in (1, 100, 256, 257, 300):
        assert _same_bits(dart.dart_tok_stats(z[:n], y[:n]), [x[:n] for x in want]), n


@pytest.mark.parametrize("flags,cols", [(SKIP, 40), (SKIP, 24), (SKIP | BF16, 40),
                                        (SKIP | BF16, 24)])
def test_lmhead_backward_puts_back_more_rows_than_one_sweep(flags, cols):
    """Skipped rows: the kept rows' dhidden, put back by the GEMM or from its fp32 sums
    (more than the 65,536 workgroups of one sweep put back), bit for bit those of the
    dense call (the sums over short vocabulary blocks run in the same order)."""
    import torch

    import paper_2509_23866_amd as dart

    T, d, V = 9000, 8192, 40
    g = torch.Generator(device="cuda").manual_seed(3)
    h = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn(V, d, generator=g, device="cuda") * 3 / d ** 0.5).to(torch.bfloat16)
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    coef = torch.randn(T, generator=g, device="cuda") * 1e-2
    coef[torch.rand(T, generator=g, device="cuda") < 0.05] = 0.0
    logp, _, lse = dart.dart_lmhead_tok_stats(h, w, y)
    run = lambda f: dart.dart_lmhead_backward_ex(h, w, y, lse, logp, coef, chunk_rows=T,  # noqa: E731
                                                 chunk_cols=cols, flags=f)[0]
    got, dense = run(flags), run(flags & BF16)
    kept = coef != 0
    assert int(kept.sum()) * d > 65536 * 1024
    assert torch.equal(got[kept], dense[kept]) and bool((got[~kept] == 0).all())


@pytest.mark.parametrize("call", ["step ratios", "selection"])
def test_workspace_that_stays_untouched(call):
    """Step ratios, and the loss of a small fused selection, leave a workspace of
    dart_tis_loss_workspace_bytes alone, and of one of the split size as much;
    with either, the same coefficients bit for bit and the same loss."""
    import torch

    import paper_2509_23866_amd as dart

    rng = np.random.default_rng(5)
    lens = rng.integers(20, 31, 120)  # 120 steps, more than 2048 and less than 4096 tokens
    logp, lp_old, lp_roll, lp_ref, adv, off, mask = _loss_inputs(rng, lens)
    T = int(lens.sum())
    assert 2048 < T <= 4096
    ent = _cuda(rng.random(T).astype(np.float32))
    x = [_cuda(a) for a in (logp, lp_old, lp_roll, adv, off)]
    small, full = dart.dart_tis_loss_workspace_bytes(T), dart.dart_tis_loss_split_workspace_bytes(T)
    got = []
    for nbytes, alone in ((small, small), (full, small)):
        ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        if call == "selection":
            out = dart.dart_select_tis_loss_fwd(ent, *x, 0.6, 0.2, 0.28, 2.0, workspace=ws)[3:5]
        else:
            out = dart.dart_tis_loss_fwd_ex(*x, _cuda(mask), 0.2, 0.28, 2.0, logp_ref=_cuda(lp_ref),
                                            kl="k3", beta=0.05, ratio="step_geomean",
                                            workspace=ws)[:2]
        assert bool((ws[:alone] == 0xA5).all())
        assert nbytes == small or bool((ws[alone:] != 0xA5).any())
        got.append(out)
    (la, ca), (lb, cb) = got
    assert torch.equal(ca.view(torch.int32), cb.view(torch.int32))
    assert abs(la.item() - lb.item()) <= 1e-12 * abs(lb.item())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_a_nan_or_infinite_logit_of_a_dropped_row(dtype, value):
    """What the header says of logits that the statistics do not take: in a row that
    counts they give a NaN in the gradient, in a row with a zero coefficient zeros
    where lse is finite; other rows do not change."""
    import torch

    import paper_2509_23866_amd as dart

    T, V = 6, 20011
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(1)
    z = (torch.randn(T, V, generator=g, device="cuda") * 3).to(dt)
    y = torch.full((T,), 5, dtype=torch.int32, device="cuda")
    coef = torch.full((T,), 0.1, device="cuda")
    coef[[1, 3]] = 0.0
    logp, _, lse = dart.dart_tok_stats(z, y)
    clean = dart.dart_tis_grad(z, y, logp, lse, coef)
    z[[1, 2], 9000] = value
    got = dart.dart_tok_stats(z, y)
    dz = dart.dart_tis_grad(z, y, got[0], got[2], coef)
    assert bool(dz[2].isnan().any()) or bool(dz[2].isinf().any())
    assert not bool(got[2][1].isfinite()) or bool((dz[1] == 0).all())
    for rows in ([0], [3], [4], [5]):
        assert torch.equal(dz[rows], clean[rows])


@pytest.mark.parametrize("flags", [None, 0, BF16])
def test_lmhead_backward_where_memory_is_short(flags, monkeypatch):
    """With no room for the larger workspace the call runs in the one that every call
    needs, and gives the bits of a call that is handed that one."""
    import torch

    import paper_2509_23866_amd as dart

    T, d, V = 300, 136, 9001
    g = torch.Generator(device="cuda").manual_seed(2)
    h = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn(V, d, generator=g, device="cuda") * 3 / d ** 0.5).to(torch.bfloat16)
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    coef = torch.randn(T, generator=g, device="cuda") * 1e-2
    logp, _, lse = dart.dart_lmhead_tok_stats(h, w, y)
    least = dart.dart_lmhead_backward_ex_workspace_bytes(T, d, V, T, V, flags or 0)
    assert least < dart.dart_lmhead_backward_split_workspace_bytes(T, d, V, T, V, flags or 0)

    def run(**kw):
        if flags is None:
            return dart.dart_lmhead_backward(h, w, y, lse, logp, coef, chunk_rows=T, **kw)
        return dart.dart_lmhead_backward_ex(h, w, y, lse, logp, coef, chunk_rows=T, chunk_cols=V,
                                            flags=flags, **kw)

    want = run(workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    empty = torch.empty

    def short(*size, **kw):
        if kw.get("dtype") == torch.uint8 and size[0] > least:
            raise torch.OutOfMemoryError("no room")
        return empty(*size, **kw)

    monkeypatch.setattr(torch, "empty", short)
    got = run()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("T,d,V", [(64, 72, 300), (300, 136, 700), (257, 8, 513)])
def test_lmhead_operands_that_end_their_buffers(T, d, V):
    """Hidden states and weight as the last columns of wider matrices, d no multiple
    of a K slice: the last row ends the buffer, and nothing past it is read. The bits
    of the call on contiguous copies."""
    import torch

    import paper_2509_23866_amd as dart

    g = torch.Generator(device="cuda").manual_seed(d)
    wide = lambda n: torch.randn(n, d + 8, generator=g, device="cuda").to(torch.bfloat16)[:, 8:]  # noqa: E731
    h, w = wide(T), wide(V)
    y = torch.randint(V, (T,), generator=g, device="cuda", dtype=torch.int32)
    coef = torch.randn(T, generator=g, device="cuda") * 1e-2
    a, b = [dart.dart_lmhead_tok_stats(*x, y) for x in ((h, w), (h.contiguous(), w.contiguous()))]
    assert _same_bits(a, b)
    ld = (V + 7) // 8 * 8
    out = [torch.empty((T, ld), dtype=torch.bfloat16, device="cuda")[:, :V] for _ in range(2)]
    dart.dart_lmhead_dlogits(h, w, y, a[2], a[0], coef, dlogits=out[0])
    dart.dart_lmhead_dlogits(h.contiguous(), w.contiguous(), y, a[2], a[0], coef, dlogits=out[1])
    assert torch.equal(out[0], out[1])
