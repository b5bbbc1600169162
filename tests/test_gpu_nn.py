"""The learned warm start on the GPU: MFMA convolution kernels against the
float64 CPU reference, whole-network outputs and gradients against the CPU
reference's autograd, the Adam update against its formula, and a small
training run showing what the trained network gains as an initial guess."""
import numpy as np
import pytest
import torch

from oracle import unet_ref as U
from paper_1305_2418_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _mg():
    from paper_1305_2418_amd import mgfr
    return mgfr


def _ref_conv(x_bf, w_bf, bias=None, relu=False):
    """float64 reference on the bf16 inputs: x [B,S,S,S,Cin], w [27,Cout,Cin]."""
    x = x_bf.float().double().cpu().permute(0, 4, 1, 2, 3)
    w = w_bf.float().double().cpu()
    co, ci = w.shape[1], w.shape[2]
    wt = w.permute(1, 2, 0).reshape(co, ci, 3, 3, 3)
    y = U.conv3d_periodic(x, wt, None if bias is None else bias.double().cpu())
    if relu:
        y = torch.relu(y)
    return y.permute(0, 2, 3, 4, 1)


@pytest.mark.parametrize("B,S,Cin,Cout", [(2, 8, 8, 16), (1, 16, 16, 32), (2, 8, 48, 16), (1, 8, 96, 32), (1, 16, 64, 64)])
def test_conv_forward_matches_reference(B, S, Cin, Cout):
    mg = _mg()
    print(f"[case] conv fwd B={B} S={S} Cin={Cin} Cout={Cout}", flush=True)
    g = torch.Generator().manual_seed(Cin * 100 + Cout)
    x = torch.randn((B, S, S, S, Cin), generator=g).to(torch.bfloat16).to(DEV)
    w = (torch.randn((27, Cout, Cin), generator=g) / np.sqrt(27 * Cin)).to(torch.bfloat16).to(DEV)
    b = torch.randn((Cout,), generator=g).float().to(DEV)
    y32 = mg.conv3d_fwd(x, w, b, relu=True, out32=True).double().cpu()
    ref = _ref_conv(x, w, b, relu=True)
    # float32 accumulation of bf16 products: error ~ 1e-6 relative to the scale of the sums
    assert torch.abs(y32 - ref).max() <= 1e-4 * max(1.0, ref.abs().max().item())
    ybf = mg.conv3d_fwd(x, w, b, relu=True).float().double().cpu()
    assert torch.all(torch.abs(ybf - ref) <= 2 ** -7 * ref.abs() + 1e-4)


@pytest.mark.parametrize("B,S,Cin,Cout", [(2, 8, 16, 16), (1, 16, 48, 16), (1, 8, 96, 32), (1, 8, 32, 64)])
def test_conv_backward_data_and_weight_match_reference(B, S, Cin, Cout):
    mg = _mg()
    print(f"[case] conv bwd B={B} S={S} Cin={Cin} Cout={Cout}", flush=True)
    g = torch.Generator().manual_seed(7 * Cin + Cout)
    x = torch.randn((B, S, S, S, Cin), generator=g).to(torch.bfloat16)
    w = (torch.randn((27, Cout, Cin), generator=g) / np.sqrt(27 * Cin)).to(torch.bfloat16)
    dz = torch.randn((B, S, S, S, Cout), generator=g).to(torch.bfloat16)
    # reference gradients of sum(dz * conv(x, w)) in float64
    xr = x.double().permute(0, 4, 1, 2, 3).requires_grad_(True)
    wr = w.double().permute(1, 2, 0).reshape(Cout, Cin, 3, 3, 3).detach().requires_grad_(True)
    y = U.conv3d_periodic(xr, wr)
    (y * dz.double().permute(0, 4, 1, 2, 3)).sum().backward()
    dx_ref = xr.grad.permute(0, 2, 3, 4, 1)
    dw_ref = wr.grad.reshape(Cout, Cin, 27).permute(2, 0, 1)
    db_ref = dz.double().sum(dim=(0, 1, 2, 3))
    dx = mg.conv3d_bwd_data(dz.to(DEV), w.to(DEV)).float().double().cpu()
    assert torch.all(torch.abs(dx - dx_ref) <= 2 ** -7 * dx_ref.abs() + 1e-3 * dx_ref.abs().max())
    dw, db = mg.conv3d_bwd_weight(x.to(DEV), dz.to(DEV))
    dw, db = dw.double().cpu(), db.double().cpu()
    assert torch.abs(dw - dw_ref).max() <= 1e-4 * dw_ref.abs().max()
    assert torch.abs(db - db_ref).max() <= 1e-4 * db_ref.abs().max()


@pytest.mark.parametrize("B,S,Cin,Cout,relu", [
    (1, 16, 16, 16, True), (3, 16, 80, 16, False), (1, 32, 48, 16, True), (4, 32, 16, 16, False), (1, 64, 48, 16, True),
    (2, 64, 16, 16, True), (5, 32, 16, 16, False), (1, 16, 16, 32, False), (2, 32, 48, 96, True), (1, 16, 16, 48, True),
    (1, 16, 32, 16, True), (3, 32, 64, 48, False), (1, 16, 32, 64, True), (1, 32, 64, 64, False), (2, 32, 96, 32, True)])
def test_conv_exact_on_integers(B, S, Cin, Cout, relu):
    """Convolutions on small integers, whose float32 sums are exact (|x| <= 3,
    |w| <= 2: 27 * 96 * 6 + 8 < 2^24): every depth of the tiles, fewer and more
    of them than workgroups, chunks of 16 and of 32 input channels, one and
    several, one and several blocks of output channels; and a non-finite voxel
    reaches its 27 neighbours and no other."""
    mg = _mg()
    print(f"[case] conv B={B} S={S} Cin={Cin} Cout={Cout} relu={relu}", flush=True)
    g = torch.Generator().manual_seed(B * 1000 + S + Cin)
    x = torch.randint(-3, 4, (B, S, S, S, Cin), generator=g).to(torch.bfloat16)
    w = torch.randint(-2, 3, (27, Cout, Cin), generator=g).to(torch.bfloat16)
    b = torch.randint(-8, 9, (Cout,), generator=g).float()
    y = mg.conv3d_fwd(x.to(DEV), w.to(DEV), b.to(DEV), relu=relu, out32=True).cpu()
    # the reference in float32, exact on these integers as well
    xt, wt = x.float().permute(0, 4, 1, 2, 3), w.float().permute(1, 2, 0).reshape(Cout, Cin, 3, 3, 3)
    ref = U.conv3d_periodic(xt, wt, b)
    ref = (torch.relu(ref) if relu else ref).permute(0, 2, 3, 4, 1)
    assert torch.equal(y, ref)
    z = (B - 1, S - 1, 0, S // 2)
    x[z + (Cin - 1,)] = float("inf")
    y = mg.conv3d_fwd(x.to(DEV), w.to(DEV), None, relu=False, out32=True).cpu()
    near = torch.zeros((B, S, S, S), dtype=torch.bool)
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                near[z[0], (z[1] + dz) % S, (z[2] + dy) % S, (z[3] + dx) % S] = True
    assert torch.equal(~torch.isfinite(y).all(-1), near)


@pytest.mark.parametrize("S,Cin,Cout", [(16, 16, 16), (16, 32, 32)])
def test_conv_into_an_output_off_the_store_width(S, Cin, Cout):
    """Outputs one element past an aligned address: the same bits as aligned ones."""
    mg = _mg()
    print(f"[case] conv into an offset output S={S} Cin={Cin} Cout={Cout}", flush=True)
    g = torch.Generator().manual_seed(S + Cin)
    x = torch.randn((1, S, S, S, Cin), generator=g).to(torch.bfloat16).to(DEV)
    w = (torch.randn((27, Cout, Cin), generator=g) / np.sqrt(27 * Cin)).to(torch.bfloat16).to(DEV)
    n = S ** 3 * Cout
    y, y32 = torch.zeros(n + 1, dtype=torch.bfloat16, device=DEV), torch.zeros(n + 1, device=DEV)
    rc = mg.lib().mgfr_conv3d_fwd(x.data_ptr(), 1, S, Cin, w.data_ptr(), None, Cout, 0, y.data_ptr() + 2,
                                  y32.data_ptr() + 4, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    assert torch.equal(y[1:].view(1, S, S, S, Cout), mg.conv3d_fwd(x, w)) and float(y[0]) == 0.0
    assert torch.equal(y32[1:].view(1, S, S, S, Cout), mg.conv3d_fwd(x, w, out32=True)) and float(y32[0]) == 0.0


@pytest.mark.parametrize("B,S,Cin,Cout,with_db", [(1, 8, 16, 16, True), (3, 8, 16, 96, True), (1, 8, 96, 16, False),
                                                  (1, 16, 64, 64, True), (2, 32, 48, 16, True), (1, 32, 16, 32, True)])
def test_conv_backward_weight_exact_on_integers(B, S, Cin, Cout, with_db):
    """Weight and bias gradients on small integers: every product and every
    float32 partial sum is an integer below 2^24, so any order of the sums is
    exact (|x|, |dz| <= 3: 9 B S^3 < 2^20).  Sides with tiles of 8 and of 16
    voxels, one tile and several per workgroup, one and many channel blocks."""
    mg = _mg()
    print(f"[case] conv wgrad B={B} S={S} Cin={Cin} Cout={Cout}", flush=True)
    g = torch.Generator().manual_seed(S * 1000 + Cin + Cout)
    x = torch.randint(-3, 4, (B, S, S, S, Cin), generator=g)
    dz = torch.randint(-3, 4, (B, S, S, S, Cout), generator=g)
    ref = torch.empty((27, Cout, Cin), dtype=torch.float64)
    zf = dz.reshape(-1, Cout).double().t().contiguous()
    for t in range(27):
        sh = (1 - t // 9, 1 - (t // 3) % 3, 1 - t % 3)
        ref[t] = zf @ torch.roll(x, sh, (1, 2, 3)).reshape(-1, Cin).double()
    xb, zb = x.to(torch.bfloat16).to(DEV), dz.to(torch.bfloat16).to(DEV)
    if with_db:
        dw, db = mg.conv3d_bwd_weight(xb, zb)
        assert torch.equal(db.double().cpu(), zf.sum(1))
    else:  # no bias gradient asked for
        dw = torch.zeros((27, Cout, Cin), dtype=torch.float32, device=DEV)
        assert mg.lib().mgfr_conv3d_bwd_weight(xb.data_ptr(), zb.data_ptr(), B, S, Cin, Cout, dw.data_ptr(), None,
                                               mg._stream_ptr()) == 0
    assert torch.equal(dw.double().cpu(), ref)


def _pairs(n, S=32, seed0=100, device=DEV):
    """(delta, u) training pairs generated by the solver itself on S^3 meshes."""
    mg = _mg()
    rng = np.random.default_rng(seed0)
    deltas, us, conds = [], [], []
    for i in range(n):
        a = float(rng.uniform(0.5, 1.0))
        fr0 = float(10 ** rng.uniform(-7, -4))
        pos = synth.clustered_load(S, 100.0, rms=5.0, seed=seed0 + i, n_halos=4).to(device)
        s = mg.Solver(mg.Params(mesh=S, a=a, fr0_abs=fr0, max_vcycles=80))
        d = s.assign_density(pos)
        u, _, st = s.solve(d, want_dfr=False)
        deltas.append(d)
        us.append(u)
        conds.append((a, fr0))
    return torch.stack(deltas), torch.stack(us), conds


def test_network_output_and_gradients_match_cpu_reference():
    mg = _mg()
    net = mg.Net(seed=3, max_voxels=32 ** 3)
    delta, u, cond = _pairs(1, 32, seed0=200)
    p = net.get_params()
    x = U.features(delta.cpu(), cond)
    y_ref = U.forward(torch.tensor(p, dtype=torch.float64), x)
    y = net.predict(delta, cond).cpu() / U.U_SCALE
    rel = (torch.linalg.norm(y - y_ref) / torch.linalg.norm(y_ref)).item()
    print(f"  forward rel L2 diff {rel:.3e}")
    assert rel < 0.02  # bf16 weights and activations
    L_ref, g_ref = U.loss_and_grad(torch.tensor(p, dtype=torch.float64), x, u.cpu())
    L, g = net.grads(delta, u, cond)
    assert abs(L / L_ref - 1) < 0.02
    g = torch.tensor(g, dtype=torch.float64)
    # layer by layer: direction and size of the gradient
    off = 0
    for ci, co in U.LAYERS:
        sl = slice(off, off + 27 * ci * co)
        off += 27 * ci * co + co
        a, b = g[sl], g_ref[sl]
        cos = torch.dot(a, b) / (torch.linalg.norm(a) * torch.linalg.norm(b))
        rn = torch.linalg.norm(a - b) / torch.linalg.norm(b)
        print(f"  layer {ci}->{co}: cos {cos:.5f} rel {rn:.3e}")
        assert cos > 0.995 and rn < 0.1


def _bf16_either(v):
    """The two bf16 values a float64 -> float32 -> bf16 rounding of v can give
    when v itself is known to within 2^-40 relative (both sides round to
    nearest even; the interval is far narrower than one float32 ulp)."""
    lo = (v * (1 - 2.0 ** -40)).float().bfloat16().double()
    hi = (v * (1 + 2.0 ** -40)).float().bfloat16().double()
    return torch.minimum(lo, hi), torch.maximum(lo, hi)


def _gamma(k):
    """Bound on the relative error of any order of k float32 additions."""
    e = k * 2.0 ** -24
    return e / (1 - e)


BF16_U = 2.0 ** -8  # unit roundoff of bf16 (8 significant bits, round to nearest)


def _check_rounded(y, z, acc_err, what):
    """y (library, bf16 or float32) against the exact value z: an accumulation
    error of at most acc_err, then (for bf16) one rounding to nearest."""
    bound = BF16_U * (z.abs() + acc_err) + acc_err + 1e-30
    worst = ((y - z).abs() / bound).max().item()
    print(f"  {what}: worst |y - z| / bound {worst:.3f}")
    assert worst <= 1.0, what


@pytest.mark.parametrize("weights", ["init", "trained"])
def test_network_forward_element_by_element(weights):
    """Each tensor of the forward pass from the library's own input to that
    stage (exported with mgfr_net_activation), against float64 arithmetic on
    the same bf16 inputs and bf16-rounded weights:
    features: one of the two roundings of the float64 value (bitwise up to
    ties); convolution + bias + ReLU: K = 27 Cin + 1 float32 additions, then a
    bf16 rounding; 2^3 mean: 8 additions, then bf16; upsampling + skip
    concatenation: bitwise; head: 17 float32 additions; output u = 5 y in
    float32."""
    import os
    mg = _mg()
    S = 32
    net = mg.Net(seed=3, max_voxels=S ** 3)
    if weights == "trained":
        path = os.path.join(os.path.dirname(mg.__file__), "weights", "unet_warmstart.npy")
        net.set_params(np.load(path))
    delta, _, cond = _pairs(1, S, seed0=210)
    u = net.predict(delta, cond).cpu()
    y32 = net.activation(15).cpu()
    A = [net.activation(i).cpu().double() for i in range(16)]
    p = torch.tensor(net.get_params(), dtype=torch.float32)
    convs, hw, hb = U.unpack(p)
    # features
    x = A[0]
    lo, hi = _bf16_either(torch.asinh(delta.cpu()[0].double()) * 0.25)
    assert torch.all((x[0, ..., 0] == lo) | (x[0, ..., 0] == hi))
    a, fr0 = cond[0]
    for c, v in ((1, (a - 0.75) * 4.0), (2, (np.log10(fr0) + 5.5) / 1.5)):
        lo, hi = _bf16_either(torch.tensor(v, dtype=torch.float64))
        assert torch.all((x[0, ..., c] == lo) | (x[0, ..., c] == hi))
    assert torch.all(x[0, ..., 3:] == 0)

    def conv_check(out_i, in_i, layer):
        wt, b = convs[layer]
        w = wt.bfloat16().double()
        xin = A[in_i].permute(0, 4, 1, 2, 3)
        z = torch.relu(U.conv3d_periodic(xin, w, b.double()))
        E = U.conv3d_periodic(xin.abs(), w.abs(), b.double().abs())
        k = 27 * w.shape[1] + 1
        _check_rounded(A[out_i].permute(0, 4, 1, 2, 3), z, _gamma(k) * E, f"conv {layer} ({in_i} -> {out_i})")

    def pool_check(out_i, in_i):
        xin = A[in_i].permute(0, 4, 1, 2, 3)
        z = torch.nn.functional.avg_pool3d(xin, 2)
        E = torch.nn.functional.avg_pool3d(xin.abs(), 2)
        _check_rounded(A[out_i].permute(0, 4, 1, 2, 3), z, _gamma(8) * E, f"pool ({in_i} -> {out_i})")

    def cat_check(out_i, up_i, skip_i):
        up = A[up_i].repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)
        assert torch.equal(A[out_i], torch.cat([up, A[skip_i]], dim=4)), f"concat {out_i}"

    conv_check(1, 0, 0)
    conv_check(2, 1, 1)
    pool_check(3, 2)
    conv_check(4, 3, 2)
    conv_check(5, 4, 3)
    pool_check(6, 5)
    conv_check(7, 6, 4)
    conv_check(8, 7, 5)
    cat_check(9, 8, 5)
    conv_check(10, 9, 6)
    conv_check(11, 10, 7)
    cat_check(12, 11, 2)
    conv_check(13, 12, 8)
    conv_check(14, 13, 9)
    h = A[14][0]
    z = (h * hw.double()).sum(-1) + float(hb)
    E = (h.abs() * hw.double().abs()).sum(-1) + abs(float(hb))
    err = (A[15][0] - z).abs() - _gamma(17) * E
    assert err.max().item() <= 1e-30, "head"
    assert torch.equal(u, (y32 * np.float32(U.U_SCALE)).double())  # one float32 product


def test_adam_step_matches_formula():
    mg = _mg()
    net = mg.Net(seed=4, max_voxels=32 ** 3)
    delta, u, cond = _pairs(1, 32, seed0=300)
    p0 = net.get_params().astype(np.float64)
    _, g = net.grads(delta, u, cond)
    lr = 1e-3
    net.train_step(delta, u, cond, lr)
    p1 = net.get_params().astype(np.float64)
    expect = p0 - lr * g / (np.abs(g) + 1e-8)
    big = np.abs(g) > 1e-6  # where the sign of g is unambiguous
    assert np.abs(p1 - expect)[big].max() < 1e-6
    assert np.abs(p1 - p0).max() <= lr * 1.0001


def test_training_reduces_loss_and_improves_the_initial_guess():
    mg = _mg()
    torch.manual_seed(0)
    delta, u, cond = _pairs(32, 32, seed0=1000)
    net = mg.Net(seed=5, max_voxels=8 * 32 ** 3)
    losses = []
    for it in range(240):
        idx = torch.randint(0, 32, (8,))
        L = net.train_step(delta[idx].contiguous(), u[idx].contiguous(), [cond[i] for i in idx.tolist()],
                           2e-3 if it < 160 else 5e-4)
        losses.append(L)
    first, last = np.mean(losses[:10]), np.mean(losses[-10:])
    print(f"  loss {first:.4f} -> {last:.4f}")
    assert last < 0.5 * first
    # warm start of a held-out 128^3 solve from the prediction on the 32^3 (N/4) mesh
    N = 128
    pos = synth.clustered_load(N, 100.0, rms=5.0, seed=4242, n_halos=20).to(DEV)
    s = mg.Solver(mg.Params(mesh=N, a=0.8, fr0_abs=1e-6, max_vcycles=80))
    d = s.assign_density(pos)
    u_star, _, st_cold = s.solve(d, want_dfr=False)
    s0 = mg.Solver(mg.Params(mesh=N, a=0.8, fr0_abs=1e-6, max_vcycles=0, nn_mode=mg.NN_COARSE))
    s0.set_net(net)
    u0, _, _ = s0.solve(d, want_dfr=False, allow_not_converged=True)
    err_nn = (torch.linalg.norm(u0 - u_star) / torch.linalg.norm(u_star)).item()
    s1 = mg.Solver(mg.Params(mesh=N, a=0.8, fr0_abs=1e-6, max_vcycles=80, nn_mode=mg.NN_COARSE))
    s1.set_net(net)
    u1, _, st_nn = s1.solve(d, want_dfr=False)
    print(f"  initial-guess rel L2 error {err_nn:.3f} (zero guess: 1.000); V-cycles cold {st_cold.vcycles}, "
          f"warm {st_nn.vcycles}; res0 cold {st_cold.res0:.2e} warm {st_nn.res0:.2e}")
    assert err_nn < 0.5
    assert st_nn.status == 0 and st_nn.res <= 1e-8
    assert torch.abs(u1 - u_star).max().item() < 1e-5 * max(1.0, u_star.abs().max().item())


@pytest.mark.parametrize("a", [0.5, 1.0])
def test_shipped_network_on_a_held_out_input(a):
    """What the shipped network gains, on a held-out load of its training
    recipe (256^3 particles and mesh in 50 Mpc/h, seed 20000, the cell of the
    512^3 workload), |f_R0| = 1e-6, the benchmark's schedule.  Reports V-cycles
    from u = 0, the screened-limit guess, the network (prediction on the N/4
    mesh, prolonged) and the best any N/4 prediction could do (the converged u
    itself, restricted to N/4 and interpolated back).  Asserts that the network
    solve reaches the cold solve's answer in no more cycles, and that even the
    ideal N/4 guess saves at most one cycle over the screened-limit guess: the
    cycle count is set by cell-scale structure that no N/4 prediction holds,
    which is why the network does not pay for itself against that guess."""
    import os
    import torch.nn.functional as F
    mg = _mg()
    from paper_1305_2418_amd import train_net as T
    print(f"[case] shipped network, held-out 256^3 load, a={a}", flush=True)
    net = mg.Net(seed=0, max_voxels=64 ** 3)
    net.set_params(np.load(os.path.join(os.path.dirname(mg.__file__), "weights", "unet_warmstart.npy")))
    pos = synth.clustered_load(256, T.BOX, rms=5.0, seed=20000, n_halos=3, device=DEV)
    s = T._solver(256, T.BOX, a, 1e-6)
    d = s.assign_density(pos)
    u_cold, _, st_cold = s.solve(d, want_dfr=False)
    u_star, _, _ = T._solver(256, T.BOX, a, 1e-6, tol=1e-11).solve(d, u=u_cold.clone(), want_dfr=False)
    _, _, st_scr = s.solve(d, u=s.screened_guess(d), want_dfr=False)
    ideal = T._prolong_trilinear(F.avg_pool3d(u_star[None, None], 4)[0, 0], 4)
    _, _, st_ideal = s.solve(d, u=ideal, want_dfr=False)
    snn = mg.Solver(mg.Params(mesh=256, box=T.BOX, a=a, fr0_abs=1e-6, tol=1e-8, precision=mg.MIXED,
                              max_vcycles=200, pre_smooth=4, post_smooth=4, coarse_sweeps=30, prolong=1,
                              nn_mode=mg.NN_COARSE))
    snn.set_relaxation32(1.2)
    snn.set_net(net)
    u_nn, _, st_nn = snn.solve(d, want_dfr=False)
    print(f"  V-cycles: cold {st_cold.vcycles}, screened {st_scr.vcycles}, network {st_nn.vcycles}, "
          f"ideal N/4 {st_ideal.vcycles}; res0 cold {st_cold.res0:.2e} screened {st_scr.res0:.2e} "
          f"network {st_nn.res0:.2e} ideal {st_ideal.res0:.2e}")
    assert st_nn.status == 0 and st_nn.res <= 1e-8
    dfr = lambda u: torch.expm1(u)
    assert (dfr(u_nn) - dfr(u_star)).abs().max().item() <= 1e-6 * dfr(u_star).abs().max().item()
    assert st_nn.vcycles <= st_cold.vcycles
    assert st_ideal.vcycles >= st_scr.vcycles - 1


def test_coarse_cycle_warm_start_reaches_the_same_solution():
    """The network's N/4 prediction corrected by V-cycles on the N/4 and N/2
    problems (coarse_cycles) starts the solve at N; the solve still iterates to
    the tolerance and returns the cold solve's answer."""
    mg = _mg()
    net = mg.Net(seed=6, max_voxels=32 ** 3)
    net.set_params(np.zeros(net.num_params, dtype=np.float32))  # prediction u = 0: isolates the coarse cycles
    N = 128
    pos = synth.clustered_load(N, 100.0, rms=5.0, seed=4343, n_halos=20).to(DEV)
    s = mg.Solver(mg.Params(mesh=N, a=0.8, fr0_abs=1e-6, max_vcycles=80))
    d = s.assign_density(pos)
    u_star, _, st_cold = s.solve(d, want_dfr=False)
    res0 = []
    for cc in (0, 2):
        s1 = mg.Solver(mg.Params(mesh=N, a=0.8, fr0_abs=1e-6, max_vcycles=80, nn_mode=mg.NN_COARSE,
                                 coarse_cycles=cc, precision=mg.MIXED))
        s1.set_net(net)
        u1, _, st = s1.solve(d, want_dfr=False)
        print(f"  coarse_cycles={cc}: res0 {st.res0:.2e}, cycles {st.vcycles} (cold {st_cold.vcycles})")
        assert st.status == 0 and st.res <= 1e-8
        assert torch.abs(u1 - u_star).max().item() < 1e-5 * max(1.0, u_star.abs().max().item())
        res0.append(st.res0)
    assert res0[1] < res0[0]  # the coarse correction lowers the initial residual



def test_checkpoint_round_trip(tmp_path):
    """save() then load() into a fresh network restores the parameters and the
    Adam state: the next training step moves both alike (the weight gradients
    sum over chunks with atomics, so the two steps agree to float32 rounding of
    the gradient, not bit for bit), and unlike a network given the same
    parameters with fresh moments; a file of another layout is rejected and
    leaves the network unchanged."""
    mg = _mg()
    delta, u, cond = _pairs(2, 32, seed0=400)
    a = mg.Net(seed=8, max_voxels=2 * 32 ** 3)
    for _ in range(3):
        a.train_step(delta, u, cond, 1e-3)
    path = str(tmp_path / "net.ckpt")
    a.save(path)
    b = mg.Net(seed=9, max_voxels=2 * 32 ** 3)
    b.load(path)
    assert np.array_equal(a.get_params(), b.get_params())
    c = mg.Net(seed=10, max_voxels=2 * 32 ** 3)
    c.set_params(a.get_params())  # same parameters, Adam state reset
    p0 = a.get_params().astype(np.float64)
    for n in (a, b, c):
        n.train_step(delta, u, cond, 1e-3)
    da, db, dc = (n.get_params().astype(np.float64) - p0 for n in (a, b, c))
    assert np.abs(da - db).max() <= 1e-3 * np.abs(da).max()  # same moments and bias-correction step
    assert np.abs(da - dc).max() >= 0.1 * np.abs(da).max()  # fresh moments would step differently
    bad = tmp_path / "bad.ckpt"
    bad.write_bytes(b"MGFRNET1" + b"\0" * 64)
    before = b.get_params()
    with pytest.raises(mg.MgfrError):
        b.load(str(bad))
    assert np.array_equal(before, b.get_params())


def test_context_network_calls(tmp_path):
    """The context-level calls on the context's own network (mgfr_nn_init,
    _predict, _train_step, _save, _load): nn_predict is exactly the initial
    guess a solve with nn_mode = MGFR_NN_COARSE starts from; a training step
    runs; a checkpoint saved through one context and loaded into another gives
    the same guess; without a network the calls fail with MGFR_ERR_ARG."""
    mg = _mg()
    N = 128
    print("[case] context network calls", flush=True)
    pos = synth.clustered_load(N, 100.0, rms=5.0, seed=4444, n_halos=20).to(DEV)
    prm = dict(mesh=N, a=0.8, fr0_abs=1e-6, max_vcycles=0, nn_mode=mg.NN_COARSE)
    s = mg.Solver(mg.Params(**prm))
    s.nn_init(seed=11)
    d = s.assign_density(pos)
    g = s.nn_predict(d)
    u0, _, _ = s.solve(d, want_dfr=False, allow_not_converged=True)
    assert torch.equal(g, u0)
    delta, u, cond = _pairs(2, 32, seed0=500)
    loss = s.nn_train_step(delta, u, cond, 1e-3)
    assert np.isfinite(loss) and loss > 0
    path = str(tmp_path / "ctx.ckpt")
    s.nn_save(path)
    s2 = mg.Solver(mg.Params(**prm))
    s2.nn_init(seed=99)
    assert not torch.equal(s2.nn_predict(d), s.nn_predict(d))
    s2.nn_load(path)
    assert torch.equal(s2.nn_predict(d), s.nn_predict(d))
    s3 = mg.Solver(mg.Params(mesh=N))
    with pytest.raises(mg.MgfrError):
        s3.nn_predict(d)


def _taps(x):
    """The 27 shifts of x [B,S,S,S,C] that the convolution's taps read: x[v + off_t]."""
    for t in range(27):
        yield torch.roll(x, (1 - t // 9, 1 - (t // 3) % 3, 1 - t % 3), (1, 2, 3)).reshape(-1, x.shape[-1])


def _up(x):
    return x.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)


def _net_on_volumes(B, S):
    """A network with non-zero biases on B volumes of side S: its bf16-rounded layers
    (w [27, Cout, Cin], b) and head, activations, target and gradient, on the GPU."""
    mg = _mg()
    net = mg.Net(seed=B + S, max_voxels=B * S ** 3)
    p = net.get_params()
    rng = np.random.default_rng(S)
    off, layers = 0, []
    for ci, co in U.LAYERS:
        sl = slice(off, off + 27 * ci * co)
        off = sl.stop + co
        p[sl.stop:off] = rng.normal(0.0, 0.1, co)
        layers.append((sl, slice(sl.stop, off), ci, co))
    net.set_params(p)
    g = torch.Generator(device=DEV).manual_seed(S)
    delta = torch.exp(torch.randn((B, S, S, S), generator=g, dtype=torch.float64, device=DEV)) - 1.0
    u = -2.0 * torch.log1p(0.1 * (delta + 1.0)) + 0.1
    cond = [(0.5 + 0.05 * b, 10.0 ** (-7 + 0.2 * b)) for b in range(B)]
    net.predict(delta, cond)
    A = [net.activation(i) for i in range(16)]
    _, grad = net.grads(delta, u, cond)  # the same forward pass again
    p = torch.tensor(p, device=DEV)
    W = [(p[w].bfloat16().double().reshape(27, co, ci), p[b].double(), w, b) for w, b, ci, co in layers]
    return W, p[off:off + 16].double(), A, u, torch.tensor(grad, dtype=torch.float64, device=DEV)


# (layer, input activations (the second of a pair is the skip connection), output activation)
_CONV_IO = [(0, (0,), 1), (1, (1,), 2), (2, (3,), 4), (3, (4,), 5), (4, (6,), 7), (5, (7,), 8), (6, (8, 5), 10),
            (7, (10,), 11), (8, (11, 2), 13), (9, (13,), 14)]


def _input_of(A, io):
    return A[io[0]].double() if len(io) == 1 else torch.cat([_up(A[io[0]]), A[io[1]]], dim=4).double()


@pytest.mark.parametrize("B,S", [(5, 32), (2, 64)])
def test_network_convolutions_element_by_element_in_batches(B, S):
    """Every convolution of the forward pass from the library's own input to it, over
    several volumes and in the tile depths that larger meshes take (the decoder's
    two-source layers too), against float64 on the same bf16 values: K = 27 Cin + 1
    float32 additions, then one bf16 rounding."""
    print(f"[case] network convolutions B={B} S={S}", flush=True)
    W, _, A, _, _ = _net_on_volumes(B, S)
    for l, io, out in _CONV_IO:
        w, b = W[l][:2]
        x = _input_of(A, io)
        z = torch.zeros((x.numel() // x.shape[-1], w.shape[1]), dtype=torch.float64, device=DEV) + b
        E = torch.zeros_like(z) + b.abs()
        for t, xt in enumerate(_taps(x)):
            z += xt @ w[t].t().contiguous()
            E += xt.abs() @ w[t].abs().t().contiguous()
        k = 27 * x.shape[-1] + 1
        _check_rounded(A[out].double().reshape(z.shape), torch.relu(z), _gamma(k) * E, f"conv {l} {io} -> {out}")


@pytest.mark.parametrize("B,S", [(5, 32), (2, 64)])
def test_network_gradient_against_the_same_steps_in_float64(B, S):
    """The gradient of a batch against the same backward steps from the library's own
    activations, in float64 with the library's bf16 rounding of every gradient that
    it stores, an explicit concatenation and a ReLU mask of its own.  A float32 sum
    falls on the other side of a bf16 rounding than its float64 value for some 0.5 %
    of the elements (2^-24 sqrt(2592) of the sum against a spacing of 2^-8): 2e-4 of
    a tensor's norm, 6e-4 after ten layers; 3e-3 per layer here, where a wrong row
    or edge of a tile changes 1e-2 and more."""
    print(f"[case] network gradient B={B} S={S}", flush=True)
    W, wh, A, u, grad = _net_on_volumes(B, S)
    bf = lambda t: t.float().bfloat16().double()  # noqa: E731
    relu = lambda d, i: torch.where(A[i].double() > 0, d, torch.zeros_like(d))  # noqa: E731
    io = {l: x for l, x, _ in _CONV_IO}

    def layer(l, dz, want_dx=True):
        """Check layer l's gradients for dz, return its input's gradient (bf16)."""
        w, _, ws, bs = W[l]
        zf = dz.reshape(-1, dz.shape[-1])
        dw = torch.stack([zf.t().contiguous() @ xt for xt in _taps(_input_of(A, io[l]))])
        for what, ref, sl in (("weights", dw.reshape(-1), ws), ("biases", zf.sum(0), bs)):
            rel = float(torch.linalg.norm(grad[sl] - ref) / torch.linalg.norm(ref))
            print(f"  layer {l} {what}: rel {rel:.2e}", flush=True)
            assert rel < 3e-3, (l, what)
        if not want_dx:
            return None
        dx = torch.zeros((zf.shape[0], w.shape[2]), dtype=torch.float64, device=DEV)
        for t in range(27):
            dx += torch.roll(dz, (t // 9 - 1, (t // 3) % 3 - 1, t % 3 - 1), (1, 2, 3)).reshape(zf.shape) @ w[t]
        return bf(dx.reshape(dz.shape[:-1] + (w.shape[2],)))

    def fold(d):  # sum over the 2^3 children
        Bd, n, C = d.shape[0], d.shape[1] // 2, d.shape[-1]
        return d.reshape(Bd, n, 2, n, 2, n, 2, C).sum(dim=(2, 4, 6))

    e = A[15].double().reshape(u.shape) - (u.float() / U.U_SCALE).double()
    d = 2.0 * e / e.numel()
    h5 = A[14].double()
    assert torch.allclose((d[..., None] * h5).sum((0, 1, 2, 3)), grad[-17:-1], rtol=1e-3, atol=1e-3 * float(grad[-17:-1].abs().max()))
    dz = relu(bf(d[..., None] * wh), 14)
    dz = relu(layer(9, dz), 13)
    dcat5 = layer(8, dz)
    dz = relu(bf(fold(dcat5[..., :32])), 11)
    dz = relu(layer(7, dz), 10)
    dcat4 = layer(6, dz)
    dz = relu(bf(fold(dcat4[..., :64])), 8)
    dz = relu(layer(5, dz), 7)
    dp2 = layer(4, dz)
    dz = relu(bf(dcat4[..., 64:] + _up(dp2) / 8), 5)
    dz = relu(layer(3, dz), 4)
    dp1 = layer(2, dz)
    dz = relu(bf(dcat5[..., 32:] + _up(dp1) / 8), 2)
    dz = relu(layer(1, dz), 1)
    layer(0, dz, want_dx=False)


@pytest.mark.parametrize("off", [1, 3, 4])
@pytest.mark.parametrize("S,Cin,Cout", [(8, 16, 32), (16, 48, 16)])
def test_conv_backward_weight_from_inputs_at_any_element(S, Cin, Cout, off):
    """x and dZ one, three and four elements past an aligned address, on small
    integers (exact in any order): the gradients of the aligned inputs."""
    mg = _mg()
    print(f"[case] conv wgrad from offset inputs S={S} Cin={Cin} Cout={Cout} off={off}", flush=True)
    g = torch.Generator().manual_seed(S + off)
    x = torch.randint(-3, 4, (1, S, S, S, Cin), generator=g).to(torch.bfloat16).to(DEV)
    dz = torch.randint(-3, 4, (1, S, S, S, Cout), generator=g).to(torch.bfloat16).to(DEV)
    want, want_b = mg.conv3d_bwd_weight(x, dz)
    xo, zo = (torch.zeros(t.numel() + off, dtype=torch.bfloat16, device=DEV) for t in (x, dz))
    xo[off:] = x.reshape(-1)
    zo[off:] = dz.reshape(-1)
    dw, db = torch.zeros_like(want), torch.zeros_like(want_b)
    assert mg.lib().mgfr_conv3d_bwd_weight(xo.data_ptr() + 2 * off, zo.data_ptr() + 2 * off, 1, S, Cin, Cout,
                                           dw.data_ptr(), db.data_ptr(), mg._stream_ptr()) == 0
    torch.cuda.synchronize()
    assert torch.equal(dw, want) and torch.equal(db, want_b)


@pytest.mark.parametrize("B,S,Cin,Cout", [(1, 8, 96, 96), (2, 16, 96, 80), (1, 16, 80, 80)])
def test_conv_backward_weight_of_the_widest_layers(B, S, Cin, Cout):
    """Up to the 36 pairs of 16-channel blocks that the entry point takes, on small
    integers (exact in any order): every block of every tap is there."""
    mg = _mg()
    print(f"[case] conv wgrad widest B={B} S={S} Cin={Cin} Cout={Cout}", flush=True)
    g = torch.Generator().manual_seed(Cin + Cout)
    x = torch.randint(-3, 4, (B, S, S, S, Cin), generator=g).to(torch.bfloat16).to(DEV)
    dz = torch.randint(-3, 4, (B, S, S, S, Cout), generator=g).to(torch.bfloat16).to(DEV)
    dw, db = mg.conv3d_bwd_weight(x, dz)
    zf = dz.double().reshape(-1, Cout).t().contiguous()
    assert torch.equal(dw.double(), torch.stack([zf @ xt for xt in _taps(x.double())]))
    assert torch.equal(db.double(), zf.sum(1))
