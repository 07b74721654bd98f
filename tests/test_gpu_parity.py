"""Parity of the HIP path against the CPU oracle, element by element, through the C ABI."""
import numpy as np
import pytest

import workloads as wl
from oracle import lpref
from tests.gpu_common import compare_step, gpu_mini_basic, gpu_mini_bottleneck, gpu_mini_wide, say
from tests.helpers import rel_err

pytestmark = pytest.mark.gpu


def test_im2col_offsets_bit_exact():
    """The device's im2col address arithmetic equals the oracle's canonical index function exactly."""
    import torch
    from paper_2112_05387_amd import binding as B
    rng = np.random.default_rng(0)
    for (N, H, W, Cin, R, stride, pad) in [(4, 8, 8, 16, 3, 1, 1), (128, 32, 32, 160, 3, 1, 1), (128, 32, 32, 160, 3, 2, 1),
                                            (64, 224, 224, 3, 7, 2, 3), (3, 6, 6, 8, 1, 2, 0), (128, 32, 32, 3, 3, 4, 1)]:
        Ho, Wo = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
        M, Kg = N * Ho * Wo, R * R * Cin
        cnt = 4096
        m = rng.integers(0, M, cnt); q = rng.integers(0, Kg, cnt)
        m[:4] = [0, 0, M - 1, M - 1]; q[:4] = [0, Kg - 1, 0, Kg - 1]
        want = np.array([lpref.im2col_index(int(a), int(b), H, W, Cin, R, R, stride, pad) for a, b in zip(m, q)], dtype=np.int64)
        dm = torch.from_numpy(m.astype(np.int64)).cuda(); dq = torch.from_numpy(q.astype(np.int64)).cuda()
        out = torch.empty(cnt, dtype=torch.int64, device="cuda")
        B.lp_debug_im2col_offsets(torch.cuda.current_stream().cuda_stream, H, W, Cin, R, R, stride, pad,
                                  dm.data_ptr(), dq.data_ptr(), out.data_ptr(), cnt)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tiny(dtype):
    net = wl.make_config("tiny")
    net.dtype = dtype
    say("case tiny", dtype)
    compare_step(net, want_dx0=True, max_uncovered=0)      # one block per module: every tensor is compared


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_mini_basic_al(dtype):
    net = gpu_mini_basic(dtype=dtype)
    net.al, net.lam_sigma, net.rho = True, 0.05, 1.5
    say("case mini_basic", dtype)
    compare_step(net, scale=0.5)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_block_options(dtype):
    """post_relu and proj_plain: the whole step end to end (entry-point pass and fused pass)."""
    from tests.gpu_common import gpu_mini_basic_flags
    net = gpu_mini_basic_flags(dtype=dtype)
    net.al, net.lam_sigma = True, 0.05
    say("case block options", dtype)
    compare_step(net)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_mini_bottleneck(dtype):
    net = gpu_mini_bottleneck(dtype=dtype)
    say("case mini_bottleneck", dtype)
    compare_step(net)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_layer_serial_k1(dtype):
    """K = 1: one module holds the whole network, the step is ordinary back-propagation of the cross-entropy
    (no interface, no auxiliary variable, no multiplier)."""
    say("case mini_basic K=1", dtype)
    compare_step(gpu_mini_basic(dtype=dtype, serial=True))


def test_wrn_layer_serial_reduced_batch():
    say("case wrn28_10 K=1 batch 2 bf16")
    compare_step(wl.make_config("wrn28_10", batch=2, split=[12]))


@pytest.mark.parametrize("dtype,serial", [("f32", False), ("bf16", False), ("f32", True)])
def test_pre_activation_order(dtype, serial):
    """BN-ReLU-conv blocks (Fig. 2), bare conv stem, BN-ReLU head: the mini network with K = 3 and as one module."""
    from workloads import configs as cfg
    net = cfg.with_order(gpu_mini_basic(dtype=dtype, serial=serial), "pre")
    net.al, net.lam_sigma, net.rho = True, 0.05, 1.5
    say("case mini_basic pre-activation", dtype, "K=1" if serial else "K=3")
    compare_step(net, scale=0.5)


def test_pre_activation_stemless_dx0():
    """Pre-activation blocks without a stem (the statistics of the module input come from the stand-alone
    reduction), dx[0] requested."""
    from workloads import configs as cfg
    net = wl.make_config("tiny")
    cfg.with_order(net, "pre")
    say("case tiny pre-activation f32")
    compare_step(net, want_dx0=True)


def test_wrn_pre_activation_reduced_batch():
    from workloads import configs as cfg
    say("case wrn28_10 pre-activation batch 2 bf16")
    compare_step(cfg.with_order(wl.make_config("wrn28_10", batch=2), "pre"))


@pytest.mark.parametrize("lanes", [None, [1, 2, 3], [0, 1, 1], [2, 0, 2]])
def test_stream_lanes(lanes):
    """The same step with every module on the caller's stream, every module on a stream of its own, and mixed
    groupings: each must meet the parity bar (run twice in a row: the second pass re-forks from the joined stream)."""
    net = gpu_mini_basic(dtype="bf16")
    net.al, net.lam_sigma = True, 0.05
    say("case stream lanes", lanes)
    compare_step(net, lanes=lanes)


@pytest.mark.parametrize("mask,fused", [(0b101, True), (0b010, True), (0b110, False), (0b001, False)])
def test_module_mask_subsets(mask, fused):
    """A call with a module mask does exactly the selected modules: their outputs equal those of the all-modules call
    (to fp32 summation order: the grouped launches hold other problems), and nothing that belongs to an unselected
    module is written (outputs, adjoints, gradients, losses, multipliers keep a sentinel)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.gpu_common import load_step
    from tests.helpers import step_inputs
    net = gpu_mini_basic(dtype="f32")
    net.al, net.lam_sigma, net.rho = True, 0.05, 1.5
    K, rho, scale, mstep = net.K, net.rho, 0.5, 0.1
    say("case module mask", bin(mask), "one call" if fused else "four calls")
    inp = step_inputs(net, lpref)

    def run(ls, m):
        if fused:
            ls.local_step(rho, scale, mstep, mask=m)
        else:
            ls.module_forward(mask=m)
            ls.local_loss_grad(rho, scale, mask=m)
            ls.module_backward(mask=m)
        torch.cuda.synchronize()

    def state(ls):
        out = {"loss": ls.loss.clone(), "logits": ls.logits.clone(), "dlogits": ls.dlogits.clone()}
        for k in range(K):
            out[f"dparams{k}"] = ls.dparams[k].clone()
            out[f"dx{k}"] = ls.dx[k].clone()
            if k < K - 1:
                out[f"y{k}"] = ls.y[k].clone(); out[f"dy{k}"] = ls.dy[k].clone(); out[f"lam{k}"] = ls.lam[k].clone()
        return out

    owner = lambda name: K - 1 if name in ("logits", "dlogits") else int(name[-1])
    ls = LocalStep(net)
    try:
        load_step(ls, net, inp)
        run(ls, None)
        full = state(ls)
        # fresh multipliers, sentinels everywhere an entry point writes
        ls.set_lams(inp["lams"])
        lam0 = [l.clone() for l in ls.lam]
        sentinel = 12345.0
        for t in [ls.loss, ls.logits, ls.dlogits] + ls.dparams + ls.dx + ls.y + ls.dy:
            t.fill_(sentinel)
        run(ls, mask)
        got = state(ls)
        for name, t in got.items():
            if name == "loss":
                for k in range(K):
                    if (mask >> k) & 1:
                        assert abs(float(t[k]) - float(full["loss"][k])) <= 1e-5 * abs(float(full["loss"][k])), (name, k)
                    else:
                        assert float(t[k]) == sentinel, (name, k)
                continue
            k = owner(name)
            sel = (mask >> k) & 1
            if name.startswith("lam"):
                want = full[name] if (sel and fused) else lam0[k]     # only the one call carries the multiplier update
                assert torch.equal(t, want) if not (sel and fused) else torch.allclose(t, want, rtol=1e-5, atol=1e-6), name
            elif name.startswith("dx") and (k == 0 or not sel):
                assert bool((t == sentinel).all()), name              # dx[0] is not asked for; unselected modules
            elif sel:
                assert torch.allclose(t, full[name], rtol=1e-4, atol=1e-6), (name, float((t - full[name]).abs().max()))
            else:
                assert bool((t == sentinel).all()), name
    finally:
        ls.close()


@pytest.mark.parametrize("which", ["mini_basic", "wrn28_10", "narrow_f32", "narrow_bf16", "narrow_lanes"])
def test_step_as_hip_graph_replays(which):
    """The local step captured into a HIP graph (the stream lanes forked and joined by events inside the capture, the
    multiplier update included): three replays, with eager work of the library and synchronisations between them, each
    against the eager step from the same state.  mini_basic: three lanes, register-staged kernels; wrn28_10 at batch 2:
    four lanes, the wide-layer kernels with their split-K atomics; narrow: the folded passes, on one stream and on two lanes."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_common import load_step
    from tests.helpers import step_inputs
    from tests.test_gpu_narrow import narrow_net
    if which == "mini_basic":
        net = gpu_mini_basic(dtype="bf16")
        net.al, net.lam_sigma, net.rho = True, 0.05, 1.5
    elif which.startswith("narrow"):
        net = narrow_net(3, (16, 16), dtype="bf16" if which == "narrow_bf16" else "f32")
        net.al, net.lam_sigma, net.rho = True, 0.05, 1.5
    else:
        net = wl.make_config("wrn28_10", batch=2)
        net.aux = None
    K, scale, mstep = net.K, 0.5, 0.1
    say("case step as a HIP graph", which)
    inp = step_inputs(net, lpref)
    ls = LocalStep(net)
    try:
        load_step(ls, net, inp)
        if which == "narrow_lanes":
            ls.set_stream_lanes([1, 2])
        assert B.lp_debug_stream_lanes(ls.net, K)[0] == which.startswith("narrow")

        def snapshot():
            torch.cuda.synchronize()
            return ([g.clone() for g in ls.dparams] + [l.clone() for l in ls.lam] + [y.clone() for y in ls.y]
                    + [ls.loss.clone(), ls.logits.clone()] + [d.clone() for d in ls.dx[1:]])

        want = []
        for _ in range(3):                       # eager: three steps in a row, multipliers carried along
            ls.step(net.rho, scale, mstep)
            want.append(snapshot())
        ls.set_lams(inp["lams"])
        g = ls.capture_step(net.rho, scale, mstep)
        for l, src in zip(ls.lam, inp["lams"]):  # the warm-up steps moved the multipliers; the graph holds these very
            l.copy_(ls.to_dev(src))              # tensors, so they are reset in place
        for rep in range(3):
            for t in ls.dparams + ls.y + [ls.loss, ls.logits]:
                t.fill_(777.0)
            torch.cuda.synchronize()
            g.replay()
            got = snapshot()
            for i, (a, b) in enumerate(zip(got, want[rep])):
                assert torch.allclose(a.float(), b.float(), rtol=2e-3, atol=1e-5), (rep, i, float((a.float() - b.float()).abs().max()))
            ls.module_forward(mask=0b001)        # eager work between the replays (it rewrites y[0] with the same values)
            torch.cuda.synchronize()
    finally:
        ls.close()


def test_mini_wide_ragged_tiles():
    say("case mini_wide bf16")
    compare_step(gpu_mini_wide())


@pytest.mark.parametrize("side,widths", [((12, 20), (136, 296)), ((12, 10), (160, 320)), ((8, 8), (320, 640))])
def test_mini_wide_stride_2(side, widths):
    """A stride-2 3x3 layer between wide widths (the 160->320 and 320->640 layers of WRN-28-10 in small): its filter
    gradient goes through the register-staged kernel (ragged 160-wide tiles, output widths 10, 5 and 4)."""
    from tests.gpu_common import gpu_mini_wide_strided
    say("case mini_wide stride 2", side, widths)
    compare_step(gpu_mini_wide_strided(side=side, widths=widths))


def test_resnet20_full_size():
    say("case resnet20 batch 128 fp32")
    compare_step(wl.make_config("resnet20"))


def test_resnet56_auxnet_al():
    say("case resnet56 batch 16 bf16")
    compare_step(wl.make_config("resnet56", batch=16))


def test_wrn_reduced_batch():
    say("case wrn28_10 batch 2 bf16")
    compare_step(wl.make_config("wrn28_10", batch=2))


def _resnet50_at(side, batch):
    """ResNet-50 (real depth and widths, 7x7 stride-2 stem + max-pool, 1000 classes) at another input resolution."""
    from workloads import configs as cfg
    ref = wl.make_config("resnet50", batch=batch)
    blocks = [b for m in ref.modules for b in m.blocks]
    m0 = ref.modules[0]
    net = cfg._assemble(f"resnet50_{side}", cfg._split(blocks, [len(m.blocks) for m in ref.modules]), batch, side, side, m0.C,
                        m0.stem, m0.stem_cout, ref.modules[-1].n_classes, seed=ref.seed)
    net.dtype = ref.dtype
    return net


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_resnet50_reduced_resolution(dtype):
    """The ImageNet-shaped network (bottleneck blocks up to 2048 channels, 7x7 stride-2 stem + max-pool, 1000 classes)
    at 64x64 and mini-batch 4: every tensor of the step, 1e-4 in fp32."""
    say("case resnet50 at 64x64, batch 4", dtype)
    net = _resnet50_at(64, 4)
    net.dtype = dtype
    compare_step(net)


def test_resnet50_full_resolution_reduced_batch():
    """The same network at 224x224, mini-batch 2, bf16 (the kernels at the real shapes: 112x112 stem output, 56x56 to
    7x7 stages).  Forward outputs and losses are held to 2e-2.  The backward tensors of these 13-16-conv modules at two
    samples per batch statistic are so sensitive to single roundings that the oracle's own spread (which the comparison
    prints and allows for) is of order one for most of them.  fp32 at this size is not a case either: after a dozen
    layers the device's fp32 forward differs from the float64 one by 2e-6, the 56x56 layers have 400k ReLU inputs each,
    two of them within 1e-6 of zero, and one flipped mask element moves a filter gradient summed over 6272 pixels by
    about 1e-2 of its norm (the oracle does the same when its stored tensors are perturbed by 1e-7; seen at 96x96
    too, where the device's and the oracle's masks of one layer differ in exactly one element whose input is
    2e-7); hence the strict comparison at 64x64 above."""
    say("case resnet50 at 224x224, batch 2, bf16")
    compare_step(wl.make_config("resnet50", batch=2))


@pytest.mark.parametrize("dtype,al", [("f32", True), ("f32", False), ("bf16", True)])
def test_aux_variable_update(dtype, al):
    """x_k <- x_k - eta*(scale*(rho*(x_k - y_{k-1}) - lam_{k-1}) + dx_k) on seeded tensors, element by element
    (ragged size: the 6x6 mini network)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.helpers import rel_err, store
    net = gpu_mini_basic(dtype=dtype)
    rho, scale, eta = 1.5, 0.5, 0.3
    say("case aux_variable_update", dtype, "AL" if al else "penalty")
    ls = LocalStep(net)
    try:
        xs = [store(net, wl.normal(31, f"x{k}", s)) for k, s in enumerate(ls.x_shapes)]
        ys = [store(net, wl.normal(31, f"y{k}", s)) for k, s in enumerate(ls.y_shapes)]
        dxs = [store(net, wl.normal(31, f"dx{k}", s, 0.3)) for k, s in enumerate(ls.x_shapes)]
        lams = [store(net, wl.normal(31, f"lam{k}", s, 0.2)) for k, s in enumerate(ls.y_shapes)] if al else None
        for k in range(net.K):
            ls.set_x(k, xs[k])
            ls.dx[k].copy_(ls.to_dev(dxs[k]))
        for k in range(net.K - 1):
            ls.y[k].copy_(ls.to_dev(ys[k]))
        ls.set_lams(lams)
        ls.aux_variable_update(rho, scale, eta)
        torch.cuda.synchronize()
        tol = 1e-6 if dtype == "f32" else 4e-3          # fp32: a few roundings; bf16: one storage rounding of the result
        assert np.array_equal(ls.to_host(ls.x[0]), xs[0])            # x_0 is the mini-batch: untouched
        for k in range(1, net.K):
            want = lpref.aux_variable_update(xs[k], ys[k - 1], dxs[k], None if lams is None else lams[k - 1], rho, eta, scale)
            assert rel_err(ls.to_host(ls.x[k]), want) <= tol, (k, rel_err(ls.to_host(ls.x[k]), want))
    finally:
        ls.close()


@pytest.mark.parametrize("dtype,momentum,wd,use_master", [("f32", 0.0, 0.0, False), ("f32", 0.9, 5e-4, False),
                                                          ("bf16", 0.0, 0.0, False), ("bf16", 0.9, 5e-4, True)])
def test_sgd_update(dtype, momentum, wd, use_master):
    """Two parameter updates in a row from seeded gradients, every tensor of every module, element by element
    (tensor sizes from 4 to a few thousand elements: ragged tails of the 4096-element blocks).  bf16 parameters
    without a master copy are re-rounded after each update, as the oracle's inputs are."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.helpers import rel_err
    net = gpu_mini_basic(dtype=dtype)
    lr = 0.05
    say("case sgd_update", dtype, momentum, wd, "master" if use_master else "")
    ls = LocalStep(net)
    try:
        W = [wl.make_params(net, k) for k in range(net.K)]
        for k in range(net.K):
            ls.set_params(k, W[k])
        from paper_2112_05387_amd import binding as B
        lowp = [[info.dtype == B.LP_BF16 for info in ls.tables[k]] for k in range(net.K)]
        stored = [[wl.round_bf16(w) if lp else np.asarray(w, np.float32).astype(np.float64) for w, lp in zip(W[k], lowp[k])]
                  for k in range(net.K)]
        vel = [torch.zeros_like(d) for d in ls.dparams] if momentum else None
        master = None
        if use_master:
            master = [torch.zeros_like(d) for d in ls.dparams]
            for k in range(net.K):
                for info, w in zip(ls.tables[k], W[k]):
                    o = info.grad_offset // 4
                    master[k][o:o + int(info.numel)].copy_(torch.from_numpy(np.asarray(w, np.float32).reshape(-1)))
        cur = [[np.asarray(w, np.float32).astype(np.float64) for w in W[k]] for k in range(net.K)] if use_master else stored
        v = [[None] * len(W[k]) for k in range(net.K)]
        for it in range(2):
            G = [[np.asarray(wl.normal(77 + it, f"g{k}.{i}", np.shape(w), 0.5), np.float32).astype(np.float64)
                  for i, w in enumerate(W[k])] for k in range(net.K)]
            for k in range(net.K):
                for info, g in zip(ls.tables[k], G[k]):
                    o = info.grad_offset // 4
                    ls.dparams[k][o:o + int(info.numel)].copy_(torch.from_numpy(g.astype(np.float32).reshape(-1)))
            ls.sgd_update(lr, momentum, wd, velocity=vel, master=master)
            torch.cuda.synchronize()
            for k in range(net.K):
                for i, info in enumerate(ls.tables[k]):
                    w_new, v_new = lpref.sgd_update(cur[k][i], G[k][i], lr, v[k][i], momentum, wd)
                    v[k][i] = v_new
                    n = int(info.numel)
                    if info.dtype == B.LP_BF16:
                        got = ls.params[k][info.offset:info.offset + 2 * n].view(torch.bfloat16)
                    else:
                        got = ls.params[k][info.offset:info.offset + 4 * n].view(torch.float32)
                    got = ls.to_host(got).reshape(np.shape(w_new))
                    tol = 4e-3 if info.dtype == B.LP_BF16 else 1e-6
                    assert rel_err(got, w_new) <= tol, (it, k, i, rel_err(got, w_new))
                    if use_master:
                        o = info.grad_offset // 4
                        gm = ls.to_host(master[k][o:o + n]).reshape(np.shape(w_new))
                        assert rel_err(gm, w_new) <= 1e-6, (it, k, i, "master", rel_err(gm, w_new))
                        cur[k][i] = w_new
                    else:
                        cur[k][i] = got              # the next update starts from the stored (re-rounded) parameters
                    if momentum:
                        o = info.grad_offset // 4
                        gv = ls.to_host(vel[k][o:o + n]).reshape(np.shape(w_new))
                        assert rel_err(gv, v_new) <= 1e-6, (it, k, i, "velocity", rel_err(gv, v_new))
    finally:
        ls.close()


def _grad_names(n):
    return [f"b{i // 3}.{('dW', 'dgamma', 'dbeta')[i % 3]}" for i in range(n)]


@pytest.mark.parametrize("dtype,extra", [("f32", 0), ("bf16", 0), ("f32", 2), ("bf16", 2)])
def test_auxnet_distill_grad(dtype, extra):
    """loss_j = scale*|AuxNet_j(image) - target_j|^2 and d loss_j / d theta_j for every AuxNet of the ResNet-56
    configuration (strides 1, 2, 4; batch 8), target = seeded perturbation of the oracle's AuxNet output.
    extra: that many more blocks in every AuxNet (the first does the change of shape)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.helpers import rel_err, store
    from workloads import configs as cfg
    net = wl.make_config("resnet56", batch=8)
    if extra:
        cfg.deepen_aux(net, extra)
    net.dtype = dtype
    scale = 0.5
    tol = 1e-4 if dtype == "f32" else 2e-2
    q = None if dtype == "f32" else wl.round_bf16
    say("case auxnet_distill_grad", dtype, "blocks per AuxNet:", extra + 1)
    image = wl.make_image(net)
    auxp = [wl.make_aux_params(net, j) for j in range(net.K - 1)]
    ls = LocalStep(net)
    try:
        ls.set_x(0, image)
        targets = []
        for j in range(net.K - 1):
            ls.set_aux_params(j, auxp[j])
            out = lpref.auxnet_forward(net.aux[j], image, auxp[j], net.bn_eps, q)
            targets.append(store(net, out + wl.normal(41, f"distill{j}", out.shape, 0.5)))
        ls.auxnet_forward()
        for j in range(net.K - 1):
            ls.x[j + 1].copy_(ls.to_dev(targets[j]))        # the corrected auxiliary variables are the targets
        ls.auxnet_distill_grad(scale)
        torch.cuda.synchronize()
        errs = {}
        for j in range(net.K - 1):
            loss, grads = lpref.auxnet_distill_grad(net.aux[j], image, auxp[j], targets[j], net.bn_eps, scale, q)
            errs[f"aux{j}.loss"] = abs(float(ls.aux_loss[j].item()) - loss) / abs(loss)
            got = ls.get_aux_grads(j)
            assert len(got) == len(grads) == 3 * (len(net.aux[j].mid) + 1)
            for name, g, r in zip(_grad_names(len(grads)), got, grads):
                errs[f"aux{j}.{name}"] = rel_err(g, r)
        top = sorted(errs.items(), key=lambda kv: -kv[1])[:4]
        say("    worst: " + ", ".join(f"{k}={v:.2e}" for k, v in top))
        bad = {k: v for k, v in errs.items() if not v <= tol}
        assert not bad, bad
    finally:
        ls.close()


@pytest.mark.parametrize("dtype,al,stack", [("f32", True, False), ("f32", False, False), ("bf16", True, False),
                                            ("f32", False, True), ("bf16", True, True)])
def test_reauxnet_grad(dtype, al, stack):
    """Gradient of the relaxed objective with respect to the parameters of every AuxNet of the ResNet-56
    configuration (strides 1, 2, 4; batch 8) when x_k = AuxNet_k(image): seeded F_{k-1}(x_{k-1}), dx_k and
    multipliers, then the sequence AuxNet gradient -> descent step on the AuxNet parameters.
    stack: x_k comes from a stack of k blocks of its own (block i maps the shape of x_i to that of x_{i+1}; K = 8, so
    up to seven blocks, two of them with stride 2), the recursion of Sec. 4.4 at full depth; else from one strided block."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.helpers import rel_err, store
    from workloads import configs as cfg
    net = wl.make_config("resnet56", batch=8)
    if stack and dtype == "bf16":
        # In bf16 a stack of five or more blocks is no longer a parity case at a fixed tolerance: with the seeded
        # (white-noise) output gradients used here, the oracle's own result moves by 2-20 % when relative noise of
        # 2e-7 (fp32 instead of fp64 accumulation) is put in front of its bf16 roundings, through ReLU masks that flip
        # block after block; up to four blocks it moves by less than 6e-3.  So bf16 runs the K = 4 wide network
        # (stacks of 1..3 blocks, 3->160, 160->320 stride 2, 320->640 stride 2) and fp32 the K = 8 one (1..7 blocks).
        net = wl.make_config("wrn28_10", batch=2)
    if stack:
        cfg.reaux(net)
        assert [len(a.mid) for a in net.aux] == list(range(net.K - 1))
    net.dtype = dtype
    rho, scale, lr = 1.3, 0.5, 0.05
    tol = 1e-4 if dtype == "f32" else 2e-2
    q = None if dtype == "f32" else wl.round_bf16
    say("case reauxnet_grad", dtype, "AL" if al else "penalty", "stacks" if stack else "one block")
    image = wl.make_image(net)
    auxp = [wl.make_aux_params(net, j) for j in range(net.K - 1)]
    ls = LocalStep(net)
    try:
        ls.set_x(0, image)
        yp, dxs, lams = [], [], []
        for j in range(net.K - 1):
            ls.set_aux_params(j, auxp[j])
            shp = ls.y_shapes[j]
            yp.append(store(net, wl.normal(43, f"yprev{j}", shp)))
            dxs.append(store(net, wl.normal(43, f"dx{j}", shp, 0.3)))
            lams.append(store(net, wl.normal(43, f"lam{j}", shp, 0.2)))
            ls.y[j].copy_(ls.to_dev(yp[j]))
            ls.dx[j + 1].copy_(ls.to_dev(dxs[j]))
        ls.set_lams(lams if al else None)
        ls.auxnet_forward()
        ls.reauxnet_grad(rho, scale)
        torch.cuda.synchronize()
        errs = {}
        want = []
        for j in range(net.K - 1):
            grads = lpref.reauxnet_grad(net.aux[j], image, auxp[j], yp[j], dxs[j], lams[j] if al else None, rho, scale,
                                        net.bn_eps, q)
            want.append(grads)
            got = ls.get_aux_grads(j)
            assert len(got) == len(grads) == 3 * (len(net.aux[j].mid) + 1)
            for name, g, r in zip(_grad_names(len(grads)), got, grads):
                errs[f"aux{j}.{name}"] = rel_err(g, r)
        top = sorted(errs.items(), key=lambda kv: -kv[1])[:4]
        say("    worst: " + ", ".join(f"{k}={v:.2e}" for k, v in top))
        bad = {k: v for k, v in errs.items() if not v <= tol}
        assert not bad, bad
        # descent step on the AuxNet parameters from the device's own gradients
        dev_g = [ls.get_aux_grads(j) for j in range(net.K - 1)]
        ls.sgd_update_aux(lr)
        torch.cuda.synchronize()
        from paper_2112_05387_amd import binding as B
        for j in range(net.K - 1):
            for info, w, g in zip(ls.aux_tables[j], auxp[j], dev_g[j]):
                n = int(info.numel)
                lowp = info.dtype == B.LP_BF16
                w0 = wl.round_bf16(w) if lowp else np.asarray(w, np.float32).astype(np.float64)
                w_new, _ = lpref.sgd_update(w0, g, lr)
                raw = ls.aux_params[j][info.offset:info.offset + (2 if lowp else 4) * n]
                got = ls.to_host(raw.view(torch.bfloat16 if lowp else torch.float32)).reshape(np.shape(w_new))
                assert rel_err(got, w_new) <= (4e-3 if lowp else 1e-6), (j, info.ndim, rel_err(got, w_new))
    finally:
        ls.close()


@pytest.mark.parametrize("dtype,extra", [("f32", 0), ("bf16", 0), ("f32", 1), ("bf16", 1)])
def test_chained_auxnet(dtype, extra):
    """AuxNets that read the previous auxiliary variable (x_{j+1} = AuxNet_j(x_j)), ResNet-56 shapes at batch 8:
    the forward chain, then the distillation gradients at corrected auxiliary variables (each AuxNet is run again from
    its corrected input).  extra: that many more blocks per AuxNet."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.helpers import rel_err, store
    from workloads import configs as cfg
    net = cfg.chain_aux(wl.make_config("resnet56", batch=8))
    if extra:
        cfg.deepen_aux(net, extra)
    net.dtype = dtype
    scale = 0.5
    tol = 1e-4 if dtype == "f32" else 2e-2
    q = None if dtype == "f32" else wl.round_bf16
    say("case chained auxnet", dtype, "blocks per AuxNet:", extra + 1)
    image = wl.make_image(net)
    auxp = [wl.make_aux_params(net, j) for j in range(net.K - 1)]
    ls = LocalStep(net)
    try:
        ls.set_x(0, image)
        for j in range(net.K - 1):
            ls.set_aux_params(j, auxp[j])
        ls.auxnet_forward()
        torch.cuda.synchronize()
        errs = {}
        x = image
        for j in range(net.K - 1):              # every block against the oracle on the DEVICE's stored input
            want = lpref.auxnet_forward(net.aux[j], x, auxp[j], net.bn_eps)
            errs[f"x{j + 1}"] = rel_err(ls.to_host(ls.x[j + 1]), want)
            x = ls.to_host(ls.x[j + 1])
        corrected = [store(net, ls.to_host(ls.x[j + 1]) + wl.normal(47, f"corr{j}", ls.x[j + 1].shape, 0.5))
                     for j in range(net.K - 1)]
        for j in range(net.K - 1):
            ls.x[j + 1].copy_(ls.to_dev(corrected[j]))
        ls.auxnet_distill_grad(scale)
        torch.cuda.synchronize()
        for j in range(net.K - 1):
            x_in = image if j == 0 else corrected[j - 1]
            loss, grads = lpref.auxnet_distill_grad(net.aux[j], x_in, auxp[j], corrected[j], net.bn_eps, scale, q)
            errs[f"aux{j}.loss"] = abs(float(ls.aux_loss[j].item()) - loss) / abs(loss)
            got = ls.get_aux_grads(j)
            assert len(got) == len(grads) == 3 * (len(net.aux[j].mid) + 1)
            for name, g, r in zip(_grad_names(len(grads)), got, grads):
                errs[f"aux{j}.{name}"] = rel_err(g, r)
        top = sorted(errs.items(), key=lambda kv: -kv[1])[:4]
        say("    worst: " + ", ".join(f"{k}={v:.2e}" for k, v in top))
        bad = {k: v for k, v in errs.items() if not v <= tol}
        assert not bad, bad
        with pytest.raises(Exception, match="recursive-AuxNet"):
            ls.reauxnet_grad(1.0)
    finally:
        ls.close()


@pytest.mark.parametrize("fused", [False, True])
def test_two_iterations_of_the_whole_method(fused):
    """Every entry point in sequence, twice: AuxNet forward -> module forward -> losses / terminal adjoints -> module
    backward -> multiplier update -> correction of the auxiliary variables -> parameter update -> AuxNet distillation
    gradient -> AuxNet parameter update, on the mini network in fp32, against the same sequence of oracle calls in
    float64.  Checks what feeds what between the calls; the tolerance allows for the cancellation in the residuals
    (see compare_step) accumulated over two iterations."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.helpers import rel_err
    from workloads.configs import AuxDesc
    net = gpu_mini_basic(dtype="f32")
    net.al, net.rho = True, 1.5
    net.aux = [AuxDesc(cin=3, cout=m.C, stride=net.modules[0].H // m.H, relu=False) for m in net.modules[1:]]
    K, scale, eta, lr, mstep = net.K, 0.5, 0.05, 0.02, 0.1
    say("case two iterations of the whole method")
    image, labels = wl.make_image(net), wl.make_labels(net)
    params = [wl.make_params(net, k) for k in range(K)]
    auxp = [wl.make_aux_params(net, j) for j in range(K - 1)]
    lams = [wl.normal(51, f"lam{k}", (net.modules[k + 1].N, net.modules[k + 1].H, net.modules[k + 1].W, net.modules[k + 1].C), 0.05)
            for k in range(K - 1)]
    f32 = lambda a: np.asarray(a, np.float32).astype(np.float64)
    params = [[f32(t) for t in p] for p in params]; auxp = [[f32(t) for t in p] for p in auxp]; lams = [f32(l) for l in lams]
    ls = LocalStep(net)
    try:
        for k in range(K):
            ls.set_params(k, params[k])
        for j in range(K - 1):
            ls.set_aux_params(j, auxp[j])
        ls.set_x(0, image)
        ls.set_lams(lams)
        ls.set_labels(labels)
        for it in range(2):
            # ---- device
            ls.auxnet_forward()
            if fused:
                ls.local_step(net.rho, scale, mult_step=mstep)
            else:
                ls.module_forward()
                ls.local_loss_grad(net.rho, scale)
                ls.module_backward()
                ls.al_multiplier_update(mstep)
            ls.aux_variable_update(net.rho, scale, eta)
            ls.sgd_update(lr)
            ls.auxnet_distill_grad(scale)
            ls.sgd_update_aux(lr)
            torch.cuda.synchronize()
            # ---- oracle, the same sequence
            xs = [image] + [lpref.auxnet_forward(net.aux[j], image, auxp[j], net.bn_eps) for j in range(K - 1)]
            out = lpref.local_step(net, xs, params, labels, lams, scale)
            new_lams = [lpref.multiplier_update(lams[k], out["y"][k], xs[k + 1], mstep) for k in range(K - 1)]
            new_xs = [image] + [lpref.aux_variable_update(xs[k], out["y"][k - 1], out["dx"][k], new_lams[k - 1], net.rho, eta, scale)
                                for k in range(1, K)]            # the multipliers were updated first, as on the device
            params = [[lpref.sgd_update(w, g, lr)[0] for w, g in zip(params[k], out["dparams"][k])] for k in range(K)]
            for j in range(K - 1):
                _, g = lpref.auxnet_distill_grad(net.aux[j], image, auxp[j], new_xs[j + 1], net.bn_eps, scale)
                auxp[j] = [lpref.sgd_update(w, gg, lr)[0] for w, gg in zip(auxp[j], g)]
            lams = new_lams
            errs = {}
            for k in range(1, K):
                errs[f"it{it}.x{k}"] = rel_err(ls.to_host(ls.x[k]), new_xs[k])
            for k in range(K - 1):
                errs[f"it{it}.lam{k}"] = rel_err(ls.to_host(ls.lam[k]), lams[k])
            for k in range(K):
                for i, info in enumerate(ls.tables[k]):
                    got = ls.to_host(ls.params[k][info.offset:info.offset + 4 * int(info.numel)].view(torch.float32))
                    errs[f"it{it}.m{k}.t{i}"] = rel_err(got.reshape(params[k][i].shape), params[k][i])
            for j in range(K - 1):
                for i, info in enumerate(ls.aux_tables[j]):
                    got = ls.to_host(ls.aux_params[j][info.offset:info.offset + 4 * int(info.numel)].view(torch.float32))
                    errs[f"it{it}.aux{j}.t{i}"] = rel_err(got.reshape(auxp[j][i].shape), auxp[j][i])
            top = sorted(errs.items(), key=lambda kv: -kv[1])[:4]
            say(f"    iteration {it}, worst: " + ", ".join(f"{k}={v:.2e}" for k, v in top))
            bad = {k: v for k, v in errs.items() if not v <= 1e-4}
            assert not bad, bad
    finally:
        ls.close()


def test_vanish_invariant_on_device():
    """x_{k+1} := the device's own F_k(x_k), zero multipliers: losses, terminal adjoints, weight gradients
    and dx of modules 0..K-2 are exactly zero."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from tests.gpu_common import load_step
    from tests.helpers import step_inputs
    net = gpu_mini_basic(dtype="bf16")
    inp = step_inputs(net, lpref)
    ls = LocalStep(net)
    try:
        load_step(ls, net, inp)
        for k in range(net.K - 1):          # serial pass on the device: x_{k+1} := F_k(x_k), one interface at a time
            ls.module_forward()
            ls.x[k + 1].copy_(ls.y[k])
        ls.module_forward()
        ls.local_loss_grad(3.0)
        ls.module_backward()
        torch.cuda.synchronize()
        for k in range(net.K - 1):
            assert float(ls.loss[k].item()) == 0.0
            assert not ls.dy[k].float().abs().max().item() > 0
            assert all(not np.any(g) for g in ls.get_grads(k))
            if k > 0:
                assert not ls.dx[k].float().abs().max().item() > 0
        assert float(ls.loss[net.K - 1].item()) > 0
    finally:
        ls.close()


@pytest.mark.parametrize("which", ["mini_basic_f32", "mini_bottleneck_bf16", "wrn28_10_batch_4"])
def test_deterministic_mode_is_bit_identical(which):
    """lp_net_set_deterministic: two runs of the same step (default stream lanes, fused call) give bit-identical
    outputs, gradients, adjoints and multipliers, and they agree with the default (atomic) mode within rounding (in
    bf16 that comparison covers the forward pass, losses' adjoints and multipliers)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    net = {"mini_basic_f32": lambda: gpu_mini_basic(batch=3, dtype="f32"),
           "mini_bottleneck_bf16": lambda: gpu_mini_bottleneck(batch=2, dtype="bf16"),
           "wrn28_10_batch_4": lambda: wl.make_config("wrn28_10", batch=4)}[which]()
    if which != "wrn28_10_batch_4":
        net.al, net.lam_sigma = True, 0.05
    params, image, labels, xs, lams = seeded_step_inputs(net)
    say("case deterministic mode", which)

    def run(ls):
        ls.set_lams(lams)
        ls.local_step(net.rho, 1.0, mult_step=net.step)
        torch.cuda.synchronize()
        out = {f"y{k}": ls.y[k].clone() for k in range(net.K - 1)}
        out.update({f"dy{k}": ls.dy[k].clone() for k in range(net.K - 1)})
        out.update({f"dx{k}": ls.dx[k].clone() for k in range(1, net.K)})
        out.update({f"lam{k}": ls.lam[k].clone() for k in range(net.K - 1)})
        out.update({f"dparams{k}": ls.dparams[k].clone() for k in range(net.K)})
        out["logits"], out["dlogits"] = ls.logits.clone(), ls.dlogits.clone()
        return out

    ls = LocalStep(net)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_labels(labels)
        ref = run(ls)                                    # default mode
        B.lp_net_set_deterministic(ls.net, 1)
        a = run(ls)
        ls.ws.zero_()                                    # nothing may depend on what an earlier run left behind
        b = run(ls)
        B.lp_net_set_deterministic(ls.net, 0)
    finally:
        ls.close()
    for name in a:
        assert torch.equal(a[name], b[name]), f"{name} differs between two deterministic runs"
    tol = 1e-4 if net.dtype == "f32" else 2e-2
    worst = {name: rel_err(a[name].float().cpu().numpy(), ref[name].float().cpu().numpy()) for name in a}
    say("    deterministic vs default mode, worst: " + ", ".join(f"{k}={v:.1e}" for k, v in sorted(worst.items(), key=lambda kv: -kv[1])[:4]))
    # fp32: everything agrees; bf16: what lies in front of the backward pass does (the backward pass of a deep bf16
    # network amplifies last-bit differences of the statistics through flipped roundings, as between any two valid runs)
    judged = {k: v for k, v in worst.items() if net.dtype == "f32" or k.startswith(("y", "logits", "dlogits", "dy", "lam"))}
    assert all(v <= tol for v in judged.values()), judged


ADDRESS_CASES = [
    # kernel, mode, (N, H, W, Cin, Cout, R, stride, pad), bk
    (0, 0, (3, 9, 7, 8, 16, 3, 1, 1), 32), (0, 0, (2, 10, 8, 8, 8, 3, 2, 1), 32), (0, 0, (2, 20, 16, 3, 8, 7, 2, 3), 32),
    (0, 1, (2, 9, 7, 8, 16, 3, 1, 1), 32), (0, 1, (2, 10, 8, 8, 16, 3, 2, 1), 32), (0, 1, (2, 8, 8, 16, 8, 1, 2, 0), 32),
    (1, 0, (4, 32, 32, 160, 160, 3, 1, 1), 32), (1, 0, (4, 16, 16, 320, 320, 3, 1, 1), 64), (1, 0, (4, 32, 32, 160, 320, 3, 2, 1), 32),
    (1, 0, (4, 32, 32, 160, 320, 1, 2, 0), 32), (1, 1, (4, 16, 16, 320, 320, 3, 1, 1), 64), (1, 1, (4, 32, 32, 160, 320, 3, 2, 1), 64),
    (1, 1, (4, 16, 16, 320, 640, 1, 2, 0), 64), (1, 0, (3, 6, 10, 160, 296, 3, 1, 1), 32),
    (2, 0, (4, 32, 32, 160, 160, 3, 1, 1), 64), (2, 1, (4, 32, 32, 160, 160, 3, 1, 1), 64), (2, 0, (8, 16, 16, 320, 320, 3, 1, 1), 64),
    (2, 1, (8, 16, 16, 320, 320, 3, 1, 1), 64), (2, 0, (16, 8, 8, 640, 640, 3, 1, 1), 64), (2, 1, (16, 8, 8, 640, 640, 3, 1, 1), 64),
    (2, 0, (4, 32, 32, 160, 320, 3, 1, 1), 64), (2, 1, (4, 32, 32, 320, 160, 3, 1, 1), 64),
    (2, 0, (4, 32, 32, 32, 160, 3, 1, 1), 64),      # one (half) slab of 32 channels
]


@pytest.mark.parametrize("kernel,mode,shape,bk", ADDRESS_CASES)
def test_conv_addresses_bit_exact(kernel, mode, shape, bk):
    """The integer work of the convolution kernels that run (general, wide-layer implicit GEMM, window): for sampled
    GEMM elements the activation offset, the filter offset and the output offset that the kernels' own address
    functions produce on the device -- lane / chunk swizzles of the direct-to-LDS loads resolved -- equal, bit for bit,
    what the oracle's index function of the convolution's definition gives.  Forward: directly.  Data-gradient (all
    parity classes of a strided layer): dX[n,hi,wi,ci] takes dY[n,ho,wo,co] * W[co,r,s,ci] exactly for the (ho,wo)
    whose forward window reads (hi,wi) at tap (r,s) -- found by brute force with the same index function."""
    import torch
    from paper_2112_05387_amd import binding as B
    N, H, W, Cin, Cout, R, stride, pad = shape
    Ho, Wo = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    n_samples = 1500 if mode == 0 else 400
    for parity in range(1 if mode == 0 else stride * stride):
        g = B.lp_debug_conv_geometry(kernel, mode, parity, N, H, W, Cin, Cout, R, stride, pad, bk)
        if g["ntr"] == 0:
            continue
        say(f"case addresses kernel {kernel} {'dgrad' if mode else 'fwd'} {shape} parity {parity}: M={g['M']} taps {g['ntr']}x{g['nts']} BM={g['BM']}")
        ms = wl.uniform_int(5, f"addr_m{parity}", (n_samples,), g["M"]).astype(np.int64)
        qs = wl.uniform_int(5, f"addr_q{parity}", (n_samples,), g["ntr"] * g["nts"] * g["C"]).astype(np.int64)
        cols = wl.uniform_int(5, f"addr_c{parity}", (n_samples,), g["Ncol"]).astype(np.int64)
        # corners: first / last rows and columns of the GEMM, first / last tap and channel
        ms[:4] = [0, g["M"] - 1, 0, g["M"] - 1]
        qs[:4] = [0, g["ntr"] * g["nts"] * g["C"] - 1, g["ntr"] * g["nts"] * g["C"] - 1, 0]
        cols[:4] = [0, g["Ncol"] - 1, 0, g["Ncol"] - 1]
        t = lambda a: torch.from_numpy(a).to(dev)
        dm, dq, dc = t(ms), t(qs), t(cols)
        outs = [torch.empty(n_samples, dtype=torch.int64, device=dev) for _ in range(3)]
        B.lp_debug_conv_offsets(stream, kernel, mode, parity, N, H, W, Cin, Cout, R, stride, pad, bk, dm.data_ptr(), dq.data_ptr(),
                                dc.data_ptr(), outs[0].data_ptr(), outs[1].data_ptr(), outs[2].data_ptr(), n_samples)
        torch.cuda.synchronize()
        in_off, w_off, out_off = (o.cpu().numpy() for o in outs)
        want_in, want_w, want_out = np.empty_like(in_off), np.empty_like(w_off), np.empty_like(out_off)
        for i in range(n_samples):
            m, q, col = int(ms[i]), int(qs[i]), int(cols[i])
            tap, c = divmod(q, g["C"])
            tr, ts = divmod(tap, g["nts"])
            r, s = g["r0"] + g["rs"] * tr, g["s0"] + g["ss"] * ts           # the filter tap the kernel multiplies with
            if mode == 0:
                assert (r, s) == (tr, ts)
                want_in[i] = lpref.im2col_index(m, (r * R + s) * Cin + c, H, W, Cin, R, R, stride, pad)
                want_w[i] = (col * R * R + r * R + s) * Cin + c             # W[co=col][r][s][ci=c]
                want_out[i] = m * Cout
            else:
                # output pixel of this GEMM row: from the device's own output offset (dX is [N,H,W,Cin], column = ci)
                pix = int(out_off[i]) // Cin
                assert int(out_off[i]) % Cin == 0
                n, rem = divmod(pix, H * W)
                hi, wi = divmod(rem, W)
                assert (hi % stride, wi % stride) == divmod(parity, stride)
                want_out[i] = out_off[i]
                want_w[i] = ((col * R + r) * R + s) * Cout + c              # re-laid-out filter [ci=col][r][s][co=c]
                target = ((n * H + hi) * W + wi) * Cin + col
                hit = [(ho, wo) for ho in range(Ho) for wo in range(Wo)
                       if lpref.im2col_index((n * Ho + ho) * Wo + wo, (r * R + s) * Cin + col, H, W, Cin, R, R, stride, pad) == target]
                assert len(hit) <= 1
                want_in[i] = ((n * Ho + hit[0][0]) * Wo + hit[0][1]) * Cout + c if hit else -1
        np.testing.assert_array_equal(in_off, want_in)
        np.testing.assert_array_equal(w_off, want_w)
        np.testing.assert_array_equal(out_off, want_out)
        assert mode == 1 or pad == 0 or (want_in < 0).any(), "the sample never touched the padding"


def _read_params(ls, k):
    """Stored parameters of module k as float64 arrays (bf16 tensors widened exactly)."""
    import torch
    from paper_2112_05387_amd import binding as B
    out = []
    for info in ls.tables[k]:
        n = int(info.numel)
        shape = tuple(info.dims[i] for i in range(info.ndim))
        if info.dtype == B.LP_BF16:
            t = ls.params[k][info.offset:info.offset + 2 * n].view(torch.bfloat16)
        else:
            t = ls.params[k][info.offset:info.offset + 4 * n].view(torch.float32)
        out.append(ls.to_host(t).reshape(shape).astype(np.float64))
    return out


def _read_like_grads(ls, buf, k):
    return [ls.to_host(buf[k][info.grad_offset // 4:info.grad_offset // 4 + int(info.numel)])
            .reshape(tuple(info.dims[i] for i in range(info.ndim))).astype(np.float64) for info in ls.tables[k]]


@pytest.mark.parametrize("case,momentum,wd,use_master,fused_call", [
    ("basic_f32", 0.9, 5e-4, False, True), ("basic_bf16", 0.9, 5e-4, True, True), ("basic_bf16", 0.0, 0.0, False, False),
    ("bottleneck_bf16", 0.9, 0.0, False, True), ("wide", 0.9, 5e-4, True, True), ("wide", 0.5, 0.0, False, False),
    ("wide_strided", 0.9, 5e-4, False, True), ("wrn_batch_8", 0.9, 5e-4, True, True),
    # the folded passes of narrow networks; "flags": a bare projection, whose filter gradient runs in the middle of the pass
    ("narrow_f32", 0.9, 5e-4, False, True), ("narrow_bf16", 0.9, 5e-4, True, True), ("narrow_f32", 0.0, 0.0, False, False),
    ("narrow_flags_f32", 0.9, 0.0, False, False), ("narrow_flags_bf16", 0.9, 5e-4, True, True)])
def test_update_inside_backward(case, momentum, wd, use_master, fused_call):
    """The parameter update in the epilogues of the filter-gradient kernels (Sec. 4.1: W is updated right after the
    adjoint at its layer): two local steps in a row with the update switched on.  After each step the oracle's update
    rule, fed the parameters / velocity the device held before the step and the gradients the device wrote in that
    step, gives the expected parameters, velocity and master copy of EVERY tensor (filters: updated by the workgroup
    that completed a gradient tile; BN affine and head: by the small grouped launch behind the module)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_common import gpu_mini_wide_strided
    from tests.gpu_unitwise import seeded_step_inputs
    from tests.test_gpu_narrow import FOLDED, narrow_net
    net = {"basic_f32": lambda: gpu_mini_basic(batch=3, dtype="f32"), "basic_bf16": lambda: gpu_mini_basic(batch=3, dtype="bf16"),
           "bottleneck_bf16": lambda: gpu_mini_bottleneck(batch=2, dtype="bf16"), "wide": lambda: gpu_mini_wide(batch=3),
           "wide_strided": lambda: gpu_mini_wide_strided(batch=5), "wrn_batch_8": lambda: wl.make_config("wrn28_10", batch=8),
           "narrow_f32": lambda: narrow_net(3, (12, 20)), "narrow_bf16": lambda: narrow_net(33, (32, 32), dtype="bf16"),
           "narrow_flags_f32": lambda: narrow_net(3, (16, 16), flags=True),
           "narrow_flags_bf16": lambda: narrow_net(5, (16, 16), dtype="bf16", flags=True)}[case]()
    lr = 1.0        # large on purpose: every tensor's update must stand far above the comparison tolerance
    say("case update inside backward", case, momentum, wd, "master" if use_master else "", "one call" if fused_call else "separate calls")
    params, image, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        vel = [torch.zeros_like(d) for d in ls.dparams] if momentum else None
        master = None
        if use_master:
            master = [torch.zeros_like(d) for d in ls.dparams]
            for k in range(net.K):
                for info, w in zip(ls.tables[k], params[k]):
                    o = info.grad_offset // 4
                    master[k][o:o + int(info.numel)].copy_(torch.from_numpy(np.asarray(w, np.float32).reshape(-1)))
        ls.set_fused_update(True, lr, momentum, wd, velocity=vel, master=master)
        worst = {"param": 0.0, "velocity": 0.0, "master": 0.0}
        smallest = 1e30
        if case.startswith("narrow"):
            B.lp_profile_enable(ls.net, 1)
        for it in range(2):
            before_w = [(_read_like_grads(ls, master, k) if use_master else _read_params(ls, k)) for k in range(net.K)]
            before_v = [(_read_like_grads(ls, vel, k) if momentum else None) for k in range(net.K)]
            if fused_call:
                ls.local_step(net.rho, 1.0)
            else:
                ls.module_forward()
                ls.local_loss_grad(net.rho, 1.0)
                ls.module_backward()
            torch.cuda.synchronize()
            for k in range(net.K):
                grads = ls.get_grads(k)
                after_w = _read_params(ls, k)
                after_v = _read_like_grads(ls, vel, k) if momentum else None
                after_m = _read_like_grads(ls, master, k) if use_master else None
                for i, info in enumerate(ls.tables[k]):
                    w_new, v_new = lpref.sgd_update(before_w[k][i], grads[i].astype(np.float64), lr,
                                                    before_v[k][i] if momentum else None, momentum, wd)
                    tol = 4e-3 if info.dtype == B.LP_BF16 else 1e-6        # bf16 parameters: one rounding of the stored value
                    e = rel_err(after_w[i], w_new)
                    assert e <= tol, (case, it, k, i, "parameter", e)
                    worst["param"] = max(worst["param"], e)
                    # the step must be large against the tolerance, or a missing update would pass
                    step_size = float(np.max(np.abs(w_new - before_w[k][i])) / np.max(np.abs(w_new)))
                    assert step_size >= 5 * tol, (case, it, k, i, "update too small for the check to mean anything", step_size)
                    smallest = min(smallest, step_size)
                    if momentum:
                        e = rel_err(after_v[i], v_new)
                        assert e <= 1e-6, (case, it, k, i, "velocity", e)
                        worst["velocity"] = max(worst["velocity"], e)
                    if use_master:
                        e = rel_err(after_m[i], w_new)
                        assert e <= 1e-6, (case, it, k, i, "master", e)
                        worst["master"] = max(worst["master"], e)
        say(f"    update inside backward, {case}: worst parameter {worst['param']:.2e}, velocity {worst['velocity']:.2e}, master {worst['master']:.2e}; "
            f"smallest update of a tensor {smallest:.1e} of its magnitude")
        assert not case.startswith("narrow") or FOLDED in {r["kind"] for r in B.lp_profile_fetch(ls.net)}
    finally:
        ls.close()


def test_update_inside_backward_deterministic_bit_identical():
    """In the deterministic mode (unsplit filter gradients) the update inside the backward pass equals the step followed
    by lp_sgd_update bit for bit: parameters, velocity and master copy."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    net = gpu_mini_wide(batch=3)
    lr, momentum, wd = 0.05, 0.9, 5e-4
    params, image, labels, xs, lams = seeded_step_inputs(net)
    res = []
    for inside in (False, True):
        ls = LocalStep(net)
        try:
            B.lp_net_set_deterministic(ls.net, 1)
            for k in range(net.K):
                ls.set_params(k, params[k])
                ls.set_x(k, xs[k])
            ls.set_lams(lams)
            ls.set_labels(labels)
            vel = [torch.zeros_like(d) for d in ls.dparams]
            master = [torch.zeros_like(d) for d in ls.dparams]
            for k in range(net.K):
                for info, w in zip(ls.tables[k], params[k]):
                    o = info.grad_offset // 4
                    master[k][o:o + int(info.numel)].copy_(torch.from_numpy(np.asarray(w, np.float32).reshape(-1)))
            if inside:
                ls.set_fused_update(True, lr, momentum, wd, velocity=vel, master=master)
            for it in range(2):
                ls.local_step(net.rho, 1.0)
                if not inside:
                    ls.sgd_update(lr, momentum, wd, velocity=vel, master=master)
            torch.cuda.synchronize()
            res.append(([p.cpu().clone() for p in ls.params], [v.cpu().clone() for v in vel], [m.cpu().clone() for m in master]))
        finally:
            ls.close()
    for name, a, b in zip(("parameters", "velocity", "master"), res[0], res[1]):
        for k in range(net.K):
            assert torch.equal(a[k], b[k]), (name, k)
    say("    update inside backward, deterministic mode: bit-identical to step + lp_sgd_update over two steps")
