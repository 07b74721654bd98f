"""The work a training program has this library do, as cases that can be timed and compared.

A case is one pass of a training program over a mini-batch that is already in device memory, through
`paper_2112_05387_amd.LocalStep`:

  step       [AuxNet forward if the workload has AuxNets,] the local step of all K modules in one call
  separate   the same through the single entry points (forward, loss / terminal adjoint, backward, multiplier update)
  iteration  one iteration of the method: AuxNet forward, local step, correction of the auxiliary variables, distillation
             gradient of the AuxNets, parameter update of modules and AuxNets (momentum, weight decay, fp32 master copy)
  forward    the modules' forward pass alone

The networks are those of `workloads/`, over mini-batches from one sample to the configuration's own (or the largest this
card is used with), both storage types, both block orders and several splits into modules.
"""
import math

import torch

import workloads as wl
from workloads import configs as cfg
from paper_2112_05387_amd import LocalStep
from paper_2112_05387_amd import binding as B

LR, MOMENTUM, WEIGHT_DECAY = 1e-6, 0.9, 5e-4       # a learning rate of the warm-up phase

#: Residual blocks per module of the splits in use: the configuration's own K first.  One module is ordinary
#: (layer-serial) back-propagation, the yardstick of the method's speed-up.
SPLITS = {"tiny": ["1,1", "2"],
          "resnet20": ["3,2,2,2", "5,4", "3,3,3", "9"],
          "resnet56": ["4,4,4,3,3,3,3,3", "7,7,7,6"],
          "wrn28_10": ["3,3,3,3", "6,6", "4,4,4"],
          "resnet50": ["3,4,6,3"]}
#: Mini-batches: the configuration's own is the largest, apart from the CIFAR-sized narrow networks, whose mini-batch fits twice.
BATCHES = {"tiny": (1, 64), "resnet20": (1, 256), "resnet56": (1, 256), "wrn28_10": (1, 128), "resnet50": (1, 64)}


def _case(name, net, batch, split=0, dtype=None, order="post", what="step"):
    dtype = dtype or wl.make_config(net, batch=1).dtype
    return {"name": name, "net": net, "batch": batch, "split": SPLITS[net][split], "dtype": dtype, "order": order, "pass": what}


def listed():
    return [
        # the smallest call anybody makes: two 16-channel blocks on 8x8 images, four samples; launches and host work
        _case("tiny", "tiny", 4),
        # CIFAR-10 with the small network in full precision, penalty method: the paper's AuxNet-sized backbone
        _case("resnet20", "resnet20", 128),
        # ... the last, short mini-batch of an epoch (50000 = 390*128 + 80), through the single entry points
        _case("resnet20_last_batch", "resnet20", 80, what="separate"),
        # ... one sample more than nothing: on-line use, debugging, per-device shards of a small mini-batch
        _case("resnet20_batch_3_bf16", "resnet20", 3, dtype="bf16"),
        # ... the layer-serial yardstick (one module): ordinary back-propagation through the same kernels
        _case("resnet20_serial", "resnet20", 128, split=3),
        # the deep narrow network, eight modules, augmented Lagrangian, AuxNets: local step as the method runs it
        _case("resnet56", "resnet56", 128),
        # ... and a whole training iteration of it
        _case("resnet56_iteration", "resnet56", 128, what="iteration"),
        # the headline workload: wide network, matrix-core bound
        _case("wrn28_10", "wrn28_10", 128),
        # ... its forward pass on an odd mini-batch (evaluation, statistics, line search on the auxiliary variables)
        _case("wrn28_10_forward", "wrn28_10", 75, what="forward"),
        # ... the pre-activation block order (the paper's figure), a quarter of the mini-batch
        _case("wrn28_10_pre", "wrn28_10", 32, order="pre"),
        # ImageNet-sized images, bottleneck blocks, bandwidth bound: the largest call
        _case("resnet50", "resnet50", 64),
        # ... and a small shard of it
        _case("resnet50_batch_6", "resnet50", 6),
    ]


def draw(rng):
    net = rng.choice(["tiny", "resnet20", "resnet20", "resnet56", "resnet56", "wrn28_10", "wrn28_10", "resnet50"])
    lo, hi = BATCHES[net]
    batch = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    split = rng.randrange(len(SPLITS[net]))
    # storage: the wide networks are trained in bf16 only, the narrow ones in either
    dtype = "bf16" if net in ("wrn28_10", "resnet50") else rng.choice(["f32", "bf16"])
    order = "pre" if net != "resnet50" and rng.random() < 0.25 else "post"
    what = rng.choice(["step", "step", "separate", "iteration", "forward"])
    if what == "iteration" and ("," not in SPLITS[net][split] or net == "tiny"):
        what = "step"                                  # one module has no auxiliary variables
    if what == "iteration":
        batch = max(1, batch * 3 // 4)                 # an iteration does more: stay below the largest listed case
    c = _case("", net, batch, split=split, dtype=dtype, order=order, what=what)
    del c["name"]
    return c


def _net(case):
    net = wl.make_config(case["net"], batch=case["batch"], split=[int(n) for n in case["split"].split(",")])
    net.dtype = case["dtype"]
    cfg.with_order(net, case["order"])
    if case["pass"] == "iteration" and net.aux is None:
        m0 = net.modules[0]
        net.aux = [cfg.AuxDesc(cin=m0.C, cout=m.C, stride=m0.H // m.H, relu=False) for m in net.modules[1:]]
    if net.K == 1:
        net.aux = None
    return net


class _State:
    """What the program holds: the library's object, its multipliers, and the optimiser's buffers."""

    def __init__(self, case, seed):
        self.what = case["pass"]
        self.net = net = _net(case)
        self.ls = ls = LocalStep(net)
        dev, K = ls.dev, net.K
        g = torch.Generator(device=dev)
        g.manual_seed(seed)

        def normal(shape, sigma=1.0, mean=0.0):
            return torch.randn(shape, generator=g, device=dev) * sigma + mean

        # Kaiming-normal filters, BN gamma = 1 + N(0, 0.1^2), beta and bias N(0, 0.1^2)
        def fill(buf, table, specs):
            for info, sp in zip(table, specs):
                n = int(info.numel)
                v = normal(n, math.sqrt(2.0 / sp.fan_in)) if sp.kind in ("conv", "fc_w") else normal(n, 0.1, 1.0 if sp.kind == "bn_gamma" else 0.0)
                size, dt = (2, torch.bfloat16) if info.dtype == B.LP_BF16 else (4, torch.float32)
                buf[info.offset:info.offset + size * n].view(dt).copy_(v)

        for k in range(K):
            fill(ls.params[k], ls.tables[k], cfg.module_tensor_specs(net.modules[k]))
        for j in range(len(ls.aux_tables)):
            fill(ls.aux_params[j], ls.aux_tables[j], cfg.aux_tensor_specs(net.aux[j]))
        # the image is white noise; an auxiliary variable is as large as a residual stream that many blocks in (every block adds
        # a normalised tensor); it is overwritten where the pass generates it with AuxNets
        blocks = 0
        for k in range(K):
            ls.x[k].copy_(normal(ls.x_shapes[k], math.sqrt(1.0 + blocks)))
            blocks += len(net.modules[k].blocks)
        ls.labels.copy_(torch.randint(0, ls.n_classes, (ls.N,), generator=g, device=dev, dtype=torch.int32))
        self.al = net.al and K > 1
        if self.al:
            ls.lam = [normal(s, net.lam_sigma).to(ls.tdtype) for s in ls.y_shapes]
        if self.what == "iteration":
            # penalty as a mean over the elements of the first interface tensor
            self.scale = 1.0 / ls.x[1].numel()
            flat = lambda ts: (lambda t: (t, list(t.split([u.numel() for u in ts]))))(torch.zeros(sum(u.numel() for u in ts), device=dev))  # noqa: E731
            self.vel_all, self.vel = flat(ls.dparams)
            self.aux_vel_all, self.aux_vel = flat(ls.daux_params)
            self.master_all, self.master = None, None
            if net.dtype == "bf16":                    # fp32 master copy of the parameters, laid out like the gradients
                self.master_all, self.master = flat(ls.dparams)
                for k in range(K):
                    for info in ls.tables[k]:
                        n, o = int(info.numel), info.grad_offset // 4
                        size, dt = (2, torch.bfloat16) if info.dtype == B.LP_BF16 else (4, torch.float32)
                        self.master[k][o:o + n].copy_(ls.params[k][info.offset:info.offset + size * n].view(dt))

    def __del__(self):
        if getattr(self, "ls", None) is not None:
            self.ls.close()


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    ls, net = s.ls, s.net
    K = net.K
    mult = net.step if s.al else None
    if s.what == "forward":
        ls.module_forward()
        return {"y": ls.y, "logits": ls.logits}
    out = {"y": ls.y, "logits": ls.logits, "loss": ls.loss, "dparams": ls.dparams, "dx": ls.dx[1:]}
    if s.al:
        out["lam"] = ls.lam
    if net.aux is not None:
        out["x"] = ls.x[1:]
    if s.what == "step":
        ls.step(net.rho, 1.0, mult_step=mult, with_aux=net.aux is not None)
    elif s.what == "separate":
        if net.aux is not None:
            ls.auxnet_forward()
        ls.module_forward()
        ls.local_loss_grad(net.rho, 1.0)
        ls.module_backward()
        if s.al:
            ls.al_multiplier_update(net.step)
    else:
        ls.auxnet_forward()
        ls.local_step(net.rho, s.scale, net.step if s.al else 0.0)
        ls.aux_variable_update(net.rho, s.scale, 0.1)
        ls.auxnet_distill_grad(s.scale)
        ls.sgd_update(LR, MOMENTUM, WEIGHT_DECAY, velocity=s.vel, master=s.master)
        ls.sgd_update_aux(LR, MOMENTUM, WEIGHT_DECAY, velocity=s.aux_vel)
        out.update(daux=ls.daux_params, aux_loss=ls.aux_loss, vel=s.vel_all, aux_vel=s.aux_vel_all)
        out["params"] = s.master_all if s.master_all is not None else [p.view(torch.float32) for p in ls.params]
    if K > 1:
        out["r2"] = ls.r2
    return out


def work(case):
    """Inputs read once and outputs written once; the convolutions' multiply-adds (and, for AuxNets, theirs)."""
    net = _net(case)
    e = 2 if net.dtype == "bf16" else 4
    elems = [m.N * m.H * m.W * m.C for m in net.modules]
    inter = sum(elems[1:])                             # elements of the interface tensors
    pw = sum(math.prod(sp.shape) for m in net.modules for sp in cfg.module_tensor_specs(m))
    fwd_b = sum(elems) * e + pw * e + inter * e        # x_k, parameters; y
    fwd_f = cfg.conv_flops_forward(net)
    if case["pass"] == "forward":
        return {"bytes": fwd_b, "flops": fwd_f}
    nbytes = fwd_b + inter * e + pw * 4                # dx; parameter gradients
    flops = cfg.conv_flops_step(net)
    if net.al and net.K > 1:
        nbytes += 2 * inter * e                        # multipliers read and written
    if net.aux is not None:
        aux_f = sum(2.0 * m.N * m.H * m.W * m.C * 9 * a.cin for a, m in zip(net.aux, net.modules[1:]))
        aw = sum(math.prod(sp.shape) for a in net.aux for sp in cfg.aux_tensor_specs(a))
        flops += aux_f
        nbytes += aw * e
        if case["pass"] == "iteration":
            flops += aux_f                             # filter gradient of the distillation
            nbytes += inter * e + aw * 4               # x_k corrected; AuxNet gradients
            nbytes += (pw + aw) * 16 + (pw * 8 if net.dtype == "bf16" else 0)      # parameters, velocities, master copy
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16 storage: one rounding of a stored value is 2^-9 relative, and the tensors of a module pass through some ten of
    them.  Where two correct runs round a value near zero to different sides, a ReLU lets a gradient element pass in
    one of them only: at the depth of these modules that is worth up to a few percent of a gradient's norm and, for
    single elements, their whole size.  fp32: the same decisions are taken on values that agree to 1e-7, and one element
    that decides differently moves the gradient of a module's input by 2e-3 of its norm (measured with another order of
    the sums of the batch statistics)."""
    if case["dtype"] == "bf16":
        return {"rel": 0.03, "max": 0.99}
    return {"rel": 4e-3, "max": 0.99}
