"""The work whose speed is measured: what a program that trains or deploys a quantized visual-odometry
front end has this library do, through its public entry points.

Every case is a dict of plain values.  `kind` says what the program does in one pass:

  layer     one tensor: fq_forward, then fq_backward (an activation, or the weights of a convolution)
  codes     one tensor: fq_forward that writes the packed int8 codes and the scales (deployment)
  list      a list of mixed tensors: forward and backward in one launch each, by a prepared plan or by
            fq_multi_tensor (a program whose tensors move between the passes)
  weights   the weights of all convolutions of the front end, frozen: forward plan, then the backward plan
            with the fused Adam step on the scales
  frame     the activations of all convolutions of the front end, one call per layer as they come up in a
            training step, forward and backward, captured in a HIP graph once and replayed
  autograd  fake_quantize() under torch.autograd, forward and gradients
  distill   the distillation loss of a pair of feature maps, with or without its gradient

Inputs are synthetic, made on the GPU from the seed, with the distributions of
paper_2511_12653_amd/workloads.py: activations with a mean and a spread per channel (or standard normal
with one value in a hundred ten times as large, for a single scale), weights of variance 2 / fan-in,
scales from the spread or the largest magnitude, so that a few elements clip.
"""
import math
import random

import torch

from paper_2511_12653_amd import binding as fq
from paper_2511_12653_amd.autograd import fake_quantize

# The 22 convolutions of the front end: two ResNet-like encoders of 11, which differ in their last
# output width: (in channels, out channels, kernel, resolution of the input: image / this).
_ENCODER = [(3, 32, 7, 1)] + [(32, 32, 3, 2)] * 4 + [(32, 64, 3, 2), (32, 64, 1, 2)] + [(64, 64, 3, 4)] * 3
FRONT_END = _ENCODER + [(64, 128, 1, 4)] + _ENCODER + [(64, 384, 1, 4)]

ADAM = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8)
LOSS_SCALE = 65536.0          # keeps an FP16 distillation gradient out of the subnormal range
LAMBDA = 0.5


def listed():
    return [
        # the smallest call: a 30x40 FP32 map with one scale; launches and latency
        dict(name="act_fp32_per_tensor", kind="layer", dtype="fp32", n=1, c=128, h=30, w=40, scales="tensor",
             values="act", gx=True),
        # the benchmark's tensor: one frame's feature map, a scale per channel
        dict(name="feature_fp16", kind="layer", dtype="fp16", n=1, c=384, h=120, w=160, scales="channel",
             values="act", gx=True),
        # a training batch of fifteen frames
        dict(name="train_batch_fp16", kind="layer", dtype="fp16", n=15, c=128, h=120, w=160, scales="channel",
             values="act", gx=True),
        # a crop whose rows are no whole number of vectors: most slabs start off the 16-byte grid
        dict(name="ragged_fp16", kind="layer", dtype="fp16", n=3, c=131, h=61, w=79, scales="channel",
             values="act", gx=True),
        # PyTorch's front door: a batch of activations with one scale each
        dict(name="autograd_fp16", kind="autograd", dtype="fp16", n=8, c=64, h=120, w=160, scales="channel",
             values="act", gx=True),
        # deployment: integer codes of a batch of feature maps
        dict(name="codes_fp16", kind="codes", dtype="fp16", n=4, c=128, h=120, w=160, scales="channel",
             values="act"),
        # scale-only training of the frozen weights, all layers at once
        dict(name="weights_adam_fp32", kind="weights", dtype="fp32", width=1),
        # the benchmark's list: 64 mixed tensors, about 1 GiB of x
        dict(name="list_mixed", kind="list", tensors=64, elements=347000000, mix=5, call="plan"),
        # one QAT step's activations of a 480x640 frame, layer by layer
        dict(name="frame_fp16", kind="frame", dtype="fp16", n=1, h=480, w=640),
        # the loss between two feature maps of one frame, and of a batch
        dict(name="distill_feature_fp16", kind="distill", dtype="fp16", n=1, c=384, h=120, w=160, grad=True),
        dict(name="distill_batch_fp16", kind="distill", dtype="fp16", n=15, c=128, h=120, w=160, grad=True),
        # the same in FP32 on a crop with an odd number of positions
        dict(name="distill_ragged_fp32", kind="distill", dtype="fp32", n=2, c=128, h=61, w=79, grad=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _map(rng, most):
    """An activation's extents: odd ones among them, at most `most` elements."""
    c, h, w = _log(rng, 16, 512), _log(rng, 15, 240), _log(rng, 20, 320)
    n = _log(rng, 1, 16)
    while n > 1 and n * c * h * w > most:
        n -= 1
    while c * h * w > most:
        h, w = max(1, h // 2), max(1, w // 2)
    return dict(n=n, c=c, h=h, w=w)


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "weight", "autograd", "codes", "weights", "list", "frame",
                       "distill", "distill"])
    dtype = rng.choice(["fp16", "fp32"])
    scales = rng.choice(["channel", "channel", "tensor"])
    if kind == "weight":      # one convolution's weights: kernel 1, 3 or 7
        k = rng.choice([1, 3, 3, 7])
        return dict(kind="layer", dtype=dtype, n=1, c=_log(rng, 16, 512), h=_log(rng, 16, 512), w=k * k,
                    scales="channel", values="weights", gx=rng.choice([True, False]))
    if kind == "layer":
        return dict(kind="layer", dtype=dtype, scales=scales, values="act", gx=True, **_map(rng, 60000000))
    if kind == "autograd":
        return dict(kind="autograd", dtype=dtype, scales=scales, values="act", gx=True, **_map(rng, 60000000))
    if kind == "codes":
        return dict(kind="codes", dtype=dtype, scales=scales, values="act", **_map(rng, 60000000))
    if kind == "weights":
        return dict(kind="weights", dtype=dtype, width=rng.randint(1, 4))
    if kind == "list":
        return dict(kind="list", tensors=_log(rng, 4, 64), elements=_log(rng, 1000000, 200000000),
                    mix=rng.randint(6, 1 << 20), call=rng.choice(["plan", "multi"]))
    if kind == "frame":
        return dict(kind="frame", dtype=dtype, n=rng.randint(1, 3), h=4 * _log(rng, 30, 130),
                    w=4 * _log(rng, 40, 190))
    return dict(kind="distill", dtype=dtype, grad=rng.random() < 0.8, **_map(rng, 60000000))


# ------------------------------------------------------------------------------------------- tensors
def _spec(outer, channels, inner, dtype, values, qmin=-127, qmax=127):
    return dict(outer=outer, channels=channels, inner=inner, dtype=dtype, values=values, qmin=qmin, qmax=qmax)


def _activation(n, c, hw, dtype, scales, qmin=-128, qmax=127):
    if scales == "tensor":
        return _spec(1, 1, n * c * hw, dtype, "act", qmin, qmax)
    return _spec(n, c, hw, dtype, "act", qmin, qmax)


def _specs(case):
    """The tensors of a case, as [outer, channels, inner] views."""
    kind = case["kind"]
    if kind in ("layer", "codes", "autograd"):
        if case["values"] == "weights":
            return [_spec(case["n"], case["c"], case["h"] * case["w"], case["dtype"], "weights")]
        return [_activation(case["n"], case["c"], case["h"] * case["w"], case["dtype"], case["scales"])]
    if kind == "weights":
        m = case["width"]
        return [_spec(1, co * m, (ci if ci == 3 else ci * m) * k * k, case["dtype"], "weights")
                for ci, co, k, _ in FRONT_END]
    if kind == "frame":
        return [_activation(case["n"], ci, (case["h"] // div) * (case["w"] // div), case["dtype"], "tensor")
                for ci, _, _, div in FRONT_END]
    # list: three activations to one weight tensor; dtypes, bit widths and kinds of scale mixed
    rng = random.Random(case["mix"])
    acts = []
    for i in range(case["tensors"]):
        dtype = rng.choice(["fp16", "fp32"])
        qmin, qmax = rng.choice([(-8, 7), (-128, 127)])
        scales = rng.choice(["channel", "tensor"])
        if i % 4 == 3:
            co, ci = rng.choice([64, 128, 384]), rng.choice([64, 128, 384])
            acts.append(_spec(1, co if scales == "channel" else 1, ci * 9 * (1 if scales == "channel" else co),
                              dtype, "weights", qmin, qmax))
        else:
            acts.append(_activation(rng.randint(1, 8), rng.choice([64, 128, 384]),
                                    rng.randint(30, 120) * rng.randint(40, 160), dtype, scales, qmin, qmax))
    # as many frames per activation as the wanted number of elements gives
    total = sum(s["outer"] * s["channels"] * s["inner"] for s in acts)
    ratio = case["elements"] / total
    for s in acts:
        if s["values"] == "act":
            if s["channels"] > 1 and ratio >= 1:
                s["outer"] = max(1, round(s["outer"] * ratio))
            else:
                s["inner"] = max(1, round(s["inner"] * ratio))
    return acts


def _numel(s):
    return s["outer"] * s["channels"] * s["inner"]


def _torch(dtype):
    return torch.float16 if dtype == "fp16" else torch.float32


def _values(spec, gen):
    """x and theta of a tensor."""
    o, c, k = spec["outer"], spec["channels"], spec["inner"]
    dev = gen.device
    x = torch.randn((o, c, k), generator=gen, device=dev, dtype=torch.float32)
    if spec["values"] == "weights":
        fan_in = max(1, k if c > 1 else 576)
        x *= math.sqrt(2.0 / fan_in)
        s = x.abs().amax(dim=(0, 2)).clamp_min(1e-6).double() / spec["qmax"]
    elif c == 1:
        big = torch.rand((o, c, k), generator=gen, device=dev) < 0.01
        x = torch.where(big, x * 10.0, x)
        s = torch.full((1,), 6.0 / spec["qmax"], dtype=torch.float64, device=dev)
    else:
        mu = torch.rand((c,), generator=gen, device=dev) * 2.0 - 1.0
        sigma = torch.rand((c,), generator=gen, device=dev) * 2.8 + 0.2
        x.mul_(sigma[None, :, None]).add_(mu[None, :, None])
        s = (mu.abs() + 3.0 * sigma).double() / spec["qmax"]
    return x.to(_torch(spec["dtype"])), torch.log(torch.expm1(s)).float()


def _upstream(spec, gen):
    gy = torch.randn((spec["outer"], spec["channels"], spec["inner"]), generator=gen, device=gen.device,
                     dtype=torch.float32)
    if spec["values"] == "weights":
        gy *= 0.1
    return gy.to(_torch(spec["dtype"]))


def _generator(seed, device="cuda"):
    return torch.Generator(device=device).manual_seed(int(seed))


class _Pool:
    """One buffer per name and dtype that holds a part for each tensor (a program's flat buffers; the
    parts start on 256-byte boundaries, as separate allocations would)."""

    def __init__(self, specs):
        self.at, used = [], {}
        for s in specs:
            per = 256 // (2 if s["dtype"] == "fp16" else 4)
            begin = used.get(s["dtype"], 0)
            self.at.append((s["dtype"], begin, _numel(s)))
            used[s["dtype"]] = begin + -(-_numel(s) // per) * per
        self.used = used
        self.chan, self.channels = [], 0
        for s in specs:
            self.chan.append((self.channels, s["channels"]))
            self.channels += -(-s["channels"] // 64) * 64

    def make(self, double=False):
        return {d: torch.zeros(n, dtype=torch.float64 if double else _torch(d), device="cuda")
                for d, n in self.used.items()}

    def part(self, buf, i):
        d, begin, n = self.at[i]
        return buf[d][begin:begin + n]

    def make_channels(self, double=False):
        return torch.zeros(self.channels, dtype=torch.float64 if double else torch.float32, device="cuda")

    def part_channels(self, buf, i):
        begin, n = self.chan[i]
        return buf[begin:begin + n]


class _Plan:
    """Keeps a plan and its workspace; gives the plan back."""

    def __init__(self, tensors, mode):
        self.array = fq.fq_tensor_array(tensors)
        self.workspace = torch.zeros(fq.fq_workspace_bytes(self.array, mode) // 4, dtype=torch.int32, device="cuda")
        self.handle = fq.fq_plan_create(self.array, mode, self.workspace)

    def __del__(self):
        if getattr(self, "handle", None):
            fq.fq_plan_destroy(self.handle)


# --------------------------------------------------------------------------------------------- passes
def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    if kind == "distill":
        return _prepare_distill(case, gen)
    specs = _specs(case)
    if kind == "autograd":
        s = specs[0]
        x, theta = _values(s, gen)
        shape = (case["n"], case["c"], case["h"], case["w"])
        return dict(case=case, x=x.view(shape).requires_grad_(), theta=theta.requires_grad_(),
                    gy=_upstream(s, gen).view(shape), channel_dim=1 if case["scales"] == "channel" else None,
                    qmin=s["qmin"], qmax=s["qmax"])

    pool = _Pool(specs)
    train = kind != "codes"
    want_gx = case.get("gx", kind in ("list", "frame"))
    x, y = pool.make(), (pool.make() if train else None)
    gy, gx = (pool.make() if train else None), (pool.make() if want_gx else None)
    theta, gtheta = pool.make_channels(), pool.make_channels()
    state = dict(case=case, x=x, y=y, gy=gy, gx=gx, theta=theta, gtheta=gtheta)
    if kind == "codes":
        state["q"] = torch.zeros(_numel(specs[0]), dtype=torch.int8, device="cuda")
        state["s"] = pool.make_channels()
    if kind == "weights":
        state["m"], state["v"], state["step"] = pool.make_channels(), pool.make_channels(), 0
    tensors = []
    for i, s in enumerate(specs):
        xv, tv = _values(s, gen)
        pool.part(x, i).copy_(xv.view(-1))
        pool.part_channels(theta, i).copy_(tv)
        del xv
        if train:
            pool.part(gy, i).copy_(_upstream(s, gen).view(-1))
        t = fq.FqTensor.from_torch(
            s["outer"], s["channels"], s["inner"], s["qmin"], s["qmax"], x=pool.part(x, i),
            y=pool.part(y, i) if y else None, q=state.get("q"), theta=pool.part_channels(theta, i),
            s=state.get("s"), gy=pool.part(gy, i) if gy else None, gx=pool.part(gx, i) if gx else None,
            gtheta=pool.part_channels(gtheta, i), flags=0 if want_gx or not train else fq.FQ_FLAG_NO_DX)
        if kind == "weights":
            th = pool.part_channels(theta, i)
            t.set_adam(fq.FqAdam.from_torch(pool.part_channels(state["m"], i), pool.part_channels(state["v"], i),
                                            th, step=1, **ADAM))
        tensors.append(t)
    state["tensors"] = tensors

    if kind == "layer":
        nbytes = fq.fq_workspace_bytes(tensors[0], fq.FQ_MODE_BACKWARD)
        state["workspace"] = torch.zeros(nbytes // 4, dtype=torch.int32, device="cuda")
    elif kind == "weights" or (kind == "list" and case["call"] == "plan"):
        state["forward"] = _Plan(tensors, fq.FQ_MODE_FORWARD)
        state["backward"] = _Plan(tensors, fq.FQ_MODE_BACKWARD)
    elif kind == "list":
        state["array"] = fq.fq_tensor_array(tensors)
        for mode, name in ((fq.FQ_MODE_FORWARD, "ws_f"), (fq.FQ_MODE_BACKWARD, "ws_b")):
            nbytes = fq.fq_workspace_bytes(state["array"], mode)
            state[name] = torch.zeros(nbytes // 4, dtype=torch.int32, device="cuda")
    elif kind == "frame":
        workspaces = [torch.zeros(fq.fq_workspace_bytes(t, fq.FQ_MODE_BACKWARD) // 4, dtype=torch.int32,
                                  device="cuda") for t in tensors]
        state["workspaces"] = workspaces
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for t in tensors:
                fq.fq_forward(t)
            for t, ws in zip(reversed(tensors), reversed(workspaces)):
                fq.fq_backward(t, ws)
        state["graph"] = graph
    return state


def _pair(case, gen):
    """A student and a correlated teacher."""
    shape = (case["n"], case["c"], case["h"] * case["w"])
    student = torch.randn(shape, generator=gen, device="cuda") * 1.5
    teacher = student * 0.8 + torch.randn(shape, generator=gen, device="cuda") * 0.4
    return student.to(_torch(case["dtype"])), teacher.to(_torch(case["dtype"]))


def _prepare_distill(case, gen):
    n, c, m = case["n"], case["c"], case["h"] * case["w"]
    student, teacher = _pair(case, gen)
    grad = torch.zeros_like(student) if case["grad"] else None
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    d = fq.FqDistill.from_torch(n, c, m, student, teacher, out, grad, lam=LAMBDA, upstream=LOSS_SCALE)
    ws = torch.empty(fq.fq_distill_workspace_bytes(d) // 8, dtype=torch.float64, device="cuda")
    return dict(case=case, student=student, teacher=teacher, grad=grad, out=out, d=d, workspace=ws)


def run(state):
    kind = state["case"]["kind"]
    if kind == "layer":
        t = state["tensors"][0]
        fq.fq_forward(t)
        fq.fq_backward(t, state["workspace"])
    elif kind == "codes":
        fq.fq_forward(state["tensors"][0])
        return dict(q=state["q"], s=state["s"])
    elif kind == "autograd":
        y = fake_quantize(state["x"], state["theta"], state["qmin"], state["qmax"],
                          channel_dim=state["channel_dim"])
        gx, gtheta = torch.autograd.grad(y, (state["x"], state["theta"]), state["gy"])
        return dict(y=y, gx=gx, gtheta=gtheta)
    elif kind == "weights":
        state["step"] += 1
        fq.fq_plan_run(state["forward"].handle)
        fq.fq_plan_run_adam(state["backward"].handle, state["step"])
        return dict(y=state["y"], gtheta=state["gtheta"], theta=state["theta"], m=state["m"], v=state["v"])
    elif kind == "list":
        if state["case"]["call"] == "plan":
            fq.fq_plan_run(state["forward"].handle)
            fq.fq_plan_run(state["backward"].handle)
        else:
            fq.fq_multi_tensor(state["array"], fq.FQ_MODE_FORWARD, state["ws_f"])
            fq.fq_multi_tensor(state["array"], fq.FQ_MODE_BACKWARD, state["ws_b"])
    elif kind == "frame":
        state["graph"].replay()
    else:
        fq.fq_distill_loss(state["d"], state["workspace"])
        return dict(out=state["out"], grad=state["grad"])
    return dict(y=state["y"], gx=state["gx"], gtheta=state["gtheta"])


# ----------------------------------------------------------------------------- what a pass has to do
def work(case):
    """Every input read once, every output written once; the forward and the backward are separate calls,
    so each of them reads x.  Operations: about 5 per element forward, 8 backward, 20 per pair in the loss."""
    if case["kind"] == "distill":
        e, b = case["n"] * case["c"] * case["h"] * case["w"], 2 if case["dtype"] == "fp16" else 4
        return dict(bytes=float(e * b * (3 if case["grad"] else 2) + 24), flops=float(e * (20 if case["grad"] else 11)))
    nbytes = flops = 0.0
    for s in _specs(case):
        e, b = _numel(s), 2 if s["dtype"] == "fp16" else 4
        if case["kind"] == "codes":
            nbytes += e * (b + 1) + 8 * s["channels"]
            flops += 4 * e
            continue
        want_gx = case.get("gx", case["kind"] in ("list", "frame"))
        nbytes += e * b * (2 + (3 if want_gx else 2)) + 12 * s["channels"]
        if case["kind"] == "weights":
            nbytes += 24 * s["channels"]
        flops += 13 * e
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """FP16 outputs are rounded to 11 bits (measured against 64 bits: 2.1e-4 of the norm, with lists' 4-bit
    tensors the same); FP32 outputs and the scale gradients to 24 bits (3e-8 of the norm).  Codes do not differ."""
    return dict(rel=1e-3 if case.get("dtype", "fp16") == "fp16" and case["kind"] != "codes" else 2e-7)


# ------------------------------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    gen = _generator(seed)
    if case["kind"] == "distill":
        return _exact_distill(case, gen)
    specs = _specs(case)
    pool = _Pool(specs)
    kind = case["kind"]
    want_gx = case.get("gx", kind in ("list", "frame"))
    y = pool.make(True) if kind != "codes" else None
    gx = pool.make(True) if want_gx and kind != "codes" else None
    out = {k: pool.make_channels(True) for k in ("gtheta", "theta", "m", "v", "s")}
    q = None
    for i, spec in enumerate(specs):
        x, theta = _values(spec, gen)
        gy = _upstream(spec, gen) if kind != "codes" else None
        th = theta.double()
        # scales are binary32 values by definition: rounded once
        s = torch.nn.functional.softplus(th, threshold=1e9).float().double()
        # so are quotients: a channel's largest element lies exactly on the bound of the codes
        v = x.double().div_(s[None, :, None]).float().double()
        inside = (v >= spec["qmin"]) & (v <= spec["qmax"])
        code = torch.round(v.clamp(spec["qmin"], spec["qmax"]))
        if kind == "codes":
            q = code.to(torch.int8).view(-1)
            pool.part_channels(out["s"], i).copy_(s)
            continue
        pool.part(y, i).copy_((code * s[None, :, None]).view(-1))
        g = gy.double()
        if gx is not None:
            pool.part(gx, i).copy_((g * inside).view(-1))
        t = torch.where(inside, code - v, code)
        gth = (g * t).sum(dim=(0, 2)) * torch.sigmoid(th)
        pool.part_channels(out["gtheta"], i).copy_(gth)
        if kind == "weights":
            m, vv = (1 - ADAM["beta1"]) * gth, (1 - ADAM["beta2"]) * gth * gth
            step = ADAM["lr"] * (m / (1 - ADAM["beta1"])) / ((vv / (1 - ADAM["beta2"])).sqrt() + ADAM["eps"])
            for name, value in (("m", m), ("v", vv), ("theta", th - step)):
                pool.part_channels(out[name], i).copy_(value)
        del x, gy, v, inside, code, g, t
    if kind == "codes":
        return dict(q=q, s=out["s"])
    if kind == "autograd":
        shape = (case["n"], case["c"], case["h"], case["w"])
        return dict(y=y[case["dtype"]][:_numel(specs[0])].view(shape), gtheta=out["gtheta"][:specs[0]["channels"]],
                    gx=gx[case["dtype"]][:_numel(specs[0])].view(shape))
    if kind == "weights":
        return dict(y=y, gtheta=out["gtheta"], theta=out["theta"], m=out["m"], v=out["v"])
    return dict(y=y, gx=gx, gtheta=out["gtheta"])


def _exact_distill(case, gen):
    a, b = (v.double() for v in _pair(case, gen))
    diff = a - b
    mse = diff.square().mean()
    na, nb, dot = a.square().sum(1), b.square().sum(1), (a * b).sum(1)
    inv = 1.0 / (na.sqrt() * nb.sqrt())
    cos = dot * inv
    lam, positions = LAMBDA, cos.numel()
    out = torch.stack([mse, cos.mean(), mse + lam * (1.0 - cos.mean())])
    if not case["grad"]:
        return dict(out=out, grad=None)
    grad = diff * (2.0 / a.numel())
    grad -= lam / positions * (b * inv[:, None] - a * (cos / na)[:, None])
    return dict(out=out, grad=grad * LOSS_SCALE)
