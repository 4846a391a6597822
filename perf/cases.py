"""The work that a user of this framework has it do, as cases to measure.

Every case goes through the public binding (paper_2301_09266_amd.finc) on
device tensors, with the weights prepared once and the workspaces kept, as a
training or sampling program keeps them.  Kinds:

* layer: one padded masked convolution block, both directions (forward with
  log|det|, then the inverse of a latent).  Weights change every training
  step, so the forward also prepares the inverse's weights.
* unit, split: the four-block FInC unit (in sequence, or on channel quarters),
  both directions, the same way.
* banded: the inverse of images that do not fit one workgroup.
* backward: the gradients of one block.
* stack_sample: sampling from the multi-scale stack, weights prepared.
* stack_train: a training pass of the stack: latents, log|det|, loss, and the
  gradients of the input and of every parameter.
* step: one Step of the full flow (unit, actnorm, 1x1, coupling network),
  density and sampling direction.
* flow: the full multi-scale flow, density and sampling direction.

"graph" > 0: the pass is that many calls captured once in a HIP graph, as a
program does with calls of a few microseconds.
"""
import math

import torch

from paper_2301_09266_amd import finc

KINDS = ("layer", "unit", "split", "banded", "backward", "stack_sample", "stack_train", "step",
         "flow")


def listed():
    return [
        # the smallest call there is, one small image eagerly: launch and
        # host latency
        dict(name="layer_c3_8x8_b1", kind="layer", B=1, C=3, H=8, W=8, k=3, corner=0, graph=0),
        # the headline: CIFAR-10 after one squeeze, batch 64, in a graph of 20
        dict(name="layer_c12_16x16_b64", kind="layer", B=64, C=12, H=16, W=16, k=3, corner=0,
             graph=20),
        # ImageNet-64 after one squeeze with the wide kernel
        dict(name="layer_c12_32x32_b64_k5", kind="layer", B=64, C=12, H=32, W=32, k=5, corner=0,
             graph=4),
        # odd sizes, more channels than one tile, an odd batch, another corner
        dict(name="layer_c23_27x19_b33", kind="layer", B=33, C=23, H=27, W=19, k=3, corner=3,
             graph=4),
        # units of the first and the third level at a large batch
        dict(name="unit_c12_16x16_b256", kind="unit", B=256, C=12, H=16, W=16, k=3, graph=4),
        dict(name="unit_c48_8x8_b256", kind="unit", B=256, C=48, H=8, W=8, k=3, graph=4),
        # a large image: bands of rows pipelined over workgroups
        dict(name="banded_c12_128x128_b8", kind="banded", B=8, C=12, H=128, W=128, k=3, corner=0),
        # the gradients of one block at the ImageNet-64 size
        dict(name="backward_c12_32x32_b64", kind="backward", B=64, C=12, H=32, W=32, k=3,
             corner=0, graph=4),
        # sampling and a training pass of the stack of three levels of eight units
        dict(name="stack_sample_3x8_b64", kind="stack_sample", B=64, L=3, U=8, C=12, H=32, W=32,
             k=3),
        dict(name="stack_train_3x8_b64", kind="stack_train", B=64, L=3, U=8, C=12, H=32, W=32,
             k=3),
        # one Step of the CIFAR-10 flow's first level, 100 images
        dict(name="step_c12_16x16_b100", kind="step", B=100, C=12, H=16, W=16, k=3, hid=512),
        # the whole CIFAR-10 flow [28, 28, 28], 100 images, both directions
        dict(name="flow_cifar10_b100", kind="flow", B=100, L=3, K=28, C=3, H=32, W=32, k=3,
             hid=512),
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _draw(rng):
    kind = rng.choice(KINDS)
    k = rng.choice((2, 3, 3, 3, 5))
    corner = rng.randrange(4)
    if kind in ("layer", "backward"):
        return dict(kind=kind, B=_log(rng, 1, 256), C=_log(rng, 1, 48), H=_log(rng, 4, 64),
                    W=_log(rng, 4, 64), k=k, corner=corner, graph=rng.choice((0, 4)))
    if kind in ("unit", "split"):
        C = _log(rng, 1, 48) if kind == "unit" else 4 * _log(rng, 1, 12)
        return dict(kind=kind, B=_log(rng, 1, 256), C=C, H=_log(rng, 4, 40), W=_log(rng, 4, 40),
                    k=k, graph=rng.choice((0, 4)))
    if kind == "banded":
        return dict(kind=kind, B=_log(rng, 1, 16), C=_log(rng, 2, 16), H=_log(rng, 64, 256),
                    W=_log(rng, 32, 160), k=k, corner=corner)
    if kind in ("stack_sample", "stack_train"):
        L = rng.choice((1, 2, 3))
        q = 1 << (L - 1)
        return dict(kind=kind, B=_log(rng, 1, 96), L=L, U=rng.randrange(1, 9),
                    C=2 * _log(rng, 1, 6), H=q * rng.randrange(4, 11), W=q * rng.randrange(4, 11),
                    k=rng.choice((2, 3)))
    if kind == "step":
        return dict(kind=kind, B=_log(rng, 1, 128), C=4 * _log(rng, 1, 12), H=_log(rng, 4, 24),
                    W=_log(rng, 4, 24), k=3, hid=_log(rng, 32, 600))
    L = rng.choice((1, 2, 3))
    q = 2 << (L - 1)
    return dict(kind=kind, B=_log(rng, 1, 100), L=L, K=rng.randrange(1, 9), C=rng.choice((1, 3)),
                H=q * rng.randrange(2, 9 - L), W=q * rng.randrange(2, 9 - L), k=3,
                hid=_log(rng, 32, 512))


def _accepted(c):
    """Whether the library takes the case (its plans say so, on the host)."""
    kind, B, C, H, W, k = (c[n] for n in ("kind", "B", "C", "H", "W", "k"))
    if kind == "banded":
        return not isinstance(finc.banded_plan(C, H, W, k), int)
    plan = {"layer": finc.PLAN_LAYER, "unit": finc.PLAN_UNIT, "split": finc.PLAN_SPLIT}
    if kind in plan:
        return not (isinstance(finc.inverse_plan(plan[kind], C, H, W, k), int) or
                    isinstance(finc.forward_plan(plan[kind], B, C, H, W, k), int))
    if kind == "stack_sample":
        return not isinstance(finc.inverse_plan(finc.PLAN_STACK, C, H, W, k, c["L"], c["U"]), int)
    if kind == "stack_train":
        return not any(isinstance(finc.forward_plan(finc.PLAN_UNIT, B, C << l, H >> l, W >> l, k),
                                  int) for l in range(c["L"]))
    if kind == "step":
        return not isinstance(finc.inverse_plan(finc.PLAN_SPLIT, C, H, W, k), int)
    if kind == "flow":
        return not any(isinstance(finc.inverse_plan(finc.PLAN_SPLIT, C << (l + 2), H >> (l + 1),
                                                    W >> (l + 1), k), int)
                       for l in range(c["L"]))
    return True


def draw(rng):
    while True:
        c = _draw(rng)
        if c["B"] * c["C"] * c["H"] * c["W"] <= (1 << 22) and _accepted(c):
            return c


# --- inputs ----------------------------------------------------------------
# Activations and latents ~ N(0, 1).  A block's weights ~ N(0, std^2) with the
# self tap's upper triangle 0 and its diagonal 1 + U(-0.1, 0.1): std 0.05 (the
# benchmark's) for single blocks and units, less where the block is wider, so
# that the inverse stays bounded as a trained flow's; 0.02 in chains of many.

def _std(C, k, chain):
    return min(0.02 if chain else 0.05, (0.2 if chain else 0.5) / math.sqrt(C * k * k))


def _self_tap(corner, k):
    return (k - 1 if corner in (0, 1) else 0), (k - 1 if corner in (0, 2) else 0)


class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def n(self, *shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=self.g, device="cuda") * std + mean

    def blocks(self, n, C, k, corners, chain=False):
        """(n, C, C, k, k); block i has corner corners[i % len(corners)]."""
        K = self.n(n, C, C, k, k, std=_std(C, k, chain))
        d = 1.0 + 0.2 * torch.rand((n, C), generator=self.g, device="cuda") - 0.1
        low = torch.tril(torch.ones(C, C, device="cuda"), -1)
        for i, corner in enumerate(corners):
            a, b = _self_tap(corner, k)
            K[i::len(corners), :, :, a, b] = (K[i::len(corners), :, :, a, b] * low +
                                              torch.diag_embed(d[i::len(corners)]))
        return K

    def steps(self, n, C, k, hid):
        """(n, parameters): n Steps' parameters in the library's flat layout."""
        Ch = C // 2
        Wm = torch.linalg.qr(self.n(n, C, C).double().cpu())[0].float().cuda()
        b3 = self.n(n, C, std=0.01)
        b3[:, Ch:] += 2.0
        parts = [self.blocks(4 * n, C // 4, k, (0, 1, 2, 3), chain=True),
                 self.n(n, C, std=0.1).exp(), self.n(n, C, std=0.1), Wm,
                 self.n(n, hid, Ch, 3, 3, std=math.sqrt(2 / (9 * Ch))), self.n(n, hid, std=0.01),
                 self.n(n, hid, hid, std=math.sqrt(2 / hid)), self.n(n, hid, std=0.01),
                 self.n(n, C, hid, 3, 3, std=0.02 / math.sqrt(9 * hid)), b3,
                 self.n(n, C, std=0.01)]
        return torch.cat([p.reshape(n, -1) for p in parts], 1)

    def prior(self, C):
        return torch.cat([p.reshape(-1) for p in
                          (self.n(C, C // 2, 3, 3, std=0.02 / math.sqrt(9 * (C // 2))),
                           self.n(C, std=0.01), self.n(C, std=0.01))])


def _inputs(case, seed):
    """The tensors that a user's program has: the same for run and exact."""
    kind, B, C, H, W, k = (case[n] for n in ("kind", "B", "C", "H", "W", "k"))
    g = _Gen(seed)
    if kind in ("layer", "unit", "split", "banded", "backward"):
        s = dict(x=g.n(B, C, H, W), z=g.n(B, C, H, W))
        if kind == "split":
            s["K"] = g.blocks(4, C // 4, k, (0, 1, 2, 3))
        elif kind == "unit":
            s["K"] = g.blocks(4, C, k, (0, 1, 2, 3))
        else:
            s["K"] = g.blocks(1, C, k, (case["corner"],))[0]
        return s
    if kind in ("stack_sample", "stack_train"):
        L, U = case["L"], case["U"]
        dims = [(C << l, H >> l, W >> l) for l in range(L)]
        return dict(
            x=g.n(B, C, H, W),
            z=[g.n(B, c if l == L - 1 else c // 2, h, w) for l, (c, h, w) in enumerate(dims)],
            K=torch.cat([g.blocks(4 * U, c, k, (0, 1, 2, 3), chain=True).reshape(-1)
                         for c, _, _ in dims]),
            scale=torch.cat([g.n(U, c, std=0.1).exp().reshape(-1) for c, _, _ in dims]),
            bias=torch.cat([g.n(U, c, std=0.1).reshape(-1) for c, _, _ in dims]))
    if kind == "step":
        return dict(x=g.n(B, C, H, W), z=g.n(B, C, H, W),
                    params=g.steps(1, C, k, case["hid"]).reshape(-1))
    L = case["L"]
    parts = []
    for l in range(L):
        parts.append(g.steps(case["K"], C << (l + 2), k, case["hid"]).reshape(-1))
        if l < L - 1:
            parts.append(g.prior(C << (l + 2)))
    return dict(x=g.n(B, C, H, W), params=torch.cat(parts),
                z=[g.n(*shape) for shape in finc.flow_latent_shapes(B, L, C, H, W)])


# --- the measured passes ---------------------------------------------------

def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _pass(s):
    """One call of each direction of the case; its outputs."""
    c, kind = s["case"], s["case"]["kind"]
    k = c["k"]
    if kind == "layer":
        finc.forward(s["x"], s["K"], c["corner"], out=s["y"], logdet=s["ld"], prepared=s["prep"])
        finc.inverse_prepared(s["z"], s["prep"], k, c["corner"], out=s["xi"])
        return s["y"], s["ld"], s["xi"]
    if kind == "unit":
        finc.unit_forward(s["x"], s["K"], out=s["y"], logdet=s["ld"], prepared=s["prep"])
        finc.unit_inverse_prepared(s["z"], s["prep"], k, out=s["xi"])
        return s["y"], s["ld"], s["xi"]
    if kind == "split":
        finc.split_forward(s["x"], s["K"], out=s["y"], logdet=s["ld"], prepared=s["prep"])
        finc.split_inverse_prepared(s["z"], s["prep"], k, out=s["xi"])
        return s["y"], s["ld"], s["xi"]
    if kind == "banded":
        return finc.inverse_banded(s["z"], s["K"], c["corner"], out=s["xi"], workspace=s["ws"])[0]
    if kind == "backward":
        return finc.backward(s["x"], s["z"], s["K"], c["corner"], gld=-float(c["B"]), dx=s["xi"],
                             dK=s["dK"], workspace=s["ws"])
    if kind == "stack_sample":
        return finc.stack_inverse_prepared(s["z"], s["prep"], s["scale"], s["bias"], c["L"],
                                           c["U"], c["C"], c["H"], c["W"], k, out=s["xi"])
    if kind == "stack_train":
        par = (s["K"], s["scale"], s["bias"], c["L"], c["U"], k)
        z, ld = finc.stack_forward(s["x"], *par, workspace=s["ws"])
        nll, bpd = finc.gauss_nll(z, ld)
        grads = finc.stack_backward(s["x"], z, *par, gld=-float(c["B"]), workspace=s["ws"])
        return list(z), ld, nll, bpd, list(grads)
    if kind == "step":
        s["ld"].zero_()
        finc.step_forward(s["x"], s["params"], s["prep"], k, c["hid"], out=s["y"], logdet=s["ld"],
                          workspace=s["ws"])
        finc.step_inverse(s["z"], s["params"], s["prep"], k, c["hid"], out=s["xi"],
                          workspace=s["ws"])
        return s["y"], s["ld"], s["xi"]
    z, ld = finc.flow_forward(s["x"], s["params"], s["prep"], c["L"], c["K"], k, c["hid"],
                              workspace=s["ws"])
    x = finc.flow_sample(s["z"], s["params"], s["prep"], c["L"], c["K"], c["C"], c["H"], c["W"],
                         k, c["hid"], out=s["xi"], workspace=s["ws"])
    return list(z), ld, x


def prepare(case, seed):
    kind, B, C, H, W, k = (case[n] for n in ("kind", "B", "C", "H", "W", "k"))
    s = dict(_inputs(case, seed), case=case)
    s["xi"] = torch.empty(B, C, H, W, device="cuda")
    if kind in ("layer", "unit", "split"):
        s["y"] = torch.empty_like(s["x"])
        s["ld"] = torch.empty(1, dtype=torch.float64, device="cuda")
        s["prep"] = _bytes(finc.workspace_bytes(C // 4 if kind == "split" else C, k,
                                                1 if kind == "layer" else 4))
    elif kind == "banded":
        s["ws"] = _bytes(finc.lib().finc_banded_workspace_bytes(B, C, H, W, k, 1))
    elif kind == "backward":
        s["dK"] = torch.empty_like(s["K"])
        s["ws"] = _bytes(finc.lib().finc_backward_workspace_bytes(B, C, H, W, k))
    elif kind == "stack_sample":
        s["prep"] = finc.stack_prepare(s["K"], case["L"], case["U"], C, k)
    elif kind == "stack_train":
        s["ws"] = _bytes(finc.lib().finc_stack_train_workspace_bytes(B, case["L"], case["U"], C, H,
                                                                     W, k))
    elif kind == "step":
        s["y"] = torch.empty_like(s["x"])
        s["ld"] = torch.empty(B, dtype=torch.float64, device="cuda")
        s["prep"] = finc.step_prepare(s["params"], C, k, case["hid"])
        s["ws"] = _bytes(finc.lib().finc_step_workspace_bytes(B, C, H, W, case["hid"]))
    else:
        s["prep"] = finc.flow_prepare(s["params"], case["L"], case["K"], C, k, case["hid"])
        s["ws"] = _bytes(finc.lib().finc_flow_workspace_bytes(B, case["L"], C, H, W, case["hid"]))
    if case.get("graph"):
        s["out"] = _pass(s)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for _ in range(case["graph"]):
                _pass(s)
        torch.cuda.synchronize()
    return s


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    return _pass(state)


# --- what a pass cannot do without -----------------------------------------

def _conv_flops(C, k, hw):
    return 2 * hw * (C * C * k * k - C * (C - 1) // 2)


def work(case):
    kind, B, C, H, W, k = (case[n] for n in ("kind", "B", "C", "H", "W", "k"))
    act, hw, n = 4 * B * C * H * W, B * H * W, max(1, case.get("graph", 0))
    wts = 4 * C * C * k * k
    if kind == "layer":
        return dict(bytes=n * (4 * act + wts), flops=n * 2 * _conv_flops(C, k, hw))
    if kind == "unit":
        return dict(bytes=n * (4 * act + 4 * wts), flops=n * 8 * _conv_flops(C, k, hw))
    if kind == "split":
        return dict(bytes=n * (4 * act + wts // 4), flops=n * 8 * _conv_flops(C // 4, k, hw))
    if kind == "banded":
        return dict(bytes=2 * act + wts, flops=_conv_flops(C, k, hw))
    if kind == "backward":
        return dict(bytes=n * (3 * act + 2 * wts), flops=n * 2 * _conv_flops(C, k, hw))
    if kind in ("stack_sample", "stack_train"):
        L, U = case["L"], case["U"]
        f = sum(4 * U * _conv_flops(C << l, k, hw >> (2 * l)) for l in range(L))
        w = sum(4 * U * (wts << (2 * l)) for l in range(L))
        if kind == "stack_sample":
            return dict(bytes=2 * act + w, flops=f)
        return dict(bytes=3 * act + 2 * w, flops=3 * f)   # forward, both gradients

    def step_flops(C, hw):
        hid = case["hid"]
        net = 2 * hw * (9 * hid * (C // 2) + hid * hid + 9 * hid * C)
        return 4 * _conv_flops(C // 4, k, hw) + 2 * hw * C * C + net

    if kind == "step":
        return dict(bytes=4 * act + 4 * finc.step_param_count(C, k, case["hid"]),
                    flops=2 * step_flops(C, hw))
    L, K = case["L"], case["K"]
    f = 0
    for l in range(L):
        c, q = C << (l + 2), hw >> (2 * (l + 1))
        f += K * step_flops(c, q) + (2 * q * 9 * c * (c // 2) if l < L - 1 else 0)
    return dict(bytes=4 * act + 4 * finc.flow_param_count(L, K, C, k, case["hid"]), flops=2 * f)


def tolerance(case):
    """About four times the relative errors (2-norm) against 64 bits that these
    32-bit sums show over the declared ranges: single blocks, units and their
    gradients up to 3.3e-7 (twice that between two summation orders), one Step
    1.6e-7 (more where its log|det| is near 0), chains of units or Steps up to
    4.9e-6 by their condition."""
    if case["kind"] in ("layer", "unit", "split", "banded", "backward"):
        return {"rel": 2e-6}
    if case["kind"] == "step":
        return {"rel": 5e-6}
    return {"rel": 2e-5}


# --- the same in 64 bits, in plain torch -----------------------------------

def _taps64(x, K, corner):
    """y = K * pad_corner(x), the self tap's upper triangle left out."""
    B, C, H, W = x.shape
    k = K.shape[-1]
    oh, ow = _self_tap(corner, k)
    xp = torch.nn.functional.pad(x, (ow, k - 1 - ow, oh, k - 1 - oh))
    y = 0
    for a in range(k):
        for b in range(k):
            Kt = K[:, :, a, b]
            if (a, b) == (oh, ow):
                Kt = torch.tril(Kt)
            y = y + torch.matmul(Kt, xp[:, :, a:a + H, b:b + W].reshape(B, C, H * W))
    return y.view(B, C, H, W)


def _logdet64(K, corner, hw):
    a, b = _self_tap(corner, K.shape[-1])
    return hw * torch.diagonal(K[:, :, a, b]).abs().log().sum()


def _solve64(y, K, corner):
    """The inverse, diagonal by diagonal of the top-left frame."""
    C, k = K.shape[0], K.shape[-1]
    fl = [d for d, f in ((2, corner in (2, 3)), (3, corner in (1, 3))) if f]
    y, K = y.flip(fl), K.flip(fl)
    B, _, H, W = y.shape
    P = k - 1
    Li = torch.linalg.solve_triangular(torch.tril(K[:, :, P, P]),
                                       torch.eye(C, dtype=K.dtype, device=K.device), upper=False)
    taps = [(p, q) for p in range(k) for q in range(k) if (p, q) != (0, 0)]
    WP = W + P
    xp = torch.zeros(B, C, (H + P) * WP, dtype=y.dtype, device=y.device)
    if taps:
        M = torch.matmul(Li, torch.stack([K[:, :, P - p, P - q] for p, q in taps], 0))
        M = M.permute(1, 0, 2).reshape(C, -1).contiguous()    # (C, taps C)
        back = torch.tensor([p * WP + q for p, q in taps], device=y.device)
    y = torch.matmul(Li, y.reshape(B, C, H * W))
    for d in range(H + W - 1):
        lo, hi = max(0, d - W + 1), min(H - 1, d)
        i = torch.arange(lo, hi + 1, device=y.device)
        at = (i + P) * WP + (d - i) + P
        v = y[:, :, i * W + (d - i)]
        if taps:
            src = xp[:, :, at[None, :] - back[:, None]]       # (B, C, taps, n)
            v = v - torch.matmul(M, src.transpose(1, 2).reshape(B, len(taps) * C, -1))
        xp[:, :, at] = v
    return xp.view(B, C, H + P, WP)[:, :, P:, P:].flip(fl)


def _unit64(x, K4):
    for q in range(4):
        x = _taps64(x, K4[q], q)
    return x


def _unit_solve64(y, K4):
    for q in (3, 2, 1, 0):
        y = _solve64(y, K4[q], q)
    return y


def _split64(x, Kq4, f):
    return torch.cat([f(xq.contiguous(), Kq4[q], q) for q, xq in enumerate(x.chunk(4, 1))], 1)


def _squeeze(x):
    B, C, H, W = x.shape
    return x.view(B, C, H // 2, 2, W // 2, 2).permute(0, 1, 3, 5, 2, 4).reshape(B, 4 * C, H // 2,
                                                                               W // 2)


def _unsqueeze(x):
    B, C, H, W = x.shape
    return x.view(B, C // 4, 2, 2, H, W).permute(0, 1, 4, 2, 5, 3).reshape(B, C // 4, 2 * H, 2 * W)


def _stack_parts(case, s):
    """Per level: blocks (U, 4, C, C, k, k), scales and biases (U, C)."""
    out, ko, so = [], 0, 0
    for l in range(case["L"]):
        C, U, k = case["C"] << l, case["U"], case["k"]
        nk, ns = U * 4 * C * C * k * k, U * C
        out.append((s["K"][ko:ko + nk].view(U, 4, C, C, k, k), s["scale"][so:so + ns].view(U, C),
                    s["bias"][so:so + ns].view(U, C)))
        ko, so = ko + nk, so + ns
    return out


def _ch(v):
    return v.view(1, -1, 1, 1)


def _same64(x, Wt):
    """Zero-padded "same" convolution, Wt (co, ci, R, R)."""
    B, C, H, W = x.shape
    R = Wt.shape[-1]
    xp = torch.nn.functional.pad(x, (R // 2,) * 4)
    y = 0
    for a in range(R):
        for b in range(R):
            y = y + torch.matmul(Wt[:, :, a, b], xp[:, :, a:a + H, b:b + W].reshape(B, C, H * W))
    return y.view(B, -1, H, W)


def _step_parts(p, C, k, hid):
    q, Ch = C // 4, C // 2
    shapes = [(4, q, q, k, k), (C,), (C,), (C, C), (hid, Ch, 3, 3), (hid,), (hid, hid, 1, 1),
              (hid,), (C, hid, 3, 3), (C,), (C,)]
    out, o = [], 0
    for sh in shapes:
        n = math.prod(sh)
        out.append(p[o:o + n].view(sh))
        o += n
    return out, o


def _net64(va, parts):
    _, _, _, _, W1, b1, W2, b2, W3, b3, ls = parts
    h = torch.relu(_same64(va, W1) + _ch(b1))
    h = torch.relu(_same64(h, W2) + _ch(b2))
    h = (_same64(h, W3) + _ch(b3)) * _ch(torch.exp(3 * ls))
    t, r = h.chunk(2, 1)
    return t, torch.sigmoid(r + 2)


def _step64(x, parts, k):
    Kq4, s, b, Wm = parts[:4]
    B, C, H, W = x.shape
    v = _split64(x, Kq4, _taps64)
    v = torch.matmul(Wm, (_ch(s) * v + _ch(b)).reshape(B, C, H * W)).view(B, C, H, W)
    va, vb = v.chunk(2, 1)
    t, sc = _net64(va, parts)
    ld = sum(_logdet64(Kq4[q], q, H * W) for q in range(4))
    ld = ld + H * W * (s.abs().log().sum() + torch.linalg.slogdet(Wm.cpu())[1].to(s.device))
    return torch.cat([va, (vb + t) * sc], 1), ld + sc.log().sum((1, 2, 3))


def _step_solve64(y, parts, k):
    Kq4, s, b, Wm = parts[:4]
    B, C, H, W = y.shape
    va, vb = y.chunk(2, 1)
    t, sc = _net64(va, parts)
    v = torch.cat([va, vb / sc - t], 1).reshape(B, C, H * W)
    v = torch.matmul(torch.linalg.inv(Wm.cpu()).to(y.device), v).view(B, C, H, W)
    return _split64((v - _ch(b)) / _ch(s), Kq4, _solve64)


def _flow_parts(case, p):
    """Per level: its Steps' parts, and its prior's (or None)."""
    out, o = [], 0
    for l in range(case["L"]):
        C, steps = case["C"] << (l + 2), []
        for _ in range(case["K"]):
            parts, n = _step_parts(p[o:], C, case["k"], case["hid"])
            steps.append(parts)
            o += n
        prior = None
        if l < case["L"] - 1:
            n = C * (C // 2) * 9
            prior = p[o:o + n].view(C, C // 2, 3, 3), p[o + n:o + n + C], p[o + n + C:o + n + 2 * C]
            o += n + 2 * C
        out.append((steps, prior))
    return out


def _prior64(h1, prior):
    Wp, bp, ls = prior
    return ((_same64(h1, Wp) + _ch(bp)) * _ch(torch.exp(3 * ls))).chunk(2, 1)


def exact(case, seed):
    kind, H, W, k = (case[n] for n in ("kind", "H", "W", "k"))
    s = {n: ([t.double() for t in v] if isinstance(v, list) else v.double())
         for n, v in _inputs(case, seed).items()}
    K = s.get("K")
    if kind == "layer":
        c = case["corner"]
        return (_taps64(s["x"], K, c), _logdet64(K, c, H * W).view(1), _solve64(s["z"], K, c))
    if kind == "unit":
        ld = sum(_logdet64(K[q], q, H * W) for q in range(4))
        return _unit64(s["x"], K), ld.view(1), _unit_solve64(s["z"], K)
    if kind == "split":
        ld = sum(_logdet64(K[q], q, H * W) for q in range(4))
        return _split64(s["x"], K, _taps64), ld.view(1), _split64(s["z"], K, _solve64)
    if kind == "banded":
        return _solve64(s["z"], K, case["corner"])
    if kind == "backward":
        c = case["corner"]
        x, K = s["x"].requires_grad_(), K.requires_grad_()
        loss = (_taps64(x, K, c) * s["z"]).sum() - case["B"] * _logdet64(K, c, H * W)
        return torch.autograd.grad(loss, (x, K))
    if kind == "stack_sample":
        levels, h = _stack_parts(case, s), None
        for l in reversed(range(case["L"])):
            h = s["z"][l] if h is None else torch.cat([_unsqueeze(h), s["z"][l]], 1)
            Kl, sc, bi = levels[l]
            for u in reversed(range(case["U"])):
                h = _unit_solve64((h - _ch(bi[u])) / _ch(sc[u]), Kl[u])
        return h
    if kind == "stack_train":
        for n in ("x", "K", "scale", "bias"):
            s[n].requires_grad_()
        h, z, ld = s["x"], [], 0
        for l, (Kl, sc, bi) in enumerate(_stack_parts(case, s)):
            hw = h.shape[2] * h.shape[3]
            for u in range(case["U"]):
                h = _ch(sc[u]) * _unit64(h, Kl[u]) + _ch(bi[u])
                ld = ld + hw * sc[u].abs().log().sum()
                ld = ld + sum(_logdet64(Kl[u, q], q, hw) for q in range(4))
            if l < case["L"] - 1:
                h, zl = h.chunk(2, 1)
                z.append(zl)
                h = _squeeze(h)
        z.append(h)
        D = math.prod(s["x"].shape[1:])
        nll = sum(0.5 * (v * v).sum((1, 2, 3)) for v in z) + 0.5 * D * math.log(2 * math.pi) - ld
        grads = torch.autograd.grad(nll.sum(), (s["x"], s["K"], s["scale"], s["bias"]))
        nll = nll.detach()
        return ([v.detach() for v in z], ld.detach().expand(case["B"]), nll,
                nll / (D * math.log(2)), list(grads))
    if kind == "step":
        parts = _step_parts(s["params"], case["C"], k, case["hid"])[0]
        y, ld = _step64(s["x"], parts, k)
        return y, ld, _step_solve64(s["z"], parts, k)
    levels = _flow_parts(case, s["params"])
    h, z, ld = s["x"], [], 0
    for steps, prior in levels:
        h = _squeeze(h)
        for parts in steps:
            h, d = _step64(h, parts, k)
            ld = ld + d
        if prior is not None:
            h, h2 = h.chunk(2, 1)
            mean, logsd = _prior64(h, prior)
            z.append((h2 - mean) * torch.exp(-logsd))
            ld = ld - logsd.sum((1, 2, 3))
    z.append(h)
    x = None
    for l in reversed(range(case["L"])):
        steps, prior = levels[l]
        if prior is None:
            x = s["z"][l]
        else:
            mean, logsd = _prior64(x, prior)
            x = torch.cat([x, mean + torch.exp(logsd) * s["z"][l]], 1)
        for parts in reversed(steps):
            x = _step_solve64(x, parts, k)
        x = _unsqueeze(x)
    return z, ld, x
