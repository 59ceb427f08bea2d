"""The layer calls whose speed this library is measured by, over the ranges in
which its public entry points are used.

A case is one convolution layer x[B,C,N,N], w[K,C,n,n] (arXiv:1601.06815,
Sections 2 and 3.2) with a tiling, a method and the way a program calls it:

- "step": a training step on a ``binding.Plan``: forward, error propagation and
  weight gradient, into buffers that the program keeps. The backward passes
  reuse the spectra of the same step's forward pass.
- "autograd": the same step through ``autograd.OaAConv2d``: forward and
  ``torch.autograd.grad`` with respect to the input and the weight.
- "forward": one forward pass, kernels transformed anew (the paper's forward
  timings, Sections 3.2 to 3.4).
- "infer": a forward pass with the kernel spectra the plan already holds, as a
  serving loop with fixed weights calls it.
- "noalloc": the forward pass in the library's static scratch.
- "chain": two stacked layers composed in the frequency domain, then applied.

Every input and result is float32, the only type the library takes.
"""

import math

import torch

from paper_1601_06815_amd import binding
from paper_1601_06815_amd.autograd import OaAConv2d


def _case(name, how, B, C, K, N, n, tiling="auto", method="oaa", x="uniform", g="uniform", J=0, n1=0):
    return {"name": name, "how": how, "B": B, "C": C, "K": K, "N": N, "n": n, "tiling": tiling, "method": method,
            "x": x, "g": g, "J": J, "n1": n1}


def listed():
    return [
        # the smallest layer of the tests and of the smoke check: launches and host work
        _case("tiny_step", "step", 1, 3, 4, 32, 5, tiling="paper"),
        # a single plane under one 8 x 8 kernel, the paper's headline speed-up: one latency-bound call
        _case("plane224_noalloc", "noalloc", 1, 1, 1, 224, 8),
        # Section 3.2: 32 x 32 input, 5 x 5 kernels, the most kernels of the sweep, the paper's blocks
        _case("kernels500_step", "step", 1, 1, 500, 32, 5, tiling="paper"),
        # Section 3.3: 64 x 64 input, 100 kernels, kernels beyond half the plane (transform side 128)
        _case("ksize48_step", "step", 1, 1, 100, 64, 48),
        # Section 3.4: 100 kernels of 5 x 5 over a large plane, forward only
        _case("input256_forward", "forward", 1, 1, 100, 256, 5),
        # a small batch with no size a multiple of anything, few channels: the vector contraction
        _case("ragged_autograd", "autograd", 5, 19, 27, 61, 9),
        # the output-tiled method on an ordinary middle layer
        _case("oas57_step", "step", 16, 48, 64, 57, 7, method="oas", g="normal"),
        # serving a middle layer with fixed weights
        _case("infer56_b8", "infer", 8, 64, 96, 56, 5, x="relu_normal"),
        # two stacked 64-channel layers composed and applied
        _case("chain60", "chain", 4, 64, 64, 60, 7, J=64, n1=3),
        # the RGB first layer of an image network
        _case("first224_autograd", "autograd", 64, 3, 64, 224, 7),
        # a middle layer with many channels and small kernels
        _case("mid56_autograd", "autograd", 128, 128, 128, 56, 3, x="relu_normal"),
        # the large-kernel layer that the benchmark times
        _case("large128_step", "step", 32, 96, 256, 128, 16, g="normal"),
    ]


def _log_int(rng, lo, hi):
    """An integer in [lo, hi], spread evenly over the logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _cost(c):
    w = work(c)
    return max(w["bytes"] / 5e12, w["flops"] / 100e12)


def draw(rng):
    most = _cost(listed()[-1])
    while True:
        how = rng.choice(["step", "step", "autograd", "autograd", "forward", "infer", "noalloc", "chain"])
        kind = rng.choice(["single", "first", "middle", "middle"])
        J = n1 = 0
        if kind == "single" and how != "chain":  # the paper's sweeps: one image, one channel
            B, C, K = 1, 1, _log_int(rng, 1, 750)
            N = _log_int(rng, 8, 256)
            n = _log_int(rng, 1, min(64, N))
        elif kind == "first" and how != "chain":  # few input channels, larger planes
            B, C, K = _log_int(rng, 1, 64), rng.randint(1, 4), _log_int(rng, 8, 96)
            N = _log_int(rng, 32, 224)
            n = rng.randint(3, 11)
        else:
            B, C, K = _log_int(rng, 1, 128), _log_int(rng, 5, 256), _log_int(rng, 5, 256)
            N = _log_int(rng, 14, 128)
            n = _log_int(rng, 1, min(16, N))
        if how == "chain":
            J, n1, n2 = _log_int(rng, 8, 128), rng.randint(1, 5), rng.randint(1, 5)
            n = n1 + n2 - 1
        method = "oas" if how != "autograd" and rng.random() < 0.15 else "oaa"
        if how == "chain" and (C <= 4 or N < n):
            continue
        if how == "noalloc":  # spectra within the 64 MiB of static scratch, with room for any tiling
            B, K = min(B, 2), min(K, 16)
            C = min(C, 16)
            if B * (C + 2 * K) * N * N > 1 << 19:
                continue
        # the paper's blocks of the kernel's size are used with kernels that fill them
        tiling = "paper" if how != "autograd" and n >= 3 and rng.random() < 0.25 else "auto"
        if tiling == "paper" and kind != "single" and B * (C + K) * N * N > 1 << 25:
            continue
        c = _case("", how, B, C, K, N, n, tiling=tiling, method=method, x=rng.choice(["uniform", "relu_normal"]),
                  g=rng.choice(["uniform", "normal"]), J=J, n1=n1)
        del c["name"]
        if _cost(c) <= 0.5 * most:
            return c


def _tensor(gen, dist, shape, var=1.0):
    if dist == "uniform":
        return torch.rand(shape, generator=gen, device="cuda") * 2 - 1
    t = torch.randn(shape, generator=gen, device="cuda")
    return t.clamp_(min=0) if dist == "relu_normal" else t.mul_(math.sqrt(var))


def _inputs(c, seed):
    """x, w (or w1, w2 of a chain) and g, as float32 on the GPU; kernels with fan-in variance."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, C, K, N, n, M = c["B"], c["C"], c["K"], c["N"], c["n"], c["N"] - c["n"] + 1
    x = _tensor(gen, c["x"], (B, C, N, N))
    if c["how"] == "chain":
        J, n1 = c["J"], c["n1"]
        n2 = n - n1 + 1
        ws = [_tensor(gen, "normal", (J, C, n1, n1), 1 / (C * n1 * n1)),
              _tensor(gen, "normal", (K, J, n2, n2), 1 / (J * n2 * n2))]
    else:
        ws = [_tensor(gen, "normal", (K, C, n, n), 1 / (C * n * n))]
    g = _tensor(gen, c["g"], (B, K, M, M)) if c["how"] in ("step", "autograd") else None
    return x, ws, g


def prepare(case, seed):
    c = case
    x, ws, g = _inputs(c, seed)
    B, C, K, N, n = c["B"], c["C"], c["K"], c["N"], c["n"]
    s = {"how": c["how"], "x": x, "g": g}
    if c["how"] == "autograd":
        layer = OaAConv2d(C, K, n, tiling=c["tiling"])
        with torch.no_grad():
            layer.weight.copy_(ws[0])
        layer.plan_for(B, N)
        s.update(layer=layer, x=x.requires_grad_())
        return s
    method = binding.METHOD_OVERLAP_SAVE if c["method"] == "oas" else binding.METHOD_OVERLAP_ADD
    plan = binding.Plan(B, C, K, N, n, device=x.device, tiling=c["tiling"], method=method)
    if c["how"] == "chain":
        # a chain composes unfused kernel spectra
        s.update(w1=ws[0], w2=ws[1])
    else:
        s.update(w=ws[0])
    M = plan.output_side
    s.update(plan=plan, y=torch.empty((B, K, M, M), device="cuda"))
    if c["how"] == "step":
        s.update(dx=torch.empty_like(x), dw=torch.empty_like(ws[0]))
    if c["how"] == "infer":
        plan.forward(x, ws[0], s["y"])  # a warm-up call, after which the plan holds the kernel spectra
    return s


def run(state):
    s = state
    how = s["how"]
    if how == "autograd":
        y = s["layer"](s["x"])
        dx, dw = torch.autograd.grad(y, (s["x"], s["layer"].weight), s["g"])
        return {"y": y, "dx": dx, "dw": dw}
    plan = s["plan"]
    if how == "step":
        plan.forward(s["x"], s["w"], s["y"])
        plan.backward_data(s["g"], None, s["dx"])
        plan.backward_filter(None, None if plan.caches_grad_spectra else s["g"], s["dw"])
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    if how == "forward":
        return {"y": plan.forward(s["x"], s["w"], s["y"])}
    if how == "infer":
        return {"y": plan.forward(s["x"], None, s["y"])}
    if how == "noalloc":
        return {"y": plan.forward_noalloc(s["x"], s["w"], s["y"])}
    plan.set_kernel_chain(s["w1"], s["w2"])
    return {"y": plan.forward(s["x"], None, s["y"])}


def work(case):
    """Bytes: inputs read once, results written once. Flops: the method's, at
    the cheapest tiling: real transforms of 2.5 L^2 log2(L^2) flops per tile
    and channel each way, and 6 flops per complex multiply-add of every bin
    that is not another's conjugate."""
    c = case
    B, C, K, N, n, J = c["B"], c["C"], c["K"], c["N"], c["n"], c["J"]
    M = N - n + 1
    train = c["how"] in ("step", "autograd")
    px, py, pw = B * C * N * N, B * K * M * M, K * C * n * n
    if c["how"] == "chain":
        n2 = n - c["n1"] + 1
        pw = J * C * c["n1"] ** 2 + K * J * n2 ** 2
    if c["how"] == "infer":
        pw = 0
    nbytes = 4 * (px + py + pw) * (2 if train else 1)
    L, best = 2, None
    while L < 2 * n - 1:
        L *= 2
    while L <= 128:
        tiles = B * (-(-N // (L - n + 1))) ** 2
        fft = 2.5 * L * L * math.log2(L * L)
        bins = (L // 2 + 1) ** 2 + (L // 2 - 1) ** 2
        planes = tiles * (C + K) + (0 if c["how"] == "infer" else J * (C + K) if J else C * K)
        flops = planes * fft + 6.0 * bins * tiles * C * K
        if train:
            flops = 2 * tiles * (C + K) * fft + 2 * C * K * fft + 18.0 * bins * tiles * C * K
        if J:
            flops += 6.0 * bins * C * J * K
        best = flops if best is None else min(best, flops)
        L *= 2
    return {"bytes": float(nbytes), "flops": float(best)}


def tolerance(case):
    # float32 transforms and sums: 1e-7 to 8e-7 was measured against exact()
    # over the listed and drawn cases, the most for weight gradients over many tiles
    return {"rel": 3e-6, "max": 3e-5}


def exact(case, seed):
    """Whole-plane Fourier transforms in float64: circular convolutions of side
    N, whose valid part, and whose adjoints, have no wrapped terms."""
    c = case
    x, ws, g = _inputs(c, seed)
    N, n = c["N"], c["n"]
    M = N - n + 1

    def spectra(t):  # [a, b, s, s] -> bins first, [bins, a, b]
        z = torch.fft.rfft2(t.double(), s=(N, N))
        return z.flatten(2).permute(2, 0, 1).contiguous()

    def plane(z):
        bins = N // 2 + 1
        return torch.fft.irfft2(z.permute(1, 2, 0).contiguous().unflatten(2, (N, bins)), s=(N, N))

    def product(a, b):  # per bin, a few at a time
        out = torch.empty((a.shape[0], a.shape[1], b.shape[2]), dtype=a.dtype, device=a.device)
        step = max(1, (1 << 26) // max(1, a.shape[1] * a.shape[2] + b.shape[1] * b.shape[2]))
        for f in range(0, a.shape[0], step):
            torch.matmul(a[f:f + step].contiguous().resolve_conj(), b[f:f + step].contiguous().resolve_conj(),
                         out=out[f:f + step])
        return out

    W = spectra(ws[0])
    if c["how"] == "chain":
        W = product(spectra(ws[1]), W)
    X = spectra(x)
    out = {"y": plane(product(X, W.transpose(1, 2)))[..., n - 1:, n - 1:].contiguous()}
    if g is not None:
        G = spectra(g)  # M <= N: zero-padded
        # dx[p] = sum w[u] g[p - (n-1) + u]: the correlation rotated by n - 1
        full = plane(product(G, W.conj()))
        out["dx"] = torch.roll(full, (n - 1, n - 1), (2, 3)).contiguous()
        # dw[u] = sum g[i] x[i + n - 1 - u]: the correlation of x with g at lag n - 1 - u
        lag = plane(product(G.conj().transpose(1, 2), X))[..., :n, :n]
        out["dw"] = lag.flip(2, 3).contiguous()
    return out
