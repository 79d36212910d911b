"""Performance cases of the digital shearlet transform on one GPU.

What a program built on this package runs, through the package's public entry
points (binding.System, binding.Shrinkage, binding.Multi): the analysis and
synthesis of image batches and volumes in every storage type, hard-threshold
synthesis from stored coefficients, the fused denoiser, the learned denoiser,
the training step of its network, and an uneven batch replayed from its graph.

A case is a dict of plain values.  listed() names the fixed ones, draw(rng)
gives others of the same ranges, prepare(case, seed) makes what the program
holds before the call, run(state) makes one pass, work(case) counts the bytes
and operations a pass cannot do without, and exact(case, seed) evaluates the
same outputs in 64 bits from the definitions, without the package's code.
"""
import math

import numpy as np
import torch

from paper_1402_5670_amd import binding

DEVICE = "cuda:0"
SIGMAS = (20.0 / 255.0, 30.0 / 255.0, 40.0 / 255.0)
PARAMS = binding.CNN_PARAMS


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # one thumbnail, analysed and reconstructed: the smallest call, where
        # launches and latency count
        dict(name="image_64", kind="transform", dims="64,64", levels="1,1,2", batch=1, dtype="f32"),
        # an odd number of small ragged images with half-precision storage
        dict(name="ragged_3x96x384_f16", kind="transform", dims="96,384", levels="1,1,2", batch=3,
             dtype="f16"),
        # a batch of quarter-size images, bfloat16 storage
        dict(name="batch_16x256_bf16", kind="transform", dims="256,256", levels="1,1,2,2",
             batch=16, dtype="bf16"),
        # the benchmark batch, analysis only: float32 coefficients out
        dict(name="analysis_32x512", kind="forward", dims="512,512", levels="1,1,2,2", batch=32,
             dtype="f32"),
        # the benchmark batch, synthesis: stored coefficients hard-thresholded
        # on load and reconstructed
        dict(name="synthesis_32x512", kind="threshold", dims="512,512", levels="1,1,2,2", batch=32,
             dtype="f32"),
        # large images with half-precision storage
        dict(name="large_6x1024_f16", kind="transform", dims="1024,1024", levels="1,1,2", batch=6,
             dtype="f16"),
        # one image denoised interactively, coefficients never stored
        dict(name="denoise_512", kind="denoise", dims="512,512", levels="1,1,2,2", batch=1,
             dtype="f32"),
        # a volume, analysed and reconstructed
        dict(name="volume_128", kind="transform", dims="128,128,128", levels="1,1", batch=1,
             dtype="f32"),
        # a video volume with the large system (R = 292): the largest tensors
        dict(name="video_192", kind="transform", dims="192,192,192", levels="1,1,2", batch=1,
             dtype="f32"),
        # the learned denoiser on a batch
        dict(name="learned_8x512", kind="learned", dims="512,512", levels="1,1,2,2", batch=8,
             dtype="f32"),
        # one training step of its network, up to the gradients
        dict(name="train_4x512", kind="train", dims="512,512", levels="1,1,2,2", batch=4,
             dtype="f32"),
        # images of four sizes in one captured graph, half-precision storage
        dict(name="uneven_19_f16", kind="uneven", sizes="256,384,512,1024", counts="5,6,2,6",
             levels="1,1,2", dtype="f16"),
    ]


# the largest drawn cases stay below the listed ones
MOST_COEFFS = 32 * 49 * 512 * 512
SIDES = (64, 96, 128, 192, 256, 384, 512, 768, 1024)


def _count(levels, ndim):
    r = 1
    for d in levels:
        a = 2 * 2 ** d + 1
        r += 2 * a - 2 if ndim == 2 else 3 * a * a - 6 * a + 4
    return r


def draw(rng):
    kind = rng.choice(("transform", "transform", "transform", "forward", "threshold", "denoise",
                       "volume", "volume", "learned", "train", "uneven"))
    if kind == "uneven":
        sizes = sorted(rng.sample((128, 192, 256, 384, 512, 768, 1024), rng.randint(2, 4)))
        counts = []
        for z in sizes:
            most = min(8, MOST_COEFFS // 4 // (33 * z * z))
            counts.append(rng.randint(1, max(1, most)))
        return dict(kind="uneven", sizes=",".join(map(str, sizes)),
                    counts=",".join(map(str, counts)), levels="1,1,2",
                    dtype=rng.choice(("f16", "bf16")))
    if kind == "volume":
        dims = [rng.choice((32, 48, 64, 96, 128, 192)) for _ in range(3)]
        levels = rng.choice(((1, 1), (0, 1), (1, 1, 2))) if min(dims) >= 64 else (1, 1)
        return dict(kind="transform", dims=",".join(map(str, dims)),
                    levels=",".join(map(str, levels)), batch=1, dtype=rng.choice(("f32", "f32", "f16")))
    sides = SIDES if kind not in ("learned", "train") else (64, 96, 128, 192, 256, 384, 512)
    h = rng.choice(sides)
    w = h if rng.random() < 0.5 else rng.choice(sides)
    levels = (1, 1, 2, 2) if rng.random() < 0.5 and min(h, w) >= 128 else (1, 1, 2)
    most = MOST_COEFFS // (_count(levels, 2) * h * w)
    if kind in ("transform", "denoise"):
        most //= 2
    if kind == "learned":
        most //= 4
    if kind == "train":
        most //= 8
    batch = int(round(2.0 ** rng.uniform(0.0, math.log2(max(1, min(64, most))))))
    dtype = rng.choice(("f32", "f16", "bf16")) if kind == "transform" else "f32"
    return dict(kind=kind, dims="%d,%d" % (h, w), levels=",".join(map(str, levels)),
                batch=max(1, batch), dtype=dtype)


def _ints(text):
    return tuple(int(v) for v in text.split(","))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

def _cartoons(dims, batch, seed):
    """Piecewise constant scenes in [0, 1]: twelve random ellipses (ellipsoids)
    on a random background, with Gaussian noise of 20, 30, 40 / 255 in turn.
    Returns (noisy, clean, sigma), float32 on the GPU."""
    g = torch.Generator(device=DEVICE).manual_seed(int(seed) * 7919 + 17)
    n = len(dims)
    one = (batch,) + (1,) * n
    axes = [torch.linspace(0.0, 1.0, d, device=DEVICE).view((1,) * (1 + k) + (d,) + (1,) * (n - 1 - k))
            for k, d in enumerate(dims)]
    clean = torch.rand(one, generator=g, device=DEVICE).expand((batch,) + tuple(dims)).clone()
    for _ in range(12):
        c = [torch.rand(one, generator=g, device=DEVICE) for _ in range(n)]
        r = [0.05 + 0.25 * torch.rand(one, generator=g, device=DEVICE) for _ in range(n)]
        t = math.pi * torch.rand(one, generator=g, device=DEVICE)
        v = torch.rand(one, generator=g, device=DEVICE)
        a, b = axes[-2] - c[-2], axes[-1] - c[-1]
        q = ((torch.cos(t) * a - torch.sin(t) * b) / r[-2]) ** 2 + \
            ((torch.sin(t) * a + torch.cos(t) * b) / r[-1]) ** 2
        if n == 3:
            q = q + ((axes[0] - c[0]) / r[0]) ** 2
        clean = torch.where(q <= 1.0, v, clean)
    sigma = torch.tensor([SIGMAS[k % 3] for k in range(batch)], device=DEVICE)
    noisy = clean + sigma.view(one) * torch.randn(clean.shape, generator=g, device=DEVICE)
    return noisy.contiguous(), clean.contiguous(), sigma


def _network(scales, seed):
    """Weights [J, PARAMS] of the shrinkage network as training meets them: a
    smooth threshold on channel 0 and scaled He weights elsewhere."""
    rng = np.random.default_rng([int(seed), 11])
    out = np.zeros((scales, PARAMS), dtype=np.float32)
    for j in range(scales):
        w1 = rng.standard_normal((32, 2, 3, 3)) * math.sqrt(2.0 / 18) * 0.3
        w2 = rng.standard_normal((32, 32, 3, 3)) * math.sqrt(2.0 / 288) * 0.3
        w3 = rng.standard_normal((1, 32, 3, 3)) * math.sqrt(1.0 / 288) * 0.3
        w1[0] = 0.0
        w1[0, 0, 1, 1] = 1.0
        w2[0] = 0.0
        w2[0, 0, 1, 1] = 1.0
        w3[0, 0] = 0.0
        w3[0, 0, 1, 1] = 3.0
        out[j] = np.concatenate([w1.ravel(), 0.05 * rng.standard_normal(32), w2.ravel(),
                                 0.05 * rng.standard_normal(32), w3.ravel(), [-9.0]])
    return out


def _thresholds(scales):
    return [3.0] * (scales - 1) + [4.0]


# a program builds the system of a size once and keeps it for every batch
_systems = {}


def _system(dims, levels, dtype):
    key = (dims, levels, dtype)
    if key not in _systems:
        while len(_systems) >= 6:
            _systems.pop(next(iter(_systems)))
        _systems[key] = binding.System(dims, len(levels), list(levels), dtype=dtype)
    return _systems[key]


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)


def prepare(case, seed):
    kind, levels = case["kind"], _ints(case["levels"])
    if kind == "uneven":
        sizes, counts = _ints(case["sizes"]), _ints(case["counts"])
        systems = [_system((z, z), levels, case["dtype"]) for z in sizes]
        xs = [_cartoons((z, z), c, 31 * seed + z)[0] for z, c in zip(sizes, counts)]
        buf = [s.alloc_coeffs(c, DEVICE) for s, c in zip(systems, counts)]
        st = dict(kind=kind, xs=xs, coeffs=[b[0] for b in buf], scales=[b[1] for b in buf],
                  outs=[torch.empty_like(x) for x in xs], multi=binding.Multi(systems, counts))
        st["ws"] = _workspace(st["multi"].workspace_bytes())
        st["multi"].graph_build(3, xs, st["coeffs"], st["scales"], outs=st["outs"],
                                workspace=st["ws"])
        return st
    dims, batch = _ints(case["dims"]), int(case["batch"])
    s = _system(dims, levels, case["dtype"])
    x, clean, sigma = _cartoons(dims, batch, seed)
    st = dict(kind=kind, sys=s, x=x, sigma=sigma, K=_thresholds(len(levels)),
              out=torch.empty_like(x))
    if kind == "threshold":
        st["coeffs"] = _stored_coefficients(case, x)
        st["ws"] = _workspace(s.workspace_bytes(batch))
        return st
    if kind != "denoise":
        st["coeffs"], st["scales"] = s.alloc_coeffs(batch, DEVICE)
    if kind in ("learned", "train"):
        params = torch.from_numpy(_network(len(levels), seed)).to(DEVICE)
        st["net"] = binding.Shrinkage(s, params)
    if kind == "learned":
        st["ws"] = _workspace(s.denoise_workspace_bytes(batch, True))
    else:
        st["ws"] = _workspace(s.workspace_bytes(batch))
    if kind == "train":
        st["clean"] = clean
        st["shrunk"] = torch.empty_like(st["coeffs"])
        st["dcoeffs"] = torch.empty_like(st["coeffs"])
        st["resid"] = torch.empty_like(x)
        st["grads"] = torch.empty_like(st["net"].params)
        st["scratch"] = torch.zeros(binding.SQERR_SCRATCH, device=DEVICE)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(st):
    kind = st["kind"]
    if kind == "uneven":
        st["multi"].graph_launch()
        return dict(coeffs=st["coeffs"], scales=st["scales"], outs=st["outs"])
    s, ws = st["sys"], st["ws"]
    if kind == "transform":
        s.forward(st["x"], st["coeffs"], st["scales"], workspace=ws)
        s.inverse(st["coeffs"], st["scales"], out=st["out"], workspace=ws)
        if s.dtype == "f32":
            return dict(coeffs=st["coeffs"], out=st["out"])
        return dict(coeffs=st["coeffs"], scales=st["scales"], out=st["out"])
    if kind == "forward":
        s.forward(st["x"], st["coeffs"], st["scales"], workspace=ws)
        return dict(coeffs=st["coeffs"])
    if kind == "threshold":
        s.inverse(st["coeffs"], None, sigma=st["sigma"], K=st["K"], out=st["out"], workspace=ws)
        return dict(out=st["out"])
    if kind == "denoise":
        s.denoise_fused(st["x"], st["sigma"], st["K"], out=st["out"], workspace=ws)
        return dict(out=st["out"])
    if kind == "learned":
        s.denoise(st["x"], st["sigma"], coeffs=st["coeffs"], scales=st["scales"], out=st["out"],
                  workspace=ws, model=st["net"])
        return dict(coeffs=st["coeffs"], out=st["out"])
    # a training step: noisy image -> coefficients -> gains -> reconstruction
    # -> squared error -> gradients of the network's weights
    net = st["net"]
    s.forward(st["x"], st["coeffs"], st["scales"], workspace=ws)
    net.apply(st["coeffs"], st["sigma"], out=st["shrunk"])
    s.inverse(st["shrunk"], out=st["out"], workspace=ws)
    binding.sq_error_grad(st["out"], st["clean"], 2.0 / st["x"].numel(), st["resid"], st["scratch"])
    s.inverse_adjoint(st["resid"], coeffs=st["dcoeffs"], workspace=ws)
    net.backward(st["coeffs"], st["sigma"], st["dcoeffs"], grads=st["grads"])
    return dict(grads=st["grads"], out=st["out"], loss=st["scratch"][0])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

CODE_BYTES = {"f32": 4, "f16": 2, "bf16": 2}
NET_FLOPS = 2 * (9 * 2 * 32 + 9 * 32 * 32 + 9 * 32)     # per coefficient, forward


def _transform_work(dims, levels, batch, cb, directions):
    n, r = math.prod(dims), _count(levels, len(dims))
    table = 4 * n * (r if len(dims) == 2 else 1)
    coeffs = batch * r * n
    # one real transform per signal and per subband, one product per sample
    flops = directions * batch * (r + 1) * (2.5 * n * math.log2(n) + 4 * n)
    return directions * (coeffs * cb + 4 * batch * n) + table, flops


def work(case):
    kind, levels = case["kind"], _ints(case["levels"])
    cb = CODE_BYTES[case["dtype"]]
    if kind == "uneven":
        parts = [_transform_work((z, z), levels, c, cb, 2)
                 for z, c in zip(_ints(case["sizes"]), _ints(case["counts"]))]
        return dict(bytes=sum(p[0] for p in parts), flops=sum(p[1] for p in parts))
    dims, batch = _ints(case["dims"]), int(case["batch"])
    by, fl = _transform_work(dims, levels, batch, cb, 2 if kind == "transform" else 1)
    n, r = math.prod(dims), _count(levels, len(dims))
    signal, coeffs = 4 * batch * n, 4 * batch * r * n
    detail = batch * (r - 1) * n
    if kind == "denoise":
        # image in, image out, filters once
        by, fl = 2 * signal + 4 * n * r, 2 * fl
    if kind == "learned":
        by, fl = by + signal, 2 * fl + detail * NET_FLOPS
    if kind == "train":
        # images in, reconstruction out, filters once; the network forward and
        # its two backward products, three transforms of the subbands
        by, fl = 3 * signal + 4 * n * r, 3 * fl + 3 * detail * NET_FLOPS
    return dict(bytes=by, flops=fl)


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------

def _qmf():
    """h0..h4 of the symmetric maximally flat 9-tap lowpass: H(0) = 1,
    H(pi) = 0, H''(0) = H''''(0) = 0, H(pi / 2) = 1 / sqrt(2)."""
    n = np.arange(1, 5, dtype=np.float64)
    rows = [np.r_[1.0, 2.0 * np.ones(4)], np.r_[1.0, 2.0 * (-1.0) ** n], np.r_[0.0, n ** 2],
            np.r_[0.0, n ** 4], np.r_[1.0, 2.0 * np.cos(n * np.pi / 2.0)]]
    return np.linalg.solve(np.array(rows), np.array([1.0, 0.0, 0.0, 0.0, math.sqrt(0.5)]))


_TAPS = _qmf()


def _H(xi):
    return _TAPS[0] + 2.0 * sum(_TAPS[k] * torch.cos(2.0 * math.pi * k * xi) for k in range(1, 5))


def _low(xi, order):
    out = torch.ones_like(xi)
    for k in range(order):
        out = out * _H(xi * 2 ** k)
    return out


def _high(xi, order):
    return _H(xi * 2 ** (order - 1) + 0.5) * _low(xi, order - 1)


def _fan(e1, e2):
    x = 0.5 * (torch.cos(2.0 * math.pi * e2) - torch.cos(2.0 * math.pi * e1))
    return (1.0 + x) ** 2 * (2.0 - x) / 4.0


def _freqs(n):
    return torch.arange(n, dtype=torch.float64, device=DEVICE) / n


def _sheared(main, sec, scales, j, d, k, wedge):
    """Digital shear by k / 2^d of the scale-j wedge (with the main-axis
    highpass, 2D) or of its 3D plane factor, on the frequency grid
    sec x main: upsampling, interpolation filter, integer shear and
    downsampling along the main axis become a sum over the aliases."""
    L = 2 ** d
    m, s = main[None, :], sec[:, None]
    out = torch.zeros(len(sec), len(main), dtype=torch.float64, device=DEVICE)
    for l in range(L):
        t = (m + l) / L
        interp = torch.ones_like(t)
        for q in range(d):
            interp = interp * (2.0 * _H(t * 2 ** q) ** 2)
        y = s - k * t
        v = _fan(2 ** (scales - j - 1) * m, 2 ** (scales - j + d) * y) * _low(y, scales - j + d)
        out += interp * v
    out /= L
    return out * _high(m, scales - j) if wedge else out


def _filters2d(dims, levels):
    """psi_hat of every subband in order: (j, values), j = -1 for the lowpass."""
    J = len(levels)
    f2, f1 = _freqs(dims[0]), _freqs(dims[1])
    yield -1, _low(f2, J)[:, None] * _low(f1, J)[None, :]
    for j, d in enumerate(levels):
        L = 2 ** d
        for k in range(-L, L + 1):
            yield j, _sheared(f1, f2, J, j, d, k, True)
        for k in range(-L + 1, L):
            yield j, _sheared(f2, f1, J, j, d, k, True).T.contiguous()


def _filters3d(dims, levels):
    J = len(levels)
    f = {1: _freqs(dims[2]), 2: _freqs(dims[1]), 3: _freqs(dims[0])}

    def along(v, axis):
        return v.view([len(v) if a == axis else 1 for a in (3, 2, 1)])

    def plane(p, main, sec):       # p [sec, main] placed on the axes of [3, 2, 1]
        q = p if main < sec else p.T
        return q.reshape([p.shape[1] if a == main else p.shape[0] if a == sec else 1
                          for a in (3, 2, 1)])

    yield -1, along(_low(f[3], J), 3) * along(_low(f[2], J), 2) * along(_low(f[1], J), 1)
    for j, d in enumerate(levels):
        L = 2 ** d
        for pyr, (s1, s2) in ((1, (2, 3)), (2, (1, 3)), (3, (1, 2))):
            g = along(_high(f[pyr], J - j), pyr)
            A = {k: plane(_sheared(f[pyr], f[s1], J, j, d, k, False), pyr, s1)
                 for k in range(-L, L + 1)}
            B = {k: plane(_sheared(f[pyr], f[s2], J, j, d, k, False), pyr, s2)
                 for k in range(-L, L + 1)}
            for k1 in range(-L, L + 1):
                for k2 in range(-L, L + 1):
                    if pyr >= 2 and abs(k1) == L or pyr == 3 and abs(k2) == L:
                        continue
                    yield j, g * A[k1] * B[k2]


def _filters(dims, levels):
    return _filters2d(dims, levels) if len(dims) == 2 else _filters3d(dims, levels)


def _stored_coefficients(case, x):
    """Coefficients [B, R, dims] float32 of x, as an earlier analysis left them."""
    dims, levels = _ints(case["dims"]), _ints(case["levels"])
    axes = tuple(range(1, 1 + len(dims)))
    X = torch.fft.fftn(x, dim=axes)
    c = torch.empty((x.shape[0], _count(levels, len(dims))) + dims, device=DEVICE)
    for i, (_, psi) in enumerate(_filters(dims, levels)):
        c[:, i] = torch.fft.ifftn(X * psi.float(), dim=axes).real
    return c


def _analyse(x, dims, levels, code):
    """Coefficients as stored (float64), storage scales and ||psi||_2."""
    axes = tuple(range(1, 1 + len(dims)))
    X = torch.fft.fftn(x.double(), dim=axes)
    R = _count(levels, len(dims))
    c = torch.empty((x.shape[0], R) + tuple(dims), dtype=torch.float64, device=DEVICE)
    scales = torch.ones(x.shape[0], R, dtype=torch.float64, device=DEVICE)
    top = x.double().abs().flatten(1).amax(1)
    l2 = []
    for i, (_, psi) in enumerate(_filters(dims, levels)):
        for b in range(x.shape[0]):
            c[b, i] = torch.fft.ifftn(X[b] * psi).real
        l2.append(float(psi.square().mean().sqrt()))
        if code != "f32":
            l1 = torch.fft.ifftn(psi.to(torch.complex128)).real.abs().sum()
            scales[:, i] = torch.exp2(torch.ceil(torch.log2(top * l1)) - 15.0)
            c[:, i] /= scales[:, i].view((-1,) + (1,) * len(dims))
    return c, scales, l2


def _synthesise(c, dims, levels):
    axes = tuple(range(1, 1 + len(dims)))
    acc = torch.zeros((c.shape[0],) + tuple(dims), dtype=torch.complex128, device=DEVICE)
    weight = torch.zeros(dims, dtype=torch.float64, device=DEVICE)
    for i, (_, psi) in enumerate(_filters(dims, levels)):
        acc += psi * torch.fft.fftn(c[:, i].double(), dim=axes)
        weight += psi * psi
    return torch.fft.ifftn(acc / weight, dim=axes).real


class _Product(torch.autograd.Function):
    """w [co, ci] times t [ci, N]; the weight gradient as elementwise sums, as
    64-bit products with a long reduction run on one workgroup here."""

    @staticmethod
    def forward(ctx, w, t):
        ctx.save_for_backward(w, t)
        return w @ t

    @staticmethod
    def backward(ctx, d):
        w, t = ctx.saved_tensors
        return torch.stack([(row * t).sum(1) for row in d]), w.T @ d


def _conv(x, w, b):
    """Same-padded 3x3 convolution of [ci, H, W] with w [co, ci, 3, 3]."""
    H, W = x.shape[1:]
    p = torch.nn.functional.pad(x, (1, 1, 1, 1))
    out = b.view(-1, 1)
    for dy in range(3):
        for dx in range(3):
            t = p[:, dy:dy + H, dx:dx + W].reshape(len(x), H * W)
            out = out + _Product.apply(w[:, :, dy, dx], t)
    return out.view(-1, H, W)


def _gain(c, sigma, l2, blob):
    """Gains of one detail plane [H, W] for a weight blob (float64)."""
    w1, b1, w2, b2, w3, b3 = torch.split(blob, [576, 32, 9216, 32, 288, 1])
    x0 = torch.stack([c.abs() / (sigma * l2), torch.full_like(c, sigma * 255.0 / 50.0)])
    h = torch.relu(_conv(x0, w1.view(32, 2, 3, 3), b1))
    h = torch.relu(_conv(h, w2.view(32, 32, 3, 3), b2))
    return torch.sigmoid(_conv(h, w3.view(1, 32, 3, 3), b3))[0]


def _scale_of(levels):
    out = [-1]
    for j, d in enumerate(levels):
        out += [j] * (4 * 2 ** d)
    return out


def _exact_network(case, seed):
    dims, levels, batch = _ints(case["dims"]), _ints(case["levels"]), int(case["batch"])
    x, clean, sigma = _cartoons(dims, batch, seed)
    blobs = torch.from_numpy(_network(len(levels), seed)).to(DEVICE)
    # the network's weights are bfloat16 values by definition, its biases float32
    w = blobs.bfloat16().double()
    for a, n in ((576, 32), (9824, 32), (10144, 1)):
        w[:, a:a + n] = blobs[:, a:a + n].double()
    blobs = w
    c, _, l2 = _analyse(x, dims, levels, "f32")
    jof, sg = _scale_of(levels), [float(v) for v in sigma]
    shrunk = c.clone()
    for b in range(batch):
        for i in range(1, c.shape[1]):
            shrunk[b, i] = c[b, i] * _gain(c[b, i], sg[b], l2[i], blobs[jof[i]])
    out = _synthesise(shrunk, dims, levels)
    if case["kind"] == "learned":
        return dict(coeffs=c, out=out)
    del shrunk
    err = out - clean.double()
    # gradient of the mean squared error through the reconstruction: forward
    # transform with the dual filters
    filt = list(_filters(dims, levels))
    weight = sum(psi * psi for _, psi in filt)
    Rf = torch.fft.fftn(err * (2.0 / x.numel()), dim=(1, 2)) / weight
    grads = torch.zeros_like(blobs)
    for b in range(batch):
        for i in range(1, c.shape[1]):
            dc = torch.fft.ifftn(Rf[b] * filt[i][1]).real
            blob = blobs[jof[i]].clone().requires_grad_(True)
            shr = c[b, i] * _gain(c[b, i], sg[b], l2[i], blob)
            grads[jof[i]] += torch.autograd.grad((shr * dc).sum(), blob)[0]
    return dict(grads=grads, out=out, loss=err.square().sum())


def exact(case, seed):
    kind, levels = case["kind"], _ints(case["levels"])
    if kind == "denoise":
        return None        # keeps or drops a coefficient by a comparison: no value near a tie
    if kind == "uneven":
        cs, ss, outs = [], [], []
        for z, n in zip(_ints(case["sizes"]), _ints(case["counts"])):
            x = _cartoons((z, z), n, 31 * seed + z)[0]
            c, s, _ = _analyse(x, (z, z), levels, case["dtype"])
            cs.append(c)
            ss.append(s)
            outs.append(x.double())
        return dict(coeffs=cs, scales=ss, outs=outs)
    if kind in ("learned", "train"):
        planes = int(case["batch"]) * (_count(levels, 2) - 1)
        return _exact_network(case, seed) if planes <= 400 else None    # about 20 s
    dims, batch = _ints(case["dims"]), int(case["batch"])
    x, _, sigma = _cartoons(dims, batch, seed)
    if kind == "threshold":
        c = _stored_coefficients(case, x)
        K = torch.tensor(_thresholds(len(levels)), dtype=torch.float32, device=DEVICE)
        for i, (j, psi) in enumerate(_filters(dims, levels)):
            if j >= 0:       # the float32 comparison that defines the threshold
                delta = (K[j] * sigma) * psi.square().mean().sqrt().float()
                c[:, i] *= c[:, i].abs() >= delta.view((-1,) + (1,) * len(dims))
        return dict(out=_synthesise(c, dims, levels))
    # the dual frame reconstructs what it analysed
    three = len(dims) == 3
    c, s, _ = _analyse(x, dims, levels, "f32" if three else case["dtype"])
    if kind == "forward":
        return dict(coeffs=c)
    if case["dtype"] == "f32":
        return dict(coeffs=c, out=x.double())
    if three:                # the storage scale of a volume rests on a bound of ||psi||_1
        return dict(coeffs=None, scales=None, out=x.double())
    return dict(coeffs=c, scales=s, out=x.double())
