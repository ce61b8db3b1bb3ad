"""Workloads that measure the library through its public Python entry points.

Every case is a call, or the few calls, that a program makes once its inputs
are on the GPU.  The sizes are those of the repository's own workloads
(synth/, bench.py, tests/): one 4096^2 image at N = 32, an 8192^2 uint16 band
of a multispectral stack, 4096 tiles of 32 to 512 pixels a side, the request
stream of the server (crops, N from 8 to 256, subsets of twelve offsets), the
histogram, and the statistics of many small or a few large matrices.

    listed()            the fixed cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs, plan and handle, on the GPU
    run(state)          one pass; its outputs, whole
    work(case)          bytes and operations a pass cannot do without
    exact(case, seed)   the same outputs in 64 bits from plain torch / numpy
"""

import math

import numpy as np
import torch

import paper_1710_06189_amd as G

# The four directions of a distance d: 0, 45, 90 and 135 degrees.
_UNIT = ((1, 0), (-1, 1), (0, 1), (1, 1))


def _offsets(mask):
    """Offsets of the twelve (d in {1, 2, 4} x four directions) whose bit is set."""
    every = [(ux * d, uy * d) for d in (1, 2, 4) for ux, uy in _UNIT]
    return [o for b, o in enumerate(every) if mask >> b & 1]


def listed():
    return [
        # one small tile and its statistics: what a call costs when the image
        # is nothing (latency, launches)
        dict(name="tile_64", kind="image", W=64, H=64, u16=False, N=16, lo=0, hi=255, mask=0b1111, content="smooth",
             sigma=4.0, crop=False, tuned=False, features=True),
        # served requests: a crop of a larger image (row base off the 16-byte
        # grid), a subset of the twelve offsets, with statistics
        dict(name="crop_n16_noise", kind="image", W=2937, H=3015, u16=False, N=16, lo=0, hi=255, mask=0b000111010111,
             content="noise", sigma=0.0, crop=True, tuned=False, features=True),
        dict(name="crop_n64_smooth", kind="image", W=1531, H=1489, u16=False, N=64, lo=0, hi=255, mask=0b101101001011,
             content="smooth", sigma=8.0, crop=True, tuned=False, features=True),
        # the reference square image at N = 32, four directions: smooth, on a
        # tuned plan as bench.py runs it, and noise on the plan as created
        dict(name="square_smooth", kind="image", W=4096, H=4096, u16=False, N=32, lo=0, hi=255, mask=0b1111,
             content="smooth", sigma=8.0, crop=False, tuned=True, features=False),
        dict(name="square_uniform", kind="image", W=4096, H=4096, u16=False, N=32, lo=0, hi=255, mask=0b1111,
             content="noise", sigma=0.0, crop=False, tuned=False, features=False),
        # one band of the multispectral stack: the largest image, 16-bit
        # pixels, all twelve offsets
        dict(name="band_u16", kind="image", W=8192, H=8192, u16=True, N=64, lo=0, hi=65535, mask=0b111111111111,
             content="band", sigma=13.8, crop=False, tuned=False, features=False),
        # many levels: the matrices of the twelve offsets exceed the LDS
        dict(name="large_n", kind="image", W=4096, H=4096, u16=False, N=256, lo=0, hi=255, mask=0b111111111111,
             content="smooth", sigma=8.0, crop=False, tuned=False, features=False),
        # thousands of tiles in one launch, with statistics
        dict(name="batch_tiles", kind="batch", T=4096, smin=32, smax=512, u16=False, N=16, lo=0, hi=255, mask=0b1111,
             prepared=False),
        # the quantized histogram of the square image
        dict(name="histogram", kind="histogram", W=4096, H=4096, u16=False, N=32, lo=0, hi=255, content="smooth",
             sigma=8.0, crop=False),
        # post-processing of a batch's matrices: symmetric matrices, their
        # Haralick statistics, the mean over each image's four directions
        dict(name="haralick_batch", kind="stats", K=16384, N=16),
        # the maximal correlation coefficient of a batch's matrices
        dict(name="mcc_batch", kind="mcc", K=16384, N=16),
        # post-processing of the twelve large matrices of one image
        dict(name="stats_n256", kind="stats", K=12, N=256),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def _range(rng, u16):
    """Quantization range: the whole type, or a window of it."""
    top = 65535 if u16 else 255
    if rng.random() < 0.7:
        return 0, top
    lo = rng.randrange(0, top // 4)
    return lo, rng.randrange(top // 2, top + 1)


def draw(rng):
    kind = rng.choice(["image", "image", "image", "batch", "histogram", "stats", "mcc"])
    if kind in ("image", "histogram"):
        u16 = rng.random() < 0.3
        W, H = _log(rng, 40, 8192), _log(rng, 40, 8192)
        lo, hi = _range(rng, u16)
        c = dict(kind=kind, W=W, H=H, u16=u16, lo=lo, hi=hi, content=rng.choice(["smooth", "smooth", "noise", "noise", "band"]),
                 sigma=round(rng.uniform(2.0, 16.0), 2), crop=rng.random() < 0.5)
        if kind == "histogram":
            return dict(c, N=rng.choice([8, 16, 32, 100, 256, 1000]))
        N = rng.choice([8, 16, 32, 64, 256, rng.randrange(4, 65), rng.randrange(65, 1025)])
        mask = rng.randrange(1, 4096)
        if N > 64:  # the largest of these cost what the listed one does
            c["W"], c["H"] = min(W, 4096), min(H, 4096)
            while N > 256 and len(_offsets(mask)) > 2:
                mask &= mask - 1
        return dict(c, N=N, mask=mask, tuned=False, features=rng.random() < 0.5)
    if kind == "batch":
        u16 = rng.random() < 0.3
        lo, hi = _range(rng, u16)
        mask = 0
        while not 1 <= len(_offsets(mask)) <= 4:
            mask = rng.randrange(1, 256)  # d = 1 and 2: what a batch takes
        return dict(kind=kind, T=_log(rng, 8, 3000), smin=32, smax=rng.randrange(64, 513), u16=u16,
                    N=rng.choice([8, 16, 32, rng.randrange(4, 41)]), lo=lo, hi=hi, mask=mask,
                    prepared=rng.random() < 0.5)
    if kind == "stats":
        N = rng.choice([8, 16, 32, 64, rng.randrange(4, 300), rng.randrange(65, 300)])
        most = max(8, min(16384, (1 << 20) // (N * N)))
        return dict(kind=kind, K=4 * max(1, _log(rng, 4, most) // 4), N=N)
    N = rng.choice([8, 16, 32, rng.randrange(3, 49)])
    return dict(kind=kind, K=_log(rng, 4, max(8, min(16384, (1 << 24) // N ** 3))), N=N)


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _field(h, w, sigma, g):
    """Gaussian noise blurred with a Gaussian of std sigma pixels, in [0, 1]."""
    H, W = -(-h // 64) * 64, -(-w // 64) * 64
    z = torch.randn((H, W), generator=g, device="cuda")
    fy = torch.fft.fftfreq(H, device="cuda")[:, None]
    fx = torch.fft.rfftfreq(W, device="cuda")[None, :]
    z = torch.fft.irfft2(torch.fft.rfft2(z) * torch.exp((-2.0 * math.pi ** 2 * sigma * sigma) * (fx * fx + fy * fy)),
                         s=(H, W))[:h, :w]
    lo, hi = z.min(), z.max()
    return (z - lo) / (hi - lo)


def _pixels(h, w, u16, content, sigma, g):
    top = 65535 if u16 else 255
    if content == "noise":
        v = torch.randint(0, top + 1, (h, w), generator=g, device="cuda", dtype=torch.int32)
    else:
        v = _field(h, w, sigma, g) * top
        if content == "band":  # a spectral band: the field plus noise of 5 % of the range
            v += torch.randn((h, w), generator=g, device="cuda") * (0.05 * top)
        v = v.round_().clamp_(0, top).to(torch.int32)
    return v.to(torch.uint16 if u16 else torch.uint8)


def _image(case, seed):
    """The image; a crop is a view of a larger one, off the 16-byte grid."""
    h, w = case["H"], case["W"]
    g = _gen(seed)
    if not case["crop"]:
        return _pixels(h, w, case["u16"], case["content"], case["sigma"], g)
    return _pixels(h + 8, w + 21, case["u16"], case["content"], case["sigma"], g)[3:3 + h, 5:5 + w]


def _tiles(case, seed):
    """T tiles, sides log-uniform: the first half noise, the others smooth."""
    rng = np.random.Generator(np.random.PCG64(seed))
    sides = np.floor(np.exp(rng.uniform(math.log(case["smin"]), math.log(case["smax"] + 1), size=(case["T"], 2)))).astype(int)
    g = _gen(seed)
    big = [_pixels(2048, 2048, case["u16"], c, 4.0, g) for c in ("noise", "smooth")]
    tiles = []
    for t in range(case["T"]):
        h, w = int(sides[t, 0]), int(sides[t, 1])
        y, x = int(rng.integers(0, 2049 - h)), int(rng.integers(0, 2049 - w))
        tiles.append(big[2 * t >= case["T"]][y:y + h, x:x + w].contiguous())
    order = rng.permutation(case["T"])
    return [tiles[i] for i in order]


def _counts(case, seed):
    """K matrices of N x N counts concentrated along the diagonal, as images
    give them; pairs per matrix log-uniform, one matrix in 64 empty."""
    K, N = case["K"], case["N"]
    g = _gen(seed)
    u = torch.rand((K, 2), generator=g, device="cuda", dtype=torch.float64)
    T = torch.exp(math.log(3000.0) + u[:, 0] * math.log(260000.0 / 3000.0)) * max(1.0, N * N / 256.0)
    s = (0.3 + u[:, 1] * 5.7) * max(1.0, N / 16.0)
    d = (torch.arange(N, device="cuda")[:, None] - torch.arange(N, device="cuda")[None, :]).double()
    shape = torch.exp(-(d * d) / (2.0 * s[:, None, None] ** 2))
    lam = shape / shape.sum((1, 2), keepdim=True) * T[:, None, None]
    P = torch.poisson(lam.float(), generator=g).to(torch.int64).to(torch.int32)
    if K >= 64:
        P[63::64] = 0
    return P


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("image", "histogram"):
        img = _image(case, seed)
        state = dict(case=case, img=img)
        if kind == "image":
            offs = _offsets(case["mask"])
            plan = G.glcm_plan_create(img.dtype, case["N"], offs, case["W"], case["H"])
            if case["tuned"]:
                plan.autotune(img, case["lo"], case["hi"])
            state.update(offsets=offs, plan=plan)
        return state
    if kind == "batch":
        tiles = _tiles(case, seed)
        plan = G.glcm_plan_create(tiles[0].dtype, case["N"], _offsets(case["mask"]), case["smax"], case["smax"])
        batch = G.PreparedBatch(tiles, plan) if case["prepared"] else G.prepare_tiles(tiles, plan)
        return dict(case=case, plan=plan, batch=batch)
    return dict(case=case, P=_counts(case, seed).view(torch.uint32))


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "image":
        P = G.glcm_compute(state["img"], c["N"], c["lo"], c["hi"], state["offsets"], plan=state["plan"])
        return [P, G.glcm_features(P)] if c["features"] else [P]
    if kind == "histogram":
        return [G.glcm_histogram(state["img"], c["N"], c["lo"], c["hi"])]
    if kind == "batch":
        if c["prepared"]:
            P, F = state["batch"].run(c["lo"], c["hi"], features=True)
        else:
            P, F = G.glcm_batch_compute(state["batch"], state["plan"], c["lo"], c["hi"])
        return [P.view(torch.int32), F]  # (torch indexes no uint32 tensors)
    P = state["P"]
    if kind == "mcc":
        return [G.glcm_haralick_mcc(P)]
    S = G.glcm_symmetrize(P)
    out = [S.view(torch.int32), G.glcm_haralick(S), G.glcm_average(P, 4)]
    if c["K"] <= 64:  # one image's matrices: also the five statistics and the probabilities
        out += [G.glcm_features(P), G.glcm_normalize(P)]
    return out


def work(case):
    kind, N = case["kind"], case["N"]
    if kind in ("image", "histogram"):
        pixels = case["W"] * case["H"]
        b = pixels * (2 if case["u16"] else 1)
        if kind == "histogram":
            return dict(bytes=b + 4 * N, flops=pixels)
        offs = _offsets(case["mask"])
        pairs = sum(max(0, case["W"] - abs(dx)) * max(0, case["H"] - abs(dy)) for dx, dy in offs)
        return dict(bytes=b + len(offs) * (4 * N * N + (20 if case["features"] else 0)), flops=pairs)
    if kind == "batch":
        K = len(_offsets(case["mask"]))
        side = (case["smax"] - case["smin"]) / math.log(case["smax"] / case["smin"])  # mean of a log-uniform side
        pixels = case["T"] * side * side
        return dict(bytes=pixels * (2 if case["u16"] else 1) + case["T"] * K * (4 * N * N + 20), flops=K * pixels)
    K, words = case["K"], case["K"] * N * N
    if kind == "mcc":
        # S = B B^T (symmetric) and the reduction of S to tridiagonal form
        return dict(bytes=4 * words + 4 * K, flops=K * (N ** 3 + 4 * N ** 3 / 3))
    # symmetrize (read, write), Haralick (read), average (read, write a
    # quarter); with few matrices also features (read), normalize (read, write)
    per = 4 * words * (2 + 1 + 1.25) + 52 * K
    if K <= 64:
        per += 4 * words * 3 + 20 * K
    return dict(bytes=per, flops=30 * words)


# --------------------------------------------------------------------------
# The same outputs in 64 bits
# --------------------------------------------------------------------------

def _levels(img, N, lo, hi):
    v = img.to(torch.int32).to(torch.int64)
    q = ((v - lo) * N).div(hi - lo + 1, rounding_mode="floor")
    return torch.where(v < lo, 0, torch.where(v > hi, N - 1, q))


def _glcm(img, N, lo, hi, offsets):
    L = _levels(img, N, lo, hi)
    h, w = L.shape
    out = []
    for dx, dy in offsets:
        if abs(dx) >= w or abs(dy) >= h:
            out.append(torch.zeros((N, N), dtype=torch.int64, device=L.device))
            continue
        y0, y1, x0, x1 = max(0, -dy), h - max(0, dy), max(0, -dx), w - max(0, dx)
        pair = L[y0:y1, x0:x1] * N + L[y0 + dy:y1 + dy, x0 + dx:x1 + dx]
        out.append(torch.bincount(pair.reshape(-1), minlength=N * N).reshape(N, N))
    return torch.stack(out)


def _xlogx(p):
    return torch.where(p > 0, p * torch.log(torch.where(p > 0, p, 1.0)), 0.0)


def _prob(P):
    P = P.double()
    T = P.sum((-2, -1), keepdim=True)
    return torch.where(T > 0, P / torch.where(T > 0, T, 1.0), 0.0), T[..., 0, 0] > 0


def _correlation(p, px, py, n):
    mx, my = (px * n).sum(-1), (py * n).sum(-1)
    vx = (px * (n - mx[..., None]) ** 2).sum(-1)
    vy = (py * (n - my[..., None]) ** 2).sum(-1)
    cov = (p * (n[:, None] - mx[..., None, None]) * (n[None, :] - my[..., None, None])).sum((-2, -1))
    one = ((px > 0).sum(-1) == 1) | ((py > 0).sum(-1) == 1)
    return torch.where(one, 1.0, cov / torch.sqrt(torch.where(one, 1.0, vx * vy))), vx


def _features(P):
    p, some = _prob(P)
    n = torch.arange(P.shape[-1], device=P.device, dtype=torch.float64)
    d2 = (n[:, None] - n[None, :]) ** 2
    corr, _ = _correlation(p, p.sum(-1), p.sum(-2), n)
    f = torch.stack([(p * d2).sum((-2, -1)), (p * p).sum((-2, -1)), -_xlogx(p).sum((-2, -1)),
                     (p / (1.0 + d2)).sum((-2, -1)), corr], -1)
    return torch.where(some[..., None], f, 0.0)


def _haralick(P):
    N = P.shape[-1]
    p, some = _prob(P)
    n = torch.arange(N, device=P.device, dtype=torch.float64)
    d2 = (n[:, None] - n[None, :]) ** 2
    i, j = torch.meshgrid(torch.arange(N, device=P.device), torch.arange(N, device=P.device), indexing="ij")
    flat = p.reshape(-1, N * N)
    ps = torch.zeros((flat.shape[0], 2 * N - 1), dtype=torch.float64, device=P.device)
    pd = torch.zeros((flat.shape[0], N), dtype=torch.float64, device=P.device)
    ps.index_add_(1, (i + j).reshape(-1), flat)
    pd.index_add_(1, (i - j).abs().reshape(-1), flat)
    t = torch.arange(2 * N - 1, device=P.device, dtype=torch.float64)
    px, py = p.sum(-1), p.sum(-2)
    corr, vx = _correlation(p, px, py, n)
    sa, da = (ps * t).sum(-1), (pd * n).sum(-1)
    ent, hx, hy = -_xlogx(p).sum((-2, -1)), -_xlogx(px).sum(-1), -_xlogx(py).sum(-1)
    q = px[:, :, None] * py[:, None, :]
    lq = torch.log(torch.where(q > 0, q, 1.0))
    hxy1, hxy2 = -(p * lq).sum((-2, -1)), -(q * lq).sum((-2, -1))
    hmax = torch.maximum(hx, hy)
    f = torch.stack([
        (p * p).sum((-2, -1)), (p * d2).sum((-2, -1)), corr, vx, (p / (1.0 + d2)).sum((-2, -1)), sa,
        (ps * (t - sa[:, None]) ** 2).sum(-1), -_xlogx(ps).sum(-1), ent, (pd * (n - da[:, None]) ** 2).sum(-1),
        -_xlogx(pd).sum(-1), torch.where(hmax > 0, (ent - hxy1) / torch.where(hmax > 0, hmax, 1.0), 0.0),
        torch.sqrt(torch.clamp(-torch.expm1(-2.0 * (hxy2 - ent)), min=0.0))], -1)
    return torch.where(some[:, None], f, 0.0)


def _mcc(P):
    """The second singular value of p(i, j) / sqrt(px(i) py(j))."""
    p, some = _prob(P)
    r = p.sum(-1, keepdim=True) * p.sum(-2, keepdim=True)
    B = torch.where(r > 0, p / torch.sqrt(torch.where(r > 0, r, 1.0)), 0.0)
    if P.shape[-1] == 1:
        return torch.zeros(P.shape[0], dtype=torch.float64)
    sv = torch.from_numpy(np.linalg.svd(B.cpu().numpy(), compute_uv=False)[:, 1])
    return torch.where(some.cpu(), sv, 0.0)


def exact(case, seed):
    kind, N = case["kind"], case["N"]
    if kind == "image":
        P = _glcm(_image(case, seed), N, case["lo"], case["hi"], _offsets(case["mask"]))
        return [P, _features(P)] if case["features"] else [P]
    if kind == "histogram":
        return [torch.bincount(_levels(_image(case, seed), N, case["lo"], case["hi"]).reshape(-1), minlength=N)]
    if kind == "batch":
        offs = _offsets(case["mask"])
        P = torch.stack([_glcm(t, N, case["lo"], case["hi"], offs) for t in _tiles(case, seed)])
        return [P, _features(P)]
    P = _counts(case, seed).to(torch.int64)
    if kind == "mcc":
        return [_mcc(P)]
    S = P + P.transpose(-1, -2)
    p, _ = _prob(P)
    out = [S, _haralick(S), p.reshape(-1, 4, N, N).mean(1)]
    return out + [_features(P), p] if case["K"] <= 64 else out
