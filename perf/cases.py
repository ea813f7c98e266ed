"""The work that users of libfb have it do, as cases that can be timed and checked.

A case is a dict of plain values.  `kind` says which calls it makes:

  transform  fb_fft3d_exec, forward into a second grid and inverse back,
             or the forward transform alone
  block      the spectral block: a forward transform, then `steps` fused
             steps (evolve, inverse, checksum) into one output grid
  steps      one serving request's device work: forward transform of a
             generated input, then all steps from one fb_spectral_steps call
  batch      fb_batch_exec, many 1D lengths and some 2D transforms at once
  lu         fb_lu_factor

All of it runs through the public binding (paper_2004_09883_amd.fb).  Inputs
come from torch's generator on the device, seeded; grids are N(0, 1) or
U[-1, 1) as in the block's workloads.
"""
import math

import torch

from paper_2004_09883_amd import fb, inputs

DTYPES = {"c128": fb.FB_C128, "c64": fb.FB_C64, "splitbf16": fb.FB_C64_SPLITBF16}
ALPHA = 1e-6


def listed():
    return [
        # the smallest call in use: the 32^3 request of the serving mix, launch bound
        {"name": "transform-32-c64", "kind": "transform", "dtype": "c64", "nx": 32, "ny": 32, "nz": 32,
         "inverse": False, "inplace": False},
        # repeated radix-3 stages, the inverse in place: a grid whose owner keeps one buffer
        {"name": "roundtrip-162x96x216-c128", "kind": "transform", "dtype": "c128", "nx": 162, "ny": 96, "nz": 216,
         "inverse": True, "inplace": True},
        # odd axis lengths: no two strided pencils pair up, tiles are ragged
        {"name": "roundtrip-81x243x81-c64", "kind": "transform", "dtype": "c64", "nx": 81, "ny": 243, "nz": 81,
         "inverse": True, "inplace": False},
        # the split-bf16 matrix-core form on the large block's grid
        {"name": "roundtrip-512x256x256-bf16", "kind": "transform", "dtype": "splitbf16", "nx": 512, "ny": 256,
         "nz": 256, "inverse": True, "inplace": False},
        # the paper's own workload: one 2048 x 2048 transform
        {"name": "transform-2048x2048-c128", "kind": "transform", "dtype": "c128", "nx": 1, "ny": 2048, "nz": 2048,
         "inverse": False, "inplace": False},
        # the small spectral block: 27 launches of a few microseconds each
        {"name": "block-64-c128", "kind": "block", "dtype": "c128", "nx": 64, "ny": 64, "nz": 64, "steps": 6},
        # the benchmark's block, in both storage precisions: larger than the last-level cache
        {"name": "block-512x256x256-c128", "kind": "block", "dtype": "c128", "nx": 512, "ny": 256, "nz": 256,
         "steps": 10},
        {"name": "block-512x256x256-c64", "kind": "block", "dtype": "c64", "nx": 512, "ny": 256, "nz": 256,
         "steps": 10},
        # a middle request of the serving mix: 70 % of it is complex64
        {"name": "steps-128-c64", "kind": "steps", "dtype": "c64", "nx": 128, "ny": 128, "nz": 128, "steps": 5},
        # the batched workload: 4096 mixed lengths 2^k and 3 2^k, and 64 images
        {"name": "batch-4096x1d-64x512x512", "kind": "batch", "n1d": 4096, "n2d": 64, "side": 512, "lens_seed": 3,
         "inverse": False},
        # the paper's other block at its size, and a small odd one with a row stride
        {"name": "lu-2048", "kind": "lu", "n": 2048, "pad": 0},
        {"name": "lu-333", "kind": "lu", "n": 333, "pad": 3},
    ]


def _axis(rng, lo, hi):
    """A supported axis length (2^a 3^b) in [lo, hi], spread over the logarithm."""
    every = sorted(2 ** a * 3 ** b for a in range(13) for b in range(8) if lo <= 2 ** a * 3 ** b <= hi)
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(every, key=lambda n: abs(math.log(n / want)))


def _shape(rng, lo, hi):
    """A grid of lo..hi elements, of one to three axes of length above 1."""
    while True:
        d = [_axis(rng, 8, 1024) for _ in range(3)]
        flat = rng.random()
        if flat < 0.15:
            d[0] = 1
            d[1], d[2] = _axis(rng, 64, 4096), _axis(rng, 64, 4096)
        if lo <= d[0] * d[1] * d[2] <= hi:
            return dict(zip(("nx", "ny", "nz"), d))


def draw(rng):
    kind = rng.choice(["transform", "transform", "block", "steps", "batch", "lu"])
    if kind == "transform":
        return {"kind": kind, "dtype": rng.choice(["c128", "c64", "splitbf16"]), **_shape(rng, 1 << 13, 1 << 25),
                "inverse": rng.random() < 0.6, "inplace": rng.random() < 0.4}
    if kind == "block":
        return {"kind": kind, "dtype": rng.choice(["c128", "c64", "splitbf16"]), **_shape(rng, 1 << 15, 1 << 25),
                "steps": rng.randint(1, 10)}
    if kind == "steps":
        return {"kind": kind, "dtype": rng.choice(["c128", "c64"]), **_shape(rng, 1 << 15, 1 << 24),
                "steps": rng.randint(1, 10)}
    if kind == "batch":
        return {"kind": kind, "n1d": int(round(math.exp(rng.uniform(math.log(8), math.log(4096))))),
                "n2d": rng.randint(0, 64), "side": _pow2_or_3(rng, 64, 512), "lens_seed": rng.randint(0, 1 << 20),
                "inverse": rng.random() < 0.5}
    return {"kind": kind, "n": int(round(math.exp(rng.uniform(math.log(24), math.log(2048))))),
            "pad": rng.choice([0, 0, rng.randint(1, 64)])}


def _pow2_or_3(rng, lo, hi):
    every = sorted({n for k in range(13) for n in (1 << k, 3 << k) if lo <= n <= hi})
    return rng.choice(every)


def _shape_of(case):
    return case["nx"], case["ny"], case["nz"]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _torch_dtype(case):
    return torch.complex128 if case["dtype"] == "c128" else torch.complex64


def _grid(case, seed):
    """The input grid: N(0, 1) in each part."""
    real = torch.float64 if case["dtype"] == "c128" else torch.float32
    return torch.view_as_complex(torch.randn(_shape_of(case) + (2,), dtype=real, device="cuda",
                                             generator=_generator(seed)))


def _batch_data(case, elements, seed):
    """Packed U[-1, 1) elements."""
    x = torch.rand((elements, 2), dtype=torch.float32, device="cuda", generator=_generator(seed))
    return torch.view_as_complex(x.mul_(2.0).sub_(1.0))


def _matrix(case, seed):
    n = case["n"]
    x = torch.rand((n, n), dtype=torch.float64, device="cuda", generator=_generator(seed))
    return x.mul_(2.0).sub_(1.0)


def _lens(case):
    return [int(v) for v in inputs.batch_lengths(case["n1d"], case["lens_seed"])]


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("transform", "block", "steps"):
        s["plan"] = fb.Plan(*_shape_of(case), DTYPES[case["dtype"]])
        dt = _torch_dtype(case)
        s["u"] = torch.empty(_shape_of(case), dtype=dt, device="cuda")
    if kind == "transform":
        s["x"] = _grid(case, seed)
        if case["inverse"] and not case["inplace"]:
            s["y"] = torch.empty_like(s["x"])
    elif kind == "block":
        s["x"] = _grid(case, seed)
        s["y"] = torch.empty_like(s["x"])
        s["sums"] = torch.zeros((case["steps"], 2), dtype=torch.float64, device="cuda")
    elif kind == "steps":
        s["seed"] = inputs.stream_seed(4, seed)
        s["ts"] = [float(t) for t in range(1, case["steps"] + 1)]
        s["y"] = torch.empty((case["steps"],) + _shape_of(case), dtype=dt, device="cuda")
        s["sums"] = torch.zeros((case["steps"], 2), dtype=torch.float64, device="cuda")
    elif kind == "batch":
        s["batch"] = fb.Batch(_lens(case), case["n2d"], case["side"])
        s["x"] = _batch_data(case, s["batch"].elements, seed)
        s["y"] = torch.empty_like(s["x"])
        s["ws"] = torch.empty(256, dtype=torch.uint8, device="cuda")
    elif kind == "lu":
        n = case["n"]
        s["a0"] = _matrix(case, seed)
        s["a"] = torch.zeros((n, n + case["pad"]), dtype=torch.float64, device="cuda")[:, :n]
        s["ipiv"] = torch.zeros(n, dtype=torch.int32, device="cuda")
        s["info"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "transform":
        fb.fb_fft3d_exec(s["plan"], s["x"], s["u"], fb.FB_FORWARD)
        if not case["inverse"]:
            return {"spectrum": s["u"]}
        if case["inplace"]:
            fb.fb_fft3d_exec(s["plan"], s["u"], s["u"], fb.FB_INVERSE)
            return {"grid": s["u"]}
        fb.fb_fft3d_exec(s["plan"], s["u"], s["y"], fb.FB_INVERSE)
        return {"spectrum": s["u"], "grid": s["y"]}
    if kind == "block":
        fb.fb_fft3d_exec(s["plan"], s["x"], s["u"], fb.FB_FORWARD)
        for t in range(1, case["steps"] + 1):
            fb.fb_spectral_step(s["plan"], s["u"], s["y"], ALPHA, float(t), s["sums"][t - 1])
        return {"spectrum": s["u"], "grid": s["y"], "sums": s["sums"]}
    if kind == "steps":
        fb.fb_fft3d_forward_uniform(s["plan"], s["seed"], s["u"])
        fb.fb_spectral_steps(s["plan"], s["u"], s["y"], ALPHA, s["ts"], s["sums"])
        return {"spectrum": s["u"], "grids": s["y"], "sums": s["sums"]}
    if kind == "batch":
        fb.fb_batch_exec(s["batch"], s["x"], s["y"], s["ws"], fb.FB_INVERSE if case["inverse"] else fb.FB_FORWARD)
        return {"out": s["y"]}
    # the matrix is kept: a program that solves again needs it beside its factors
    s["a"].copy_(s["a0"])
    fb.fb_lu_factor(s["a"], s["ipiv"], s["info"])
    return {"lu": s["a"], "ipiv": s["ipiv"], "info": s["info"]}


def work(case):
    kind = case["kind"]
    if kind in ("transform", "block", "steps"):
        n = case["nx"] * case["ny"] * case["nz"]
        e = 16 if case["dtype"] == "c128" else 8
        fft = 5.0 * n * math.log2(n)
        if kind == "transform":
            calls = 2 if case["inverse"] else 1
            return {"bytes": 2.0 * e * n * calls, "flops": fft * calls}
        if kind == "block":   # every step reads the spectrum and writes its grid
            return {"bytes": 2.0 * e * n * (1 + case["steps"]), "flops": (fft + 2.0 * n) * (1 + case["steps"])}
        # the spectrum written and read once, every grid written
        return {"bytes": e * n * (2.0 + case["steps"]), "flops": (fft + 2.0 * n) * (1 + case["steps"])}
    if kind == "batch":
        lens = _lens(case) + [case["side"] ** 2] * case["n2d"]
        return {"bytes": 16.0 * sum(lens), "flops": sum(5.0 * n * math.log2(n) for n in lens)}
    n = case["n"]
    return {"bytes": 16.0 * n * n, "flops": 2.0 / 3.0 * n ** 3}


def _k2(case):
    """|k|^2 with signed wavenumbers, shape (nx, ny, nz)."""
    total = 0.0
    for axis, n in enumerate(_shape_of(case)):
        k = torch.arange(n, dtype=torch.float64, device="cuda")
        k = torch.where(2 * k >= n, k - n, k)
        total = total + (k * k).reshape([-1 if a == axis else 1 for a in range(3)])
    return total


def _checksum(x):
    flat = x.reshape(-1)
    at = (17 * torch.arange(1024, device=flat.device)) % flat.numel()
    return torch.view_as_real(flat[at].sum())


def _uniform(case, seed):
    """The grid that the library generates from a stream seed, rounded to its storage precision."""
    x = torch.from_numpy(inputs.uniform_grid(_shape_of(case), seed)).cuda()
    return x if case["dtype"] == "c128" else x.to(torch.complex64).to(torch.complex128)


def exact(case, seed):
    kind = case["kind"]
    if kind == "transform":
        x = _grid(case, seed).to(torch.complex128)
        if case["inplace"] and case["inverse"]:
            return {"grid": x}
        u = torch.fft.fftn(x)
        return {"spectrum": u, "grid": x} if case["inverse"] else {"spectrum": u}
    if kind in ("block", "steps"):
        x = _grid(case, seed).to(torch.complex128) if kind == "block" else _uniform(case,
                                                                                    inputs.stream_seed(4, seed))
        u = torch.fft.fftn(x)
        k2 = _k2(case)
        grids, sums = [], []
        for t in range(1, case["steps"] + 1):
            y = torch.fft.ifftn(u * torch.exp(-4.0 * math.pi ** 2 * ALPHA * t * k2))
            sums.append(_checksum(y))
            if kind == "steps":
                grids.append(y)
        if kind == "block":
            return {"spectrum": u, "grid": y, "sums": torch.stack(sums)}
        return {"spectrum": u, "grids": torch.stack(grids), "sums": torch.stack(sums)}
    if kind == "batch":
        lens, n2d, side = _lens(case), case["n2d"], case["side"]
        x = _batch_data(case, sum(lens) + n2d * side * side, seed)
        out = torch.empty(x.shape, dtype=torch.complex128, device="cuda")
        one, two = (torch.fft.ifft, torch.fft.ifft2) if case["inverse"] else (torch.fft.fft, torch.fft.fft2)
        at = 0
        for n in lens:
            out[at:at + n] = one(x[at:at + n].to(torch.complex128))
            at += n
        for _ in range(n2d):
            n = side * side
            out[at:at + n] = two(x[at:at + n].to(torch.complex128).reshape(side, side)).reshape(-1)
            at += n
        return {"out": out}
    lu, piv, info = torch.linalg.lu_factor_ex(_matrix(case, seed).cpu())
    return {"lu": lu, "ipiv": piv - 1, "info": info.reshape(1)}
