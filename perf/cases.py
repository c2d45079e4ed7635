"""The calls that a program using this library spends its time in.

One case is one call (or one forward + backward step) through the public
Python entry points, on matrices or bodies of the sizes that the library's
benchmark, tests and configurations use: from a matrix-vector product of a
few hundred rows to the fp8 product of 16384 x 8192 x 16384.

Kinds
  product   hs_gemm, or hs_gemm_tn (tn): forward only, as in inference
  noalloc   hs_gemm_noalloc into a kept output: serving loops that must not
            allocate
  step      hs_gemm and hs_gemm_backward: a training step without autograd
  train     the same through autograd.matmul
  gemv      hs_gemv
  nbody     hs_nbody: one force evaluation of an integrator
"""
import torch

from paper_cs_9809105_amd import autograd, binding

_IN = {"f64": torch.float64, "bf16": torch.bfloat16, "f16": torch.float16}
# MFMA products that each form is defined by (include/hs.h); 4 real
# multiplications per complex one are counted in _flops
_PRODUCTS = {"split3_bf16": 6, "split2_f16": 3, "fp8_e4m3_r1": 3, "c32_split3_bf16": 6, "c32_split2_f16": 3}


def listed():
    return [
        # one layer's matrix-vector product with nothing aligned: the
        # shortest call, latency only
        {"name": "gemv_f32_1000x777", "kind": "gemv", "form": "f32", "m": 1000, "n": 777, "p": 8, "K": 2},
        # the matrix-vector benchmark: bound by reading A once
        {"name": "gemv_f32_8192", "kind": "gemv", "form": "f32", "m": 8192, "n": 8192, "p": 64, "K": 0},
        # the FP64 configuration: a small product, launch bound
        {"name": "f64_256", "kind": "product", "form": "f64", "m": 256, "n": 256, "k": 256, "p": 16, "K": 4,
         "tn": False},
        # a serving loop's ragged product into a kept buffer
        {"name": "noalloc_split3_1100x900x1000", "kind": "noalloc", "form": "split3_bf16", "m": 1100, "n": 900,
         "k": 1000, "p": 8, "K": 2},
        # a complex training step with ragged sizes
        {"name": "c32_split3_step_1000x700x900", "kind": "step", "form": "c32_split3_bf16", "m": 1000, "n": 700,
         "k": 900, "p": 8, "K": 2},
        # the FP32 configuration, on the transposed product
        {"name": "f32_tn_4096", "kind": "product", "form": "f32", "m": 4096, "n": 4096, "k": 4096, "p": 64, "K": 0,
         "tn": True},
        # the differentiation workload through autograd, FP32-accurate on FP16 units
        {"name": "split2_train_4096x8192x2048", "kind": "train", "form": "split2_f16", "m": 4096, "n": 8192,
         "k": 2048, "p": 16, "K": 4},
        # 16-bit inference at full size
        {"name": "bf16_8192", "kind": "product", "form": "bf16", "m": 8192, "n": 8192, "k": 8192, "p": 64, "K": 2,
         "tn": False},
        # the headline step
        {"name": "split3_step_8192", "kind": "step", "form": "split3_bf16", "m": 8192, "n": 8192, "k": 8192, "p": 64,
         "K": 2},
        # the refined fp8 workload's forward product
        {"name": "fp8_r1_16384x16384x8192", "kind": "product", "form": "fp8_e4m3_r1", "m": 16384, "n": 16384,
         "k": 8192, "p": 64, "K": 2, "tn": False},
        # a star cluster of a few thousand bodies: many short force evaluations
        {"name": "nbody_f32_3000", "kind": "nbody", "form": "f32", "n": 3000, "p": 16, "K": 4},
        # the all-pairs benchmark
        {"name": "nbody_f32_262144", "kind": "nbody", "form": "f32", "n": 262144, "p": 64, "K": 8},
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _schedule(rng, most):
    """(p, K) with stripes of at least 16: K is the default or any divisor."""
    p = rng.choice([q for q in (1, 2, 4, 8, 12, 16, 32, 64) if q == 1 or q <= most // 16])
    return p, rng.choice([0] + [d for d in (1, 2, 4, 8) if p % d == 0])


def draw(rng):
    kind = rng.choice(["product", "product", "product", "noalloc", "step", "train", "gemv", "nbody"])
    if kind == "gemv":
        m, n = _log(rng, 100, 8192), _log(rng, 100, 8192)
        p, K = _schedule(rng, min(m, n))
        return {"kind": kind, "form": rng.choice(["f32", "f32", "f64", "c32"]), "m": m, "n": n, "p": p, "K": K}
    if kind == "nbody":
        form = rng.choice(["f32", "f32", "f64"])
        n = _log(rng, 500, 262144 if form == "f32" else 32768)
        p, K = _schedule(rng, n)
        return {"kind": kind, "form": form, "n": n, "p": p, "K": K}
    forms = ["f64", "f32", "split3_bf16", "split2_f16", "bf16", "f16", "fp8_e4m3", "fp8_e4m3_r1",
             "c32", "c32_split3_bf16", "c32_split2_f16"]
    if kind == "train":                       # autograd takes FP32, FP64 and complex inputs
        forms = [f for f in forms if f not in ("bf16", "f16")]
    form = rng.choice(forms)
    hi = {"f64": 2048, "noalloc": 1200}.get(kind if kind == "noalloc" else form, 2048 if form[0] == "c" else 6144)
    if form.startswith("fp8") and kind != "noalloc":
        # fp8 scales need blocks of whole 64-element chunks
        p = rng.choice([2, 4, 8, 16, 32])
        m, n, k = (64 * p * max(1, round(_log(rng, 128, hi) / (64 * p))) for _ in range(3))
        K = rng.choice([0, 1, 2])
    elif form.startswith("fp8"):
        p, K = rng.choice([1, 2, 4]), rng.choice([0, 1])
        m, n, k = (64 * p * max(1, round(_log(rng, 128, hi) / (64 * p))) for _ in range(3))
    else:
        m, n, k = (_log(rng, 64, hi) for _ in range(3))
        if rng.random() < 0.5:                # half of them on whole 16-byte rows
            m, n, k = (max(64, x // 16 * 16) for x in (m, n, k))
        p, K = _schedule(rng, min(m, n, k))
    c = {"kind": kind, "form": form, "m": m, "n": n, "k": k, "p": p, "K": K}
    if kind == "product":
        c["tn"] = rng.random() < 0.4
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _in_type(form):
    return torch.complex64 if form[0] == "c" else _IN.get(form, torch.float32)


def _randn(g, shape, form, scaled=False):
    t = _in_type(form)
    if t.is_complex:
        return torch.randn(shape, generator=g, device="cuda", dtype=t)
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float64 if t == torch.float64 else torch.float32)
    if scaled:     # rows of very different size, log-uniform in [1e-3, 1e3]
        x *= 10.0 ** (6.0 * torch.rand((shape[0], 1), generator=g, device="cuda", dtype=x.dtype) - 3.0)
    return x.to(t)


def _uniform(g, shape):
    return torch.rand(shape, generator=g, device="cuda") * 2 - 1


def _plummer(g, n, dtype):
    """n bodies (x, y, z, m) of equal mass from a Plummer sphere of scale 1."""
    r = torch.rand((3, n), generator=g, device="cuda", dtype=torch.float64)
    rad = (((r[0] * 0.999).clamp_min(1e-9)) ** (-2.0 / 3.0) - 1.0) ** -0.5
    ct, phi = 2.0 * r[1] - 1.0, 2.0 * torch.pi * r[2]
    st = (1.0 - ct * ct).clamp_min(0.0).sqrt()
    mass = torch.full_like(ct, 1.0 / n)
    return torch.stack([rad * st * phi.cos(), rad * st * phi.sin(), rad * ct, mass], dim=1).to(dtype).contiguous()


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(9809105 + 1000003 * seed)
    form = case["form"]
    if case["kind"] == "nbody":
        return {"bodies": _plummer(g, case["n"], _in_type(form))}
    if case["kind"] == "gemv":
        return {"A": _randn(g, (case["m"], case["n"]), form), "x": _randn(g, (case["n"],), form)}
    m, n, k = case["m"], case["n"], case["k"]
    a_shape = (k, m) if case.get("tn") else (m, k)
    if form.startswith("fp8"):
        s = {"A": _uniform(g, a_shape), "B": _uniform(g, (k, n))}
    else:
        # the FP32-accurate forms meet rows of very different size
        scaled = form in ("f32", "split3_bf16", "split2_f16")
        s = {"A": _randn(g, a_shape, form, scaled), "B": _randn(g, (k, n), form, scaled)}
    if case["kind"] in ("step", "train"):
        s["G"] = _uniform(g, (m, n)) if form.startswith("fp8") else _randn(g, (m, n), form)
    return s


EPS2 = 1e-4


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["kind"] == "noalloc":
        out = torch.complex64 if case["form"][0] == "c" else torch.float64 if case["form"] == "f64" else torch.float32
        s["out"] = torch.empty((case["m"], case["n"]), dtype=out, device="cuda")
    if case["kind"] == "train":
        s["A"].requires_grad_(True)
        s["B"].requires_grad_(True)
    return s


def run(s):
    c = s["case"]
    o = dict(dtype=c["form"], p=c["p"], K=c["K"])
    kind = c["kind"]
    if kind == "product":
        return (binding.hs_gemm_tn if c["tn"] else binding.hs_gemm)(s["A"], s["B"], **o)
    if kind == "noalloc":
        return binding.hs_gemm_noalloc(s["A"], s["B"], s["out"], **o)
    if kind == "step":
        C = binding.hs_gemm(s["A"], s["B"], **o)
        dA, dB = binding.hs_gemm_backward(s["A"], s["B"], s["G"], **o)
        return {"C": C, "dA": dA, "dB": dB}
    if kind == "train":
        s["A"].grad = s["B"].grad = None
        C = autograd.matmul(s["A"], s["B"], **o)
        C.backward(s["G"])
        return {"C": C.detach(), "dA": s["A"].grad, "dB": s["B"].grad}
    if kind == "gemv":
        return binding.hs_gemv(s["A"], s["x"], **o)
    return binding.hs_nbody(s["bodies"], EPS2, **o)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    form, kind = case["form"], case["kind"]
    esz = {"f64": 8, "bf16": 2, "f16": 2}.get(form, 8 if form[0] == "c" else 4)
    osz = max(4, esz)
    if kind == "nbody":
        n = case["n"]
        return {"bytes": 8 * n * esz, "flops": 20 * n * n}
    mul = 8 if form[0] == "c" else 2
    if kind == "gemv":
        m, n = case["m"], case["n"]
        return {"bytes": (m * n + n + m) * esz, "flops": mul * m * n}
    m, n, k = case["m"], case["n"], case["k"]
    one = mul * m * n * k * _PRODUCTS.get(form, 1)
    if kind in ("step", "train"):
        return {"bytes": (m * k + k * n + m * n) * (esz + osz), "flops": 3 * one}
    return {"bytes": (m * k + k * n) * esz + m * n * osz, "flops": one}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _nbody64(b, eps2):
    out = torch.empty_like(b)
    n = b.shape[0]
    rows = max(1, (1 << 26) // n)
    at = torch.arange(n, device=b.device)
    for i in range(0, n, rows):
        x = b[i:i + rows]
        d = [b[None, :, c] - x[:, c:c + 1] for c in range(3)]
        inv = (d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + eps2).rsqrt_()
        inv.masked_fill_(at[None, :] == at[i:i + rows, None], 0.0)
        out[i:i + rows, 3] = -(inv @ b[:, 3])
        w = inv.pow(3).mul_(b[:, 3])
        for c in range(3):
            out[i:i + rows, c] = (w * d[c]).sum(dim=1)
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "nbody":
        eps2 = torch.tensor(EPS2, dtype=_in_type(case["form"])).double().item()
        return _nbody64(s["bodies"].double(), eps2)
    s = {k: v.to(torch.complex128 if v.is_complex() else torch.float64) for k, v in s.items()}
    A = s["A"]
    if kind == "gemv":
        return A @ s["x"]
    if case.get("tn"):
        A = A.t().contiguous()
    C = A @ s["B"]
    if kind not in ("step", "train"):
        return C
    dA = s["G"] @ s["B"].mH.contiguous()
    dB = A.mH.contiguous() @ s["G"]
    return {"C": C, "dA": dA, "dB": dB}
