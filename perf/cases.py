"""The work that programs have this library do, as cases that can be timed.

Each case is one call (or, for a prepared constant operand, one call of the
serving loop) through the package's public functions: the FP32-accuracy product
of two FP32 matrices in one of the three accumulation orders, its pre-scaled
form with the range report, and the FP16 baseline.  The listed sizes are those
of this repository's workloads (workloads.py), of its accuracy sweeps
(bench_accuracy.py) and of its tests; draw() gives others of the same ranges.

    entry   matmul    sgc.matmul, the library takes its own workspace
            held      sgc.matmul into a result and a workspace the program keeps
            serve     sgemm_cube_compute_a: rows of A against a constant B whose
                      planes were prepared once
            prescale  sgc.matmul_ex with pre-scaling and the range report
            hgemm     sgc.hgemm, the FP16 baseline
    values  uniform   U[-1, 1]
            normal    N(0, 1)
            wide      sign * U[1, 2) * 2^e, e in -12 .. 12 (s B_hi overflows FP16)
            tiny      U[-1, 1] * 2^-14 (FP16-subnormal high words)
            lines     rows of A and columns of B from 2^-28 to 2^24 (pre-scaling)
    pad     extra elements between the rows of A (a view of a wider matrix)
"""
import math

import torch

import paper_2507_23387_amd as sgc


def _case(name, entry, m, n, k, order="elementwise", log2_scale=11, values="uniform", pad=0):
    return {"name": name, "entry": entry, "m": m, "n": n, "k": k, "order": order,
            "log2_scale": log2_scale, "values": values, "pad": pad}


def listed():
    return [
        # One small product: what a program pays for the call itself.
        _case("square256", "matmul", 256, 256, 256),
        # A ragged small product in a tight loop that keeps its buffers.
        _case("ragged300_held", "held", 300, 200, 1000, "termwise", values="normal"),
        # A point of the accuracy sweep over exponents.
        _case("square1024", "matmul", 1024, 1024, 1024, log2_scale=12),
        # A point of the accuracy sweep over k: few tiles, a long contraction.
        _case("longk1024", "matmul", 1024, 1024, 16384, "termwise"),
        # A point of the pre-scaling sweep, with the range report.
        _case("prescale1024", "prescale", 1024, 1024, 1024, values="lines"),
        # A few rows against constant weights: a step of a serving loop.
        _case("serve48", "serve", 48, 4096, 4096, values="normal"),
        # An ordinary product of odd sizes, rows not aligned to anything.
        _case("ragged2777_cross", "matmul", 2777, 3001, 1531, "elementwise_cross_first", pad=2),
        # The FP16 baseline at the k of the accuracy sweep over m = n.
        _case("hgemm2048", "hgemm", 2048, 2048, 2816),
        # The named workloads of the benchmark.
        _case("square4096", "matmul", 4096, 4096, 4096, "termwise", values="normal"),
        _case("rect_subnormal", "matmul", 16384, 1024, 8192, log2_scale=13, values="tiny"),
        _case("longk_wide", "matmul", 4096, 4096, 16384, values="wide"),
        _case("square8192", "matmul", 8192, 8192, 8192),
    ]


def _size(rng, low, high):
    v = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
    return max(64, v // 64 * 64) if v > 96 and rng.random() < 0.4 else v


def draw(rng):
    entry = rng.choice(["matmul"] * 6 + ["held"] * 2 + ["serve"] * 2 + ["prescale", "hgemm"])
    while True:
        m = _size(rng, 1, 256) if entry == "serve" else _size(rng, 16, 16384)
        n = _size(rng, 512, 8192) if entry == "serve" else _size(rng, 16, 8192)
        k = _size(rng, 64, 16384)
        # Well below the largest listed case, also in time.
        if 2**17 <= m * n * k <= 2**37 and m * k + k * n <= 2**27:
            break
    order = rng.choice(["elementwise", "elementwise", "termwise", "elementwise_cross_first"])
    values = rng.choice(["uniform", "normal", "uniform", "normal", "wide", "tiny"])
    if entry == "hgemm":
        order, values = "elementwise", rng.choice(["uniform", "normal"])
    if entry == "prescale":
        values = "lines"
    return {"entry": entry, "m": m, "n": n, "k": k, "order": order,
            "log2_scale": 13 if values == "tiny" else rng.choice([11, 12]), "values": values,
            "pad": rng.choice([0, 0, 0, 4, 1])}


def _values(case, shape, gen, lines_dim):
    kind = case["values"]
    dev = torch.device("cuda")
    if kind == "normal":
        return torch.randn(shape, generator=gen, device=dev)
    if kind == "wide":
        u = torch.rand(shape, generator=gen, device=dev).add_(1.0)
        e = torch.randint(-12, 13, shape, generator=gen, device=dev, dtype=torch.int32)
        sign = torch.randint(0, 2, shape, generator=gen, device=dev, dtype=torch.int32)
        return torch.ldexp(u, e).mul_(1 - 2 * sign)
    x = torch.rand(shape, generator=gen, device=dev).mul_(2.0).sub_(1.0)
    if kind == "tiny":
        x.mul_(2.0**-14)
    elif kind == "lines":
        line = [1, 1]
        line[lines_dim] = shape[lines_dim]
        x = torch.ldexp(x, torch.randint(-28, 25, line, generator=gen, device=dev,
                                         dtype=torch.int32))
    return x


def _operands(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 17)
    m, n, k, pad = case["m"], case["n"], case["k"], case["pad"]
    A = _values(case, (m, k), gen, 0)
    B = _values(case, (k, n), gen, 1)
    if pad:
        wide = torch.zeros((m, k + pad), device="cuda")
        wide[:, :k].copy_(A)
        A = wide[:, :k]
    return A, B


def prepare(case, seed):
    m, n, k = case["m"], case["n"], case["k"]
    A, B = _operands(case, seed)
    state = {"case": dict(case), "A": A, "B": B, "scale": 2.0 ** case["log2_scale"]}
    if case["entry"] in ("held", "serve"):
        state["C"] = torch.empty((m, n), device="cuda")
        state["ws"] = sgc.workspace(m, n, k)
    if case["entry"] == "serve":
        ws = state["ws"]
        status = sgc.sgemm_cube_prepare(m, n, k, None, max(k, 1), B.data_ptr(), B.stride(0),
                                        state["scale"], ws.data_ptr(), ws.numel(),
                                        torch.cuda.current_stream().cuda_stream)
        if status != 0:
            raise RuntimeError(sgc.sgemm_cube_status_string(status))
    return state


def run(state):
    case, A, B, scale = state["case"], state["A"], state["B"], state["scale"]
    entry, order = case["entry"], case["order"]
    if entry == "matmul":
        return sgc.matmul(A, B, scale=scale, order=order)
    if entry == "held":
        return sgc.matmul(A, B, scale=scale, order=order, out=state["C"], workspace=state["ws"])
    if entry == "prescale":
        return sgc.matmul_ex(A, B, scale=scale, order=order, prescale=True, report=True)
    if entry == "hgemm":
        return sgc.hgemm(A, B)
    C, ws = state["C"], state["ws"]
    status = sgc.sgemm_cube_compute_a(case["m"], case["n"], case["k"], A.data_ptr(), A.stride(0),
                                      C.data_ptr(), C.stride(0), scale, sgc.binding.ORDERS[order],
                                      ws.data_ptr(), ws.numel(),
                                      torch.cuda.current_stream().cuda_stream)
    if status != 0:
        raise RuntimeError(sgc.sgemm_cube_status_string(status))
    return C


def work(case):
    m, n, k = case["m"], case["n"], case["k"]
    # B's prepared planes (serve) have the four bytes per entry of FP32 B.
    return {"bytes": 4.0 * (m * k + k * n + m * n),
            "flops": (2.0 if case["entry"] == "hgemm" else 6.0) * m * n * k}


def tolerance(case):
    # FP32 sums of exact FP16 products: another order of summation differs by
    # the order's own rounding error, which grows like sqrt(k) (elementwise,
    # the longest chain, against 64 bits: 2.0e-7 at k = 256, 7.2e-7 at 4096,
    # 1.5e-6 at 16384); about four times that.
    return {"rel": 4.0e-7 + 4.8e-8 * math.sqrt(case["k"])}


def exact(case, seed):
    A, B = _operands(case, seed)
    if case["entry"] == "hgemm":
        return A.half().double() @ B.half().double()
    C = A.double() @ B.double()
    return (C, None) if case["entry"] == "prescale" else C
