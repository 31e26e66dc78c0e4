"""The matrix products that users of the library run, as cases to time.

A case is one GEMM  C = act(alpha * op(A) * op(B) + beta * C + bias)  through the package's public entry
points: the plan, the operands, the workspace and the stream are what the program holds; a pass is one run of the
plan.  Sizes are those of the library's own workloads (the square and the streaming products), of transformer
layers in its selector table, and ragged or odd ones of the same ranges.
"""
import math

import torch

import paper_2512_19018_amd as pg

_DT = {"f32": (pg.PEAK_DT_F32, torch.float32, 4), "f16": (pg.PEAK_DT_F16, torch.float16, 2),
       "bf16": (pg.PEAK_DT_BF16, torch.bfloat16, 2)}
_BIAS = {"none": pg.PEAK_BIAS_NONE, "column": pg.PEAK_BIAS_PER_COLUMN, "row": pg.PEAK_BIAS_PER_ROW}
_ACT = {"none": pg.PEAK_ACT_NONE, "relu": pg.PEAK_ACT_RELU, "gelu": pg.PEAK_ACT_GELU_TANH}


def _case(dtype, ta, tb, M, N, K, alpha=1.0, beta=0.0, bias="none", act="none", c_f32=False, entry="run",
          dist="normal", scale=0.02, pad=0, off=0, **name):
    """pad: elements a stored row of A, B and C is longer than its data; off: elements that the first one of A
    and B lies behind a 256-byte boundary (both 0: whole matrices; else blocks of larger ones)."""
    return dict(name, dtype=dtype, ta=ta, tb=tb, M=M, N=N, K=K, alpha=alpha, beta=beta, bias=bias, act=act,
                c_f32=c_f32, entry=entry, dist=dist, scale=scale, pad=pad, off=off)


def listed():
    return [
        # the smallest product that programs call in earnest: one launch's latency is the cost (workload C1)
        _case("f32", 0, 0, 256, 256, 256, dist="uniform", scale=1.0, name="f32_256_nn"),
        # single-precision BLAS call that updates C in place (workload C2)
        _case("f32", 0, 0, 4096, 4096, 4096, beta=0.5, dist="uniform", scale=1.0, name="f32_4096_nn_beta"),
        # the headline: a large bf16 product of weights and activations as stored by a linear layer (workload C3)
        _case("bf16", 0, 1, 8192, 8192, 8192, scale=1.0 / math.sqrt(8192.0), name="bf16_8192_nt"),
        # f16, deep K, edges inside tiles (workload C4)
        _case("f16", 0, 0, 5000, 3000, 12288, dist="uniform", scale=1.0, name="f16_5000x3000x12288_nn"),
        # decode: a batch of 16 tokens against a square weight; the weight's bytes are the cost (workload C5)
        _case("bf16", 0, 1, 16, 16384, 16384, name="bf16_decode_16x16384_nt"),
        # decode with a ragged batch, weights stored in x out, bias and ReLU fused
        _case("f16", 0, 0, 37, 14336, 4096, bias="column", act="relu", name="f16_decode_37x14336x4096_nn"),
        # prefill of an MLP's first layer: ragged number of tokens, bias and GELU fused
        _case("bf16", 0, 1, 1000, 14336, 4096, scale=1.0 / 64, bias="column", act="gelu", name="bf16_mlp_up_gelu_nt"),
        # backward of a linear layer, weight gradient: summed over the tokens into an fp32 master gradient
        _case("bf16", 1, 0, 4096, 4096, 2000, beta=1.0, c_f32=True, scale=1.0 / 64, name="bf16_wgrad_f32acc_tn"),
        # backward of a linear layer, input gradient: few tokens, deep K
        _case("bf16", 0, 0, 512, 4096, 14336, scale=1.0 / 64, name="bf16_dgrad_512x4096x14336_nn"),
        # odd sizes throughout, blocks of larger matrices that start one element in: no row is 16-byte aligned
        _case("bf16", 0, 1, 1023, 2047, 3001, scale=1.0 / 64, pad=6, off=1, name="bf16_odd_block_nt"),
        # scientific single precision of no particular size, both operands transposed
        _case("f32", 1, 1, 777, 1234, 1555, dist="uniform", scale=1.0, name="f32_odd_777x1234x1555_tt"),
        # small batch in a serving loop that passes no workspace
        _case("bf16", 0, 1, 100, 4096, 4096, entry="static", name="bf16_serve_100x4096_static_nt"),
    ]


_MAX_FLOPS = {"f32": 2.0 * 4096 ** 3, "f16": 2.0 * 8192 ** 3, "bf16": 2.0 * 8192 ** 3}
_MAX_BYTES = 2.0 ** 30


def _size(rng, lo, hi, grain):
    """log-uniform in [lo, hi], a multiple of `grain`"""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(grain, v // grain * grain)


def _draw(rng):
    kind = rng.choice(["product", "product", "decode", "layer", "wgrad", "dgrad", "odd", "odd", "serve"])
    half = rng.choice(["bf16", "bf16", "f16"])
    if kind == "product":                    # BLAS calls of any type, layout and size
        dt = rng.choice(["f32", "f16", "bf16"])
        dims = [_size(rng, 128, 8192, rng.choice([1, 8, 8, 64])) for _ in range(3)]
        beta = rng.choice([0.0, 0.0, 0.5, 1.0])
        return _case(dt, rng.randint(0, 1), rng.randint(0, 1), *dims, alpha=rng.choice([1.0, 0.75]), beta=beta,
                     dist="uniform", scale=1.0)
    if kind == "decode":
        dt = rng.choice([half, half, "f32"])
        N, K = _size(rng, 2048, 32768, 64), _size(rng, 2048, 16384, 128)
        return _case(dt, rng.choice([0, 0, 0, 1]), rng.randint(0, 1), rng.randint(1, 64), N, K,
                     bias=rng.choice(["none", "column"]), act=rng.choice(["none", "relu", "gelu"]))
    if kind == "layer":
        N, K = _size(rng, 1024, 28672, 128), _size(rng, 1024, 16384, 128)
        return _case(half, 0, rng.choice([1, 1, 0]), _size(rng, 65, 8192, rng.choice([1, 64])), N, K,
                     scale=1.0 / 64, bias=rng.choice(["none", "column", "column", "row"]),
                     act=rng.choice(["none", "relu", "gelu"]))
    if kind == "wgrad":
        return _case(half, 1, 0, _size(rng, 512, 8192, 64), _size(rng, 512, 8192, 64),
                     _size(rng, 256, 16384, rng.choice([1, 8, 64])), beta=rng.choice([0.0, 1.0]), c_f32=True,
                     scale=1.0 / 64)
    if kind == "dgrad":
        return _case(half, 0, 0, _size(rng, 65, 8192, rng.choice([1, 64])), _size(rng, 1024, 8192, 64),
                     _size(rng, 1024, 28672, 64), scale=1.0 / 64)
    if kind == "odd":                        # odd sizes; whole matrices or blocks of larger ones
        dt = rng.choice(["f32", half, half])
        dims = [_size(rng, 65, 4096, 1) | 1 for _ in range(3)]
        view = rng.random() < 0.5
        return _case(dt, rng.randint(0, 1), rng.randint(0, 1), *dims, dist="uniform", scale=1.0,
                     pad=rng.randint(1, 64) if view else 0, off=rng.randint(1, 7) if view else 0)
    return _case(half, 0, 1, rng.randint(17, 128), _size(rng, 512, 4096, 64), _size(rng, 1024, 8192, 128),
                 entry="static")


def draw(rng):
    while True:
        c = _draw(rng)
        w = work(c)
        if w["flops"] <= _MAX_FLOPS[c["dtype"]] and w["bytes"] <= _MAX_BYTES:
            return c


def work(case):
    M, N, K, es = case["M"], case["N"], case["K"], _DT[case["dtype"]][2]
    es_c = 4 if case["c_f32"] else es
    bias = {"none": 0, "column": N, "row": M}[case["bias"]]
    return {"bytes": (M * K + K * N) * es + M * N * es_c * (2 if case["beta"] else 1) + 4 * bias,
            "flops": 2.0 * M * N * K}


def tolerance(case):
    # Measured against fp64 over these ranges: fp32 results up to 2e-6 (K products summed in fp32), f16 2.1e-4 and
    # bf16 1.7e-3 (the one rounding to storage).  A single element may be a unit or two in the last place off.
    if case["dtype"] == "f32" or case["c_f32"]:
        return {"rel": 8e-6, "max": 1e-4}
    return {"rel": 8e-4, "max": 4e-3} if case["dtype"] == "f16" else {"rel": 7e-3, "max": 3e-2}


class _Matrix:
    """rows x cols of a buffer with rows `ld` elements apart, starting `off` elements in."""

    def __init__(self, gen, rows, cols, dtype, case, pad, off):
        self.shape, self.ld = (rows, cols), cols + pad
        n, self.off = rows * self.ld + off, off
        x = torch.empty(n, dtype=torch.float32, device="cuda")
        if case["dist"] == "uniform":
            x.uniform_(-case["scale"], case["scale"], generator=gen)
        else:
            x.normal_(0.0, case["scale"], generator=gen)
        self.buf = x.to(dtype)

    def view(self):
        return torch.as_strided(self.buf, self.shape, (self.ld, 1), self.off)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = _DT[case["dtype"]][1]
    M, N, K, pad, off = case["M"], case["N"], case["K"], case["pad"], case["off"]
    A = _Matrix(gen, *((K, M) if case["ta"] else (M, K)), dtype, case, pad, off)
    B = _Matrix(gen, *((N, K) if case["tb"] else (K, N)), dtype, case, pad, off)
    C = _Matrix(gen, M, N, torch.float32 if case["c_f32"] else dtype, case, pad, 0)
    n = {"none": 0, "column": N, "row": M}[case["bias"]]
    bias = torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, 0.5, generator=gen)
    return A, B, C, bias


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.A, s.B, s.C, s.bias = _inputs(case, seed)
    es = _DT[case["dtype"]][2]
    s.plan = pg.Plan(case["M"], case["N"], case["K"], _DT[case["dtype"]][0], case["ta"], case["tb"], s.A.ld, s.B.ld,
                     s.C.ld, pg.PEAK_GEMM_C_F32 if case["c_f32"] else 0)
    s.nbytes = s.plan.workspace_bytes if case["entry"] == "run" else 0
    s.ws = torch.empty(max(s.nbytes, 256), dtype=torch.uint8, device="cuda")
    s.alpha, s.beta = case["alpha"], case["beta"]
    s.a, s.b, s.c = s.A.buf.data_ptr() + s.A.off * es, s.B.buf.data_ptr() + s.B.off * es, s.C.buf.data_ptr()
    s.static = case["entry"] == "static"
    s.fused = case["bias"] != "none" or case["act"] != "none"
    s.bias_kind, s.act = _BIAS[case["bias"]], _ACT[case["act"]]
    s.stream = torch.cuda.current_stream().cuda_stream
    s.out = s.C.view()
    return s


def run(s):
    if s.static:
        status = pg.peak_gemm_run_static(s.plan.handle, s.alpha, s.a, s.b, s.beta, s.c, s.stream)
        if status != pg.PEAK_OK:
            raise pg.PeakError(status, "peak_gemm_run_static")
    elif s.fused:
        s.plan.run_fused(s.alpha, s.a, s.b, s.beta, s.c, s.bias_kind, s.bias.data_ptr(), s.act, s.ws.data_ptr(),
                         s.nbytes, s.stream)
    else:
        s.plan.run(s.alpha, s.a, s.b, s.beta, s.c, s.ws.data_ptr(), s.nbytes, s.stream)
    return s.out


def exact(case, seed):
    A, B, C, bias = _inputs(case, seed)
    a, b = A.view().double(), B.view().double()
    if case["ta"]:
        a = a.t().contiguous()
    if case["tb"]:
        b = b.t().contiguous()
    x = case["alpha"] * torch.mm(a, b)
    if case["beta"]:
        x += case["beta"] * C.view().double()
    if case["bias"] != "none":
        x += bias.double()[None, :] if case["bias"] == "column" else bias.double()[:, None]
    if case["act"] == "relu":
        x = torch.relu(x)
    elif case["act"] == "gelu":
        x = torch.nn.functional.gelu(x, approximate="tanh")
    return x
