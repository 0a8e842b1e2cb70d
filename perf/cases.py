"""The calls whose speed is looked after: what programs ask of this library, through its public entry points.

`listed()` names twelve of them, from a 256^3 product whose launch is half of its time to a 4096^3 one that fills the
chip; `draw(rng)` gives more of the same ranges: any size (most of them no multiple of anything), layout,
transposition, leading dimension and storage type.  `prepare` makes what a program holds before the call (operands on
the GPU and the workspace the library asks for), `run` is the call.
"""
import math

import torch

from paper_1705_05249_amd import gemm as G
from paper_1705_05249_amd import workloads as W

ROW, COL = G.MG_ROW_MAJOR, G.MG_COL_MAJOR
N, T = G.MG_NO_TRANS, G.MG_TRANS
MOST_FLOPS = 2.0 * 4096 ** 3        # of a drawn product: the largest listed one
MOST_BATCHED_FLOPS = 8.0e9          # of a drawn batched call (the workload's largest, 10000 x 64^3, has 5.2e9)
MOST_BATCHED_BYTES = 700.0e6        # (10000 x 64^3 in FP32 moves 656e6)


def listed():
    return [
        # one small product, the smallest size of the square sweep: latency and the launch itself
        dict(name="sgemm_256", routine="gemm", dtype="f32", layout=COL, ta=N, tb=N, m=256, n=256, k=256, odd_ld=False,
             alpha=1.5, beta=0.5),
        # a large square product with a transposed operand that updates C, row-major as C and Python programs hold it
        dict(name="sgemm_4096_row_NT", routine="gemm", dtype="f32", layout=ROW, ta=N, tb=T, m=4096, n=4096, k=4096, odd_ld=False,
             alpha=1.0, beta=0.7),
        # sizes that are no multiple of any tile, odd leading dimensions (a sub-matrix of a larger one)
        dict(name="sgemm_1000x1001x999", routine="gemm", dtype="f32", layout=COL, ta=T, tb=N, m=1000, n=1001, k=999, odd_ld=True,
             alpha=1.0, beta=1.0),
        # a rank-64 update of a large C, the step of a blocked factorisation: memory, not arithmetic
        dict(name="sgemm_8192x8192x64", routine="gemm", dtype="f32", layout=COL, ta=T, tb=N, m=8192, n=8192, k=64, odd_ld=True,
             alpha=1.0, beta=1.0),
        # the product of a deep convolution layer: few outputs, a long sum
        dict(name="hgemm_512x196x2304", routine="gemm", dtype="f16", layout=COL, ta=N, tb=N, m=512, n=196, k=2304, odd_ld=False,
             alpha=1.0, beta=0.0),
        # the large square half-precision product
        dict(name="hgemm_4096", routine="gemm", dtype="f16", layout=COL, ta=N, tb=N, m=4096, n=4096, k=4096, odd_ld=False,
             alpha=1.0, beta=0.0),
        # half precision at an odd size with rows that start at odd elements
        dict(name="hgemm_2051_TN", routine="gemm", dtype="f16", layout=COL, ta=T, tb=N, m=2051, n=2051, k=2051, odd_ld=True,
             alpha=1.0, beta=0.5),
        # many tiny products in one call, each with its own scalars and place
        dict(name="sbatched_10000x16", routine="batched", dtype="f32", layout=COL, ta=N, tb=N, m=16, n=16, k=16, odd_ld=False,
             batch=10000, strided=False, beta=1.0),
        # products of the size that per-head score matrices have: Q K^T of 128 rows each
        dict(name="hbatched_512x128x128x64", routine="batched", dtype="f16", layout=ROW, ta=N, tb=T, m=128, n=128, k=64, odd_ld=False,
             batch=512, strided=True, beta=0.0),
        # a middle 3x3 convolution layer of one image, the whole call
        dict(name="hconv2d_128x28x28_f256", routine="conv", dtype="f16", channels=128, size=28, kernel=3, pad=1, stride=1, filters=256),
        # matrix-vector product in the plain order of column-major programs
        dict(name="sgemv_4096", routine="gemv", dtype="f32", layout=COL, ta=N, m=4096, n=4096, inc=1, odd_ld=False, beta=0.0),
        # a Gram matrix
        dict(name="hsyrk_4096", routine="syrk", dtype="f16", layout=COL, uplo=G.MG_LOWER, ta=N, n=4096, k=4096, odd_ld=False,
             beta=0.0),
    ]


# ------------------------------------------------------------------------------------------------ drawn cases

def _size(rng, lo, hi, unit=64):
    """spread over the logarithm of lo .. hi; two in five are multiples of `unit`"""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if v >= unit and rng.random() < 0.4:
        v = v // unit * unit
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(("gemm", "gemm", "gemm", "batched", "batched", "conv", "gemv", "level3"))
    dtype = rng.choice(("f32", "f16"))
    layout = rng.choice((COL, ROW))
    odd_ld = rng.random() < 0.3
    ta, tb = rng.choice((N, T)), rng.choice((N, T))
    beta = rng.choice((0.0, 0.5, 0.7))
    if kind == "gemm":
        while True:
            m, n, k = (_size(rng, 32, 8192) for _ in range(3))
            if 2.0 * m * n * k <= MOST_FLOPS:
                return dict(routine="gemm", dtype=dtype, layout=layout, ta=ta, tb=tb, m=m, n=n, k=k, odd_ld=odd_ld, alpha=1.0,
                            beta=beta)
    if kind == "batched":
        if rng.random() < 0.5:
            m = n = k = _size(rng, 8, 160, 8)
        else:
            m, n, k = (_size(rng, 8, 160, 8) for _ in range(3))
        batch = _size(rng, 200, 20000, 100)
        flops, size = 2.0 * m * n * k, (4.0 if dtype == "f32" else 2.0) * (m * k + k * n + 2 * m * n)
        batch = max(50, int(min(batch, MOST_BATCHED_FLOPS / flops, MOST_BATCHED_BYTES / size)))
        return dict(routine="batched", dtype=dtype, layout=layout, ta=ta, tb=tb, m=m, n=n, k=k, odd_ld=odd_ld, batch=batch,
                    strided=rng.random() < 0.5, beta=rng.choice((0.0, 1.0)))
    if kind == "conv":
        kernel = rng.choice((1, 3, 3, 3, 5, 7))
        size = _size(rng, max(7, kernel), 112, 7)
        channels = rng.choice((3, 16, _size(rng, 16, 512, 16), _size(rng, 16, 512, 16)))
        if kernel > 3:
            channels = min(channels, 64)
        return dict(routine="conv", dtype=dtype, channels=channels, size=size, kernel=kernel, pad=kernel // 2,
                    stride=rng.choice((1, 1, 2)), filters=_size(rng, 16, 512, 16))
    if kind == "gemv":
        return dict(routine="gemv", dtype=dtype, layout=layout, ta=ta, m=_size(rng, 64, 16384), n=_size(rng, 64, 16384),
                    inc=rng.choice((1, 1, 1, 2)), odd_ld=odd_ld, beta=beta)
    routine = rng.choice(("symm", "syrk", "trmm"))
    case = dict(routine=routine, dtype=dtype, layout=layout, uplo=rng.choice((G.MG_UPPER, G.MG_LOWER)), odd_ld=odd_ld)
    if routine == "syrk":
        return dict(case, ta=ta, n=_size(rng, 64, 4096), k=_size(rng, 64, 4096), beta=beta)
    case = dict(case, side=rng.choice((G.MG_LEFT, G.MG_RIGHT)), m=_size(rng, 64, 4096), n=_size(rng, 64, 4096))
    return dict(case, beta=beta) if routine == "symm" else dict(case, ta=ta)


# ------------------------------------------------------------------------------------------------ inputs

def _ld(minor, odd):
    return W.padded_ld(minor) if odd else minor


def _torch_type(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float16


def _code(case):
    return G.MG_F32 if case["dtype"] == "f32" else G.MG_F16


class _Draw:
    """buffers of the workloads' distributions: FP32 entries uniform in [-1, 1], FP16 ones normal with variance 1 / (length of the sum)"""

    def __init__(self, case, seed, length):
        self.type = _torch_type(case)
        self.sigma = float(max(1, length)) ** -0.5
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def __call__(self, count):
        if self.type == torch.float32:
            return torch.empty(count, device="cuda").uniform_(-1.0, 1.0, generator=self.gen)
        return torch.empty(count, device="cuda").normal_(0.0, self.sigma, generator=self.gen).to(torch.float16)

    def unit(self, count):
        """entries uniform in [-1, 1] in either type"""
        return torch.empty(count, device="cuda").uniform_(-1.0, 1.0, generator=self.gen).to(self.type)


def _workspace(count):
    return torch.empty(count, dtype=torch.uint8, device="cuda") if count else None


def _matrix(draw, layout, rows, cols, odd):
    """(buffer, leading dimension) of a stored rows x cols matrix"""
    minor, major = (rows, cols) if layout == COL else (cols, rows)
    ld = _ld(minor, odd)
    return draw(ld * major), ld


def _conv_geometry(case):
    pair = lambda v: (v, v)  # noqa: E731
    return case["channels"], case["size"], case["size"], pair(case["kernel"]), pair(case["pad"]), pair(case["stride"]), (1, 1)


def _conv_out(case):
    return W.conv_out_extent(case["size"], case["kernel"], case["pad"], case["stride"], 1)


def prepare(case, seed):
    s = dict(case)
    routine, code = case["routine"], _code(case)
    if routine == "gemm":
        m, n, k, layout = case["m"], case["n"], case["k"], case["layout"]
        draw_ = _Draw(case, seed, k)
        s["A"], s["lda"] = _matrix(draw_, layout, *W.stored_extents(case["ta"], m, k), case["odd_ld"])
        s["B"], s["ldb"] = _matrix(draw_, layout, *W.stored_extents(case["tb"], k, n), case["odd_ld"])
        s["C"], s["ldc"] = _matrix(draw_, layout, m, n, case["odd_ld"])
        s["ws"] = _workspace(G.mg_gemm_workspace_bytes(code, layout, case["ta"], case["tb"], m, n, k, s["lda"], s["ldb"], s["ldc"]))
    elif routine == "batched":
        m, n, k, layout, batch = case["m"], case["n"], case["k"], case["layout"], case["batch"]
        draw_ = _Draw(case, seed, k)
        for name, (rows, cols) in (("a", W.stored_extents(case["ta"], m, k)), ("b", W.stored_extents(case["tb"], k, n)), ("c", (m, n))):
            minor, major = (rows, cols) if layout == COL else (cols, rows)
            ld = _ld(minor, case["odd_ld"])
            # instances packed one behind the other; the generic form's lie seven elements apart
            stride = ld * major + (0 if case["strided"] else W.GAP)
            s[name.upper()], s["ld" + name], s["stride_" + name] = draw_.unit(stride * batch), ld, stride
            if not case["strided"]:
                s["off_" + name] = torch.arange(batch, dtype=torch.int64, device="cuda") * stride
        if not case["strided"]:
            # each instance has its own scalars; C is updated in place call after call, so the factors of the old C stay
            # below one (beta = 0: C is only written)
            s["alphas"] = torch.empty(batch, device="cuda").uniform_(0.5, 2.0, generator=draw_.gen)
            s["betas"] = torch.empty(batch, device="cuda").uniform_(0.5, 0.99, generator=draw_.gen) * (1.0 if case["beta"] else 0.0)
    elif routine == "conv":
        c, f, kk, o = case["channels"], case["filters"], case["channels"] * case["kernel"] ** 2, _conv_out(case)
        draw_ = _Draw(case, seed, kk)
        s["im"], s["weights"], s["out"] = draw_(c * case["size"] ** 2), draw_(f * kk), draw_(f * o * o)
        s["ws"] = _workspace(G.mg_conv2d_workspace_bytes(code, *_conv_geometry(case), f))
    elif routine == "gemv":
        m, n, layout, inc = case["m"], case["n"], case["layout"], case["inc"]
        rows, length = (m, n) if case["ta"] == N else (n, m)
        draw_ = _Draw(case, seed, length)
        s["A"], s["lda"] = _matrix(draw_, layout, m, n, case["odd_ld"])
        s["x"], s["y"] = draw_.unit(length * inc), draw_(rows * inc)
        s["ws"] = _workspace(G.mg_gemv_workspace_bytes(code, layout, case["ta"], m, n, s["lda"]))
    elif routine == "syrk":
        n, k, layout = case["n"], case["k"], case["layout"]
        draw_ = _Draw(case, seed, k)
        s["A"], s["lda"] = _matrix(draw_, layout, *((n, k) if case["ta"] == N else (k, n)), case["odd_ld"])
        s["C"], s["ldc"] = _matrix(draw_, layout, n, n, case["odd_ld"])
        s["ws"] = _workspace(G.mg_syrk_workspace_bytes(code, layout, case["ta"], n, k))
    else:
        m, n, layout = case["m"], case["n"], case["layout"]
        ka = m if case["side"] == G.MG_LEFT else n
        draw_ = _Draw(case, seed, ka)
        s["A"], s["lda"] = _matrix(draw_, layout, ka, ka, case["odd_ld"])
        s["B"], s["ldb"] = _matrix(draw_, layout, m, n, case["odd_ld"])
        if routine == "symm":
            s["C"], s["ldc"] = _matrix(draw_, layout, m, n, case["odd_ld"])
            s["ws"] = _workspace(G.mg_symm_workspace_bytes(code, layout, case["side"], m, n))
        else:
            s["B_given"] = s["B"].clone()
            s["ws"] = _workspace(G.mg_trmm_workspace_bytes(code, layout, case["side"], case["ta"], m, n))
    return s


# ------------------------------------------------------------------------------------------------ the calls

def run(s):
    routine, f32 = s["routine"], s["dtype"] == "f32"
    if routine == "gemm":
        call = G.mg_sgemm if f32 else G.mg_hgemm
        call(s["layout"], s["ta"], s["tb"], s["m"], s["n"], s["k"], s["alpha"], s["A"], s["lda"], s["B"], s["ldb"], s["beta"], s["C"],
             s["ldc"], s["ws"])
        return s["C"]
    if routine == "batched":
        if s["strided"]:
            call = G.mg_sgemm_strided_batched if f32 else G.mg_hgemm_strided_batched
            call(s["layout"], s["ta"], s["tb"], s["m"], s["n"], s["k"], 1.0, s["A"], s["lda"], s["stride_a"], s["B"], s["ldb"],
                 s["stride_b"], 0.5 if s["beta"] else 0.0, s["C"], s["ldc"], s["stride_c"], s["batch"])
        else:
            call = G.mg_sgemm_batched if f32 else G.mg_hgemm_batched
            call(s["layout"], s["ta"], s["tb"], s["m"], s["n"], s["k"], s["alphas"], s["A"], s["off_a"], s["lda"], s["B"], s["off_b"],
                 s["ldb"], s["betas"], s["C"], s["off_c"], s["ldc"], s["batch"])
        return s["C"]
    if routine == "conv":
        call = G.mg_sconv2d if f32 else G.mg_hconv2d
        call(*_conv_geometry(s), s["filters"], 1.0, s["im"], s["weights"], 0.0, s["out"], s["ws"])
        return s["out"]
    if routine == "gemv":
        call = G.mg_sgemv if f32 else G.mg_hgemv
        call(s["layout"], s["ta"], s["m"], s["n"], 1.0, s["A"], s["lda"], s["x"], s["inc"], s["beta"], s["y"], s["inc"], s["ws"])
        return s["y"]
    if routine == "syrk":
        call = G.mg_ssyrk if f32 else G.mg_hsyrk
        call(s["layout"], s["uplo"], s["ta"], s["n"], s["k"], 1.0, s["A"], s["lda"], s["beta"], s["C"], s["ldc"], s["ws"])
        return s["C"]
    if routine == "symm":
        call = G.mg_ssymm if f32 else G.mg_hsymm
        call(s["layout"], s["side"], s["uplo"], s["m"], s["n"], 1.0, s["A"], s["lda"], s["B"], s["ldb"], s["beta"], s["C"], s["ldc"],
             s["ws"])
        return s["C"]
    # the product replaces B: a program that needs the same B again keeps it and copies it in
    s["B"].copy_(s["B_given"])
    call = G.mg_strmm if f32 else G.mg_htrmm
    call(s["layout"], s["side"], s["uplo"], s["ta"], G.MG_NON_UNIT, s["m"], s["n"], 1.0, s["A"], s["lda"], s["B"], s["ldb"], s["ws"])
    return s["B"]


# ------------------------------------------------------------------------------------------------ what they cannot do without

def work(case):
    e = 4.0 if case["dtype"] == "f32" else 2.0
    routine = case["routine"]
    if routine == "conv":
        c, f, kk, o = case["channels"], case["filters"], case["channels"] * case["kernel"] ** 2, _conv_out(case)
        return {"bytes": e * (c * case["size"] ** 2 + f * kk + f * o * o), "flops": 2.0 * f * kk * o * o}
    if routine == "gemv":
        m, n = case["m"], case["n"]
        rows, length = (m, n) if case["ta"] == N else (n, m)
        return {"bytes": e * (m * n + length + rows * (2 if case["beta"] else 1)), "flops": 2.0 * m * n}
    if routine == "syrk":
        n, k, half = case["n"], case["k"], case["n"] * (case["n"] + 1) / 2
        return {"bytes": e * (n * k + half * (2 if case["beta"] else 1)), "flops": 2.0 * half * k}
    if routine in ("symm", "trmm"):
        m, n = case["m"], case["n"]
        ka = m if case["side"] == G.MG_LEFT else n
        half = ka * (ka + 1) / 2
        if routine == "symm":
            return {"bytes": e * (half + m * n * (3 if case["beta"] else 2)), "flops": 2.0 * m * n * ka}
        return {"bytes": e * (half + 2 * m * n), "flops": 2.0 * half * (m * n / ka)}
    m, n, k = case["m"], case["n"], case["k"]
    one = {"bytes": e * (m * k + k * n + m * n * (2 if case["beta"] else 1)), "flops": 2.0 * m * n * k}
    if routine == "gemm":
        return one
    per = 0.0 if case["strided"] else 8.0 + 24.0        # two scalars and three offsets per instance
    return {"bytes": case["batch"] * (one["bytes"] + per), "flops": case["batch"] * one["flops"]}


def tolerance(case):
    """four times what the products above differ from their value in 64 bits"""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5}           # 4096 terms: 1.15e-6 and 1.0e-5
    return {"rel": 8.5e-4, "max": 2e-3}             # one rounding to FP16: 2.1e-4 and 4.9e-4
