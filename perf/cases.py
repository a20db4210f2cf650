"""The work whose speed counts: what a program that uses this library has it do on one GPU.

Every path goes through the public entry points of ``paper_2105_14450_amd`` as such a program calls
them: buffers, descriptors and workspaces made once, the calls enqueued on the current stream one
after the other.

Paths
  rank        one processor's share of a linear layer at its real shape, the program of a cluster
              with one process per GPU: the three block products, forward and backward
  cube        a linear layer on the virtual cube through the explicit collectives: all-gathers, the
              batched products, reduce-scatters, the bias and its gradient, forward and backward
  mlp_serve   two in-place linears with bias around the activation, forward only, few tokens
  mlp_train   the same block forward and backward, with every gradient
  forms       the three product forms on matrices placed on the cube (C = A B and its backward pass)
  storage     full matrices spread over the cube's shards and collected again (loading parameters and
              a batch, saving results)

Sizes: M tokens, K input features, N output features of the whole layer, q the side of the cube.
"""
import torch

import paper_2105_14450_amd as c3

DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8_e4m3": torch.float8_e4m3fn}
CODE = {"f32": c3.F32, "bf16": c3.BF16, "fp8_e4m3": c3.FP8_E4M3}
BYTES = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}
ACT = {"relu": c3.ACT_RELU, "gelu": c3.ACT_GELU}
E4M3_MAX = 448.0


def listed():
    return [
        # the small fp32 layer of the benchmark, whole cube: thirteen short launches, latency only
        {"name": "cube-f32-tiny", "path": "cube", "dtype": "f32", "out": "f32", "q": 2, "M": 256, "K": 128, "N": 128},
        # a decoding step: 64 sequences, one token each, through the MLP block of the benchmarked layer
        {"name": "serve-bf16-64-tokens", "path": "mlp_serve", "dtype": "bf16", "act": "gelu", "q": 4, "M": 64, "K": 2048, "N": 8192},
        # one processor of 64, hidden 2048, 16 sequences of 512 tokens: the smallest training share of the benchmark
        {"name": "rank-bf16-small", "path": "rank", "dtype": "bf16", "out": "bf16", "q": 4, "M": 8192, "K": 2048, "N": 8192},
        # the same with 16 sequences of 500 tokens and hidden 1600: nothing is a multiple of a large tile
        {"name": "rank-bf16-ragged", "path": "rank", "dtype": "bf16", "out": "bf16", "q": 4, "M": 8000, "K": 1600, "N": 6400},
        # single precision training of the small share
        {"name": "rank-f32", "path": "rank", "dtype": "f32", "out": "f32", "q": 4, "M": 8192, "K": 2048, "N": 8192},
        # one processor of 64, hidden 8192, 32768 tokens: the headline of the benchmark
        {"name": "rank-bf16-large", "path": "rank", "dtype": "bf16", "out": "bf16", "q": 4, "M": 32768, "K": 8192, "N": 32768},
        # one processor of 512, hidden 12288, fp8 operands with per-tensor scales
        {"name": "rank-fp8", "path": "rank", "dtype": "fp8_e4m3", "out": "bf16", "q": 8, "M": 16384, "K": 12288, "N": 49152},
        # the MLP up-projection on 64 virtual processors through the collectives, fp32 partial products
        {"name": "cube-bf16-mlp-up", "path": "cube", "dtype": "bf16", "out": "f32", "q": 4, "M": 8192, "K": 2048, "N": 8192},
        # a linear of hidden 3072 on 8 virtual processors as three placed products, fp8, 6 sequences of 500 tokens
        {"name": "forms-fp8", "path": "forms", "dtype": "fp8_e4m3", "q": 2, "M": 3000, "K": 3072, "N": 12288},
        # the training step of the MLP block on 27 virtual processors, 9 sequences of 333 tokens
        {"name": "train-bf16-ragged", "path": "mlp_train", "dtype": "bf16", "act": "gelu", "q": 3, "M": 2997, "K": 1152, "N": 4608},
        # the training step of the MLP block of the benchmarked layer on 64 virtual processors
        {"name": "train-bf16-layer", "path": "mlp_train", "dtype": "bf16", "act": "gelu", "q": 4, "M": 8192, "K": 2048, "N": 8192},
        # loading and saving: the parameters and a batch of the same layer to shards and back
        {"name": "storage-bf16", "path": "storage", "dtype": "bf16", "q": 4, "M": 8192, "K": 2048, "N": 8192},
    ]


# ---- drawn cases ------------------------------------------------------------------------------------

# multiply-adds a drawn case may have, times what its arithmetic costs against bf16: the largest listed case's
LIMIT_FLOPS = 12.0 * 8192 * 2048 * 8192
LIMIT_CUBE = 8192.0 * 8192     # largest matrix of a drawn cube: bounds its gathered copies and partial products


def _between(rng, lo, hi):
    """Log-uniform."""
    return lo * (hi / lo) ** rng.random()


def _multiple(value, unit):
    return unit * max(1, round(value / unit))


def draw(rng):
    while True:
        case, odd = _draw_once(rng)
        cost = work(case)["flops"] * (16 if case["dtype"] == "f32" or odd else 1)
        largest = max(case["M"], case["K"]) * case["N"]
        if cost <= LIMIT_FLOPS and (case["path"] == "rank" or largest <= LIMIT_CUBE):
            return case


def _draw_once(rng):
    path = rng.choice(("rank", "rank", "cube", "mlp_serve", "mlp_train", "forms", "storage"))
    q = rng.choice((2, 3, 4, 8) if path == "rank" else (2, 3, 4))
    # features per shard: mostly what hidden sizes are multiples of, now and then any number
    step = rng.choice((128, 64, 32, 16, 8, rng.choice((4, 2, 1))))
    feat = lambda lo, hi: _multiple(_between(rng, lo, hi), q * q * step)
    tokens = lambda lo, hi: _multiple(_between(rng, lo, hi), q * q * rng.choice((1, 1, 16, 128)))
    case = {"path": path, "q": q, "dtype": rng.choice(("bf16", "bf16", "bf16", "fp8_e4m3", "f32"))}
    if path == "rank":
        case.update(M=tokens(q * 64, q * 8192), K=feat(q * 128, q * 2048), N=feat(q * 256, q * 8192),
                    out=rng.choice(("f32", "bf16")))
    elif path == "cube":
        case.update(M=tokens(256, 8192), K=feat(128, 8192), N=feat(128, 8192), out=rng.choice(("f32", "bf16")))
    elif path == "mlp_serve":
        hidden = feat(512, 2048)
        case.update(M=tokens(16, 1024), K=hidden, N=4 * hidden, act=rng.choice(("relu", "gelu")))
    elif path == "mlp_train":
        hidden = feat(512, 2048)
        case.update(M=tokens(1024, 8192), K=hidden, N=4 * hidden, act=rng.choice(("relu", "gelu")))
    else:
        case.update(M=tokens(256, 8192), K=feat(128, 8192), N=feat(128, 8192))
    if path in ("mlp_serve", "mlp_train") and case["dtype"] == "fp8_e4m3":
        case["dtype"] = "bf16"     # the block's activations are bf16 or fp32
    if case["dtype"] == "f32":
        case.update({"out": "f32"} if "out" in case else {})
    return case, step < 8


# ---- inputs -----------------------------------------------------------------------------------------

class _Make:
    """Seeded device tensors of a storage type; fp8 with the per-tensor scale amax / 448."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, shape, dtype, sigma=1.0):
        t = torch.randn(shape, device="cuda", generator=self.gen).mul_(sigma)
        if dtype != "fp8_e4m3":
            return t.to(DTYPE[dtype]), 1.0
        scale = float(t.abs().max()) / E4M3_MAX
        return t.div_(scale).clamp_(-E4M3_MAX, E4M3_MAX).to(DTYPE[dtype]), scale


def _empty(shape, dtype):
    return torch.empty(shape, dtype=DTYPE[dtype], device="cuda")


def _scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def _shard_dtype(dtype):
    return "f32" if dtype == "f32" else "bf16"


def _desc(q, M, K, N, dtype, out, axis=c3.AXIS_Y, scales=(1.0, 1.0, 1.0)):
    return c3.make_desc(q, M, K, N, in_dtype=CODE[dtype], out_dtype=CODE[out], shard_dtype=CODE[_shard_dtype(dtype)],
                        in_axis=axis, scale_x=scales[0], scale_w=scales[1], scale_dy=scales[2])


def prepare(case, seed):
    return _PREPARE[case["path"]](case, _Make(seed))


def run(state):
    return _RUN[state["path"]](state)


# one processor's blocks: X [M/q, K/q], W [K/q, N/q], dY [M/q, N/q]
def _prepare_rank(case, make):
    q, M, K, N, dt, out = (case[k] for k in ("q", "M", "K", "N", "dtype", "out"))
    Mb, Kb, Nb = M // q, K // q, N // q
    (X, sx), (W, sw), (G, sg) = make.normal((Mb, Kb), dt), make.normal((Kb, Nb), dt, 0.02), make.normal((Mb, Nb), dt)
    d = _desc(q, M, K, N, dt, out, scales=(sx, sw, sg))
    return {"path": "rank", "d": d, "rank": (q - 1, 0, q // 2), "X": X, "W": W, "G": G,
            "P": _empty((Mb, Nb), out), "Q": _empty((Mb, Kb), out), "R": _empty((Kb, Nb), out),
            "ws": [_scratch(c3.cube3d_workspace_bytes(d, op, False)) for op in (c3.OP_FWD, c3.OP_BWD_DX, c3.OP_BWD_DW)]}


def _run_rank(s):
    c3.cube3d_linear_fwd(s["d"], s["rank"], s["X"], s["W"], s["P"], s["ws"][0])
    c3.cube3d_linear_bwd_dx(s["d"], s["rank"], s["G"], s["W"], s["Q"], s["ws"][1])
    c3.cube3d_linear_bwd_dw(s["d"], s["rank"], s["X"], s["G"], s["R"], s["ws"][2])
    return s["P"], s["Q"], s["R"]


# the whole cube: shards in, shards out, the gathered blocks and partial products between them
def _prepare_cube(case, make):
    q, M, K, N, dt, out = (case[k] for k in ("q", "M", "K", "N", "dtype", "out"))
    n, sd = q ** 3, _shard_dtype(dt)
    Mb, Kb, Nb, Ms, Ns = M // q, K // q, N // q, M // q ** 2, N // q ** 2
    (X, sx), (W, sw), (G, sg) = make.normal((n, Ms, Kb), dt), make.normal((n, Kb, Ns), dt, 0.02), make.normal((n, Ms, Nb), dt)
    bias, _ = make.normal((n, Ns), "f32", 0.02)
    d = _desc(q, M, K, N, dt, out, scales=(sx, sw, sg))
    s = {"path": "cube", "d": d, "X": X, "W": W, "G": G, "bias": bias,
         "Xb": _empty((n, Mb, Kb), dt), "Wb": _empty((n, Kb, Nb), dt), "Gb": _empty((n, Mb, Nb), dt), "bb": _empty((n, Nb), "f32"),
         "P": _empty((n, Mb, Nb), out), "Q": _empty((n, Mb, Kb), out), "R": _empty((n, Kb, Nb), out),
         "Y": _empty((n, Ms, Nb), sd), "dX": _empty((n, Ms, Kb), sd), "dW": _empty((n, Kb, Ns), sd), "db": _empty((n, Ns), "f32"),
         "ws": [_scratch(c3.cube3d_workspace_bytes(d, op, True))
                for op in (c3.OP_FWD, c3.OP_BWD_DX, c3.OP_BWD_DW, c3.OP_BIAS_BWD)]}
    return s


def _run_cube(s):
    d = s["d"]
    # Algorithms 1 and 7
    c3.virtual_cube_gather(d, c3.OPERAND_X, c3.AXIS_Y, s["X"], s["Xb"])
    c3.virtual_cube_gather(d, c3.OPERAND_W, c3.AXIS_X, s["W"], s["Wb"])
    c3.virtual_cube_bias_gather(d, s["bias"], s["bb"])
    c3.cube3d_linear_fwd(d, c3.ALL_RANKS, s["Xb"], s["Wb"], s["P"], s["ws"][0])
    c3.virtual_cube_reduce_scatter_bias(d, c3.AXIS_Z, s["P"], s["bb"], s["Y"])
    # Algorithms 2 and 8
    c3.virtual_cube_gather(d, c3.OPERAND_DY, c3.AXIS_Z, s["G"], s["Gb"])
    c3.cube3d_linear_bwd_dx(d, c3.ALL_RANKS, s["Gb"], s["Wb"], s["Q"], s["ws"][1])
    c3.virtual_cube_reduce_scatter(d, c3.OPERAND_DX, c3.AXIS_Y, s["Q"], s["dX"])
    c3.cube3d_linear_bwd_dw(d, c3.ALL_RANKS, s["Xb"], s["Gb"], s["R"], s["ws"][2])
    c3.virtual_cube_reduce_scatter(d, c3.OPERAND_DW, c3.AXIS_X, s["R"], s["dW"])
    c3.virtual_cube_bias_bwd(d, s["G"], s["db"], s["ws"][3])
    return s["Y"], s["dX"], s["dW"], s["db"]


# two linears around the activation, shards read and written in place; the first gathers its input in
# y, the second in z, so that the activation's output is the second one's input as stored
def _prepare_mlp(case, make):
    q, M, K, N, dt = (case[k] for k in ("q", "M", "K", "N", "dtype"))
    n = q ** 3
    Kb, Nb, Ms = K // q, N // q, M // q ** 2
    s = {"path": case["path"], "kind": ACT[case["act"]], "dt": CODE[dt],
         "d1": _desc(q, M, K, N, dt, "f32"), "d2": _desc(q, M, N, K, dt, "f32", axis=c3.AXIS_Z),
         "X": make.normal((n, Ms, Kb), dt)[0],
         "W1": make.normal((n, Kb, N // q ** 2), dt, 0.02)[0], "b1": make.normal((n, N // q ** 2), "f32", 0.02)[0],
         "W2": make.normal((n, Nb, K // q ** 2), dt, 0.02)[0], "b2": make.normal((n, K // q ** 2), "f32", 0.02)[0],
         "Z": _empty((n, Ms, Nb), dt), "H": _empty((n, Ms, Nb), dt), "Y": _empty((n, Ms, Kb), dt)}
    if case["path"] == "mlp_train":
        s.update(G=make.normal((n, Ms, Kb), dt)[0], dH=_empty((n, Ms, Nb), dt), dZ=_empty((n, Ms, Nb), dt),
                 dX=_empty((n, Ms, Kb), dt), dW1=_empty(s["W1"].shape, dt), dW2=_empty(s["W2"].shape, dt),
                 db1=_empty(s["b1"].shape, "f32"), db2=_empty(s["b2"].shape, "f32"),
                 ws1=_scratch(c3.cube3d_workspace_bytes(s["d1"], c3.OP_BIAS_BWD, True)),
                 ws2=_scratch(c3.cube3d_workspace_bytes(s["d2"], c3.OP_BIAS_BWD, True)))
    return s


def _run_mlp_serve(s):
    c3.virtual_cube_linear_fwd(s["d1"], s["X"], s["W1"], s["b1"], s["Z"])
    c3.cube3d_activation_fwd(s["kind"], s["dt"], s["dt"], s["Z"], s["H"])
    c3.virtual_cube_linear_fwd(s["d2"], s["H"], s["W2"], s["b2"], s["Y"])
    return s["Y"]


def _run_mlp_train(s):
    _run_mlp_serve(s)
    c3.virtual_cube_bias_bwd(s["d2"], s["G"], s["db2"], s["ws2"])
    c3.virtual_cube_linear_bwd_dw(s["d2"], s["H"], s["G"], s["dW2"])
    c3.virtual_cube_linear_bwd_dx(s["d2"], s["G"], s["W2"], s["dH"])
    c3.cube3d_activation_bwd(s["kind"], s["dt"], s["dt"], s["dt"], s["Z"], s["dH"], s["dZ"])
    c3.virtual_cube_bias_bwd(s["d1"], s["dZ"], s["db1"], s["ws1"])
    c3.virtual_cube_linear_bwd_dw(s["d1"], s["X"], s["dZ"], s["dW1"])
    c3.virtual_cube_linear_bwd_dx(s["d1"], s["dZ"], s["W1"], s["dX"])
    return s["Y"], s["dX"], s["dW1"], s["dW2"], s["db1"], s["db2"]


# C = A B with the placements of the paper's Section 3.1.1, then dA = dC B^T and dB = A^T dC
def _prepare_forms(case, make):
    q, M, K, N, dt = (case[k] for k in ("q", "M", "K", "N", "dtype"))
    n, sd = q ** 3, _shard_dtype(dt)
    x, y, z = c3.AXIS_X, c3.AXIS_Y, c3.AXIS_Z
    placed = lambda rows, cols, ra, ca, split, t: c3.make_matrix(q, rows, cols, ra, ca, split, CODE[t])
    A, B = (lambda t: placed(M, K, x, z, c3.SPLIT_ROWS, t)), (lambda t: placed(K, N, z, y, c3.SPLIT_COLS, t))
    C = lambda t: placed(M, N, x, y, c3.SPLIT_ROWS, t)
    (a, sa), (b, sb), (g, sg) = (make.normal((n, M // q ** 2, K // q), dt), make.normal((n, K // q, N // q ** 2), dt, 0.02),
                                 make.normal((n, M // q ** 2, N // q), dt))
    return {"path": "forms", "A": A(dt), "B": B(dt), "G": C(dt), "C": C(sd), "dA": A(sd), "dB": B(sd),
            "a": a, "b": b, "g": g, "scales": (sa, sb, sg),
            "c": _empty((n, M // q ** 2, N // q), sd), "da": _empty(a.shape, sd), "db": _empty(b.shape, sd)}


def _run_forms(s):
    sa, sb, sg = s["scales"]
    c3.virtual_cube_matmul(c3.FORM_AB, s["A"], s["B"], s["C"], s["a"], s["b"], s["c"], sa, sb)
    c3.virtual_cube_matmul(c3.FORM_ABT, s["G"], s["B"], s["dA"], s["g"], s["b"], s["da"], sg, sb)
    c3.virtual_cube_matmul(c3.FORM_ATB, s["A"], s["G"], s["dB"], s["a"], s["g"], s["db"], sa, sg)
    return s["c"], s["da"], s["db"]


def _prepare_storage(case, make):
    q, M, K, N, dt = (case[k] for k in ("q", "M", "K", "N", "dtype"))
    n, sd = q ** 3, _shard_dtype(dt)
    Kb, Nb, Ms, Ns = K // q, N // q, M // q ** 2, N // q ** 2
    return {"path": "storage", "d": _desc(q, M, K, N, dt, "f32"),
            "X": make.normal((M, K), dt)[0], "W": make.normal((K, N), dt, 0.02)[0],
            "y": make.normal((n, Ms, Nb), sd)[0], "dw": make.normal((n, Kb, Ns), sd)[0],
            "x": _empty((n, Ms, Kb), dt), "w": _empty((n, Kb, Ns), dt), "Y": _empty((M, N), sd), "dW": _empty((K, N), sd)}


def _run_storage(s):
    c3.virtual_cube_scatter(s["d"], c3.OPERAND_X, s["X"], s["x"])
    c3.virtual_cube_scatter(s["d"], c3.OPERAND_W, s["W"], s["w"])
    c3.virtual_cube_assemble(s["d"], c3.OPERAND_Y, s["y"], s["Y"])
    c3.virtual_cube_assemble(s["d"], c3.OPERAND_DW, s["dw"], s["dW"])
    return s["x"], s["w"], s["Y"], s["dW"]


_PREPARE = {"rank": _prepare_rank, "cube": _prepare_cube, "mlp_serve": _prepare_mlp, "mlp_train": _prepare_mlp,
            "forms": _prepare_forms, "storage": _prepare_storage}
_RUN = {"rank": _run_rank, "cube": _run_cube, "mlp_serve": _run_mlp_serve, "mlp_train": _run_mlp_train,
        "forms": _run_forms, "storage": _run_storage}


# ---- what a pass cannot do without, and how exact it is ------------------------------------------------

def work(case):
    """Bytes: every input once and every result that the pass hands back once.  The cube path's gathered
    blocks and partial products are results of the calls that make them and count as written once; the
    MLP block's intermediate activations do not count."""
    path, q, M, K, N, dt = (case[k] for k in ("path", "q", "M", "K", "N", "dtype"))
    e, so = BYTES[dt], BYTES[_shard_dtype(dt)]
    x, w, y = M * K, K * N, M * N
    if path == "rank":
        o = BYTES[case["out"]]
        return {"bytes": (x + w + y) // q ** 2 * (e + o), "flops": 6 * M * K * N // q ** 3}
    if path == "cube":
        o = BYTES[case["out"]]
        return {"bytes": (x + w + y) * (e + e * q + o * q + so) + N * 4 * (2 + q * q), "flops": 6 * M * K * N}
    if path == "forms":
        return {"bytes": (x + w + y) * (e + so), "flops": 6 * M * K * N}
    if path == "storage":
        return {"bytes": 2 * (x + w) * e + 2 * (y + w) * so, "flops": 0}
    if path == "mlp_serve":
        return {"bytes": 2 * (x + w) * e + (K + N) * 4, "flops": 4 * M * K * N}
    return {"bytes": (4 * x + 4 * w) * e + 2 * (K + N) * 4, "flops": 12 * M * K * N}


def tolerance(case):
    """About four times the largest error of any result of the path against fp64 (2-norm, and largest
    element over the larger of its value and the root mean square), over the listed and some drawn sizes."""
    path, dt, out = case["path"], case["dtype"], case.get("out")
    if path == "storage":                       # copies
        return "exact"
    if dt == "f32":                             # the order of the sums: 1.6e-6 through the MLP block, else 8e-7
        return {"rel": 6e-6, "max": 4e-5} if path.startswith("mlp") else {"rel": 4e-6, "max": 3e-5}
    if path == "rank" and out == "f32":         # exact products, fp32 sums; fp8: the matrix cores' own sums, 1.5e-5
        return {"rel": 6e-5, "max": 6e-4} if dt == "fp8_e4m3" else {"rel": 4e-6, "max": 3e-5}
    if path.startswith("mlp"):                  # bf16 roundings of three or four stages: 3.2e-3
        return {"rel": 1.2e-2, "max": 7e-2}
    if path == "cube" and out == "bf16":        # bf16 partial products, summed and rounded again: 2.4e-3
        return {"rel": 1e-2, "max": 6e-2}
    return {"rel": 6e-3, "max": 1.6e-2}         # one bf16 rounding: 1.7e-3


# ---- the same results in 64 bits ----------------------------------------------------------------------

def _f64(t, scale=1.0):
    return t.float().double() * scale


def _by_direction(t, q, axis):
    """Cube buffer as [i, a, b, ...]: a along the input direction, b along the output direction."""
    t = t.reshape(q, q, q, *t.shape[1:])
    return t if axis == c3.AXIS_Y else t.transpose(1, 2)


# order of (i, a, b, rows of a shard, columns of a shard) in the full matrix: (row indices), (column indices)
_ORDER = {"x": ((0, 1, 3), (2, 4)), "w": ((2, 3), (1, 0, 4)), "y": ((0, 2, 3), (1, 4))}


def _whole(which, t, q, axis=c3.AXIS_Y):
    """Full matrix of a cube of shards."""
    rows, cols = _ORDER[which]
    t = _by_direction(t, q, axis).permute(*rows, *cols)
    return t.reshape(t.shape[:len(rows)].numel(), -1)


def _spread(which, full, q, axis=c3.AXIS_Y):
    """Cube of shards of a full matrix."""
    rows, cols = _ORDER[which]
    cut = lambda n, order: [q] * (len(order) - 1) + [n // q ** (len(order) - 1)]
    order = rows + cols
    t = full.reshape(*cut(full.shape[0], rows), *cut(full.shape[1], cols)).permute(*[order.index(d) for d in range(5)])
    t = t if axis == c3.AXIS_Y else t.transpose(1, 2)
    return t.reshape(q ** 3, *t.shape[3:])


def _whole_bias(t, q):
    return t.reshape(q, q, q, -1).diagonal(dim1=1, dim2=2).permute(2, 0, 1).reshape(-1)


def _spread_bias(full, q):
    t = full.new_zeros(q, q, q, full.numel() // q ** 2)
    for a in range(q):
        t[:, a, a] = full.reshape(q, q, -1)[a]
    return t.reshape(q ** 3, -1)


def exact(case, seed):
    s, q, path = prepare(case, seed), case["q"], case["path"]
    if path == "storage":
        return (_spread("x", _f64(s["X"]), q), _spread("w", _f64(s["W"]), q),
                _f64(_whole("y", s["y"], q)), _f64(_whole("w", s["dw"], q)))
    if path.startswith("mlp"):
        return _exact_mlp(s, q, path == "mlp_train")
    if path == "forms":
        sx, sw, sg = s["scales"]
        x, w, g = _whole("x", s["a"], q), _whole("w", s["b"], q), _whole("y", s["g"], q)
    else:
        sx, sw, sg = s["d"].scale_x, s["d"].scale_w, s["d"].scale_dy
        x, w, g = s["X"], s["W"], s["G"]
        if path == "cube":
            x, w, g = _whole("x", x, q), _whole("w", w, q), _whole("y", g, q)
    x, w, g = _f64(x, sx), _f64(w, sw), _f64(g, sg)
    y, dx, dw = x @ w, g @ w.t(), x.t() @ g
    if path == "rank":
        return y, dx, dw
    if path == "forms":
        return _spread("y", y, q), _spread("x", dx, q), _spread("w", dw, q)
    y += _whole_bias(_f64(s["bias"]), q)
    return _spread("y", y, q), _spread("x", dx, q), _spread("w", dw, q), _spread_bias(g.sum(0), q)


def _exact_mlp(s, q, train):
    # the hidden activations are the first linear's output (axis y) and the second one's input (axis z)
    z_ax = c3.AXIS_Z
    x, w1, w2 = (_f64(t) for t in (_whole("x", s["X"], q), _whole("w", s["W1"], q), _whole("w", s["W2"], q, z_ax)))
    z = x @ w1 + _whole_bias(_f64(s["b1"]), q)
    gelu = s["kind"] == c3.ACT_GELU
    cdf = 0.5 * torch.erfc(z * -0.5 ** 0.5) if gelu else (z > 0).double()
    h = z * cdf
    y = h @ w2 + _whole_bias(_f64(s["b2"]), q)
    out = _spread("y", y, q, z_ax)
    if not train:
        return out
    g = _f64(_whole("y", s["G"], q, z_ax))
    slope = cdf + z * torch.exp(-0.5 * z * z) * (2 * torch.pi) ** -0.5 if gelu else cdf
    dz = (g @ w2.t()) * slope
    return (out, _spread("x", dz @ w1.t(), q), _spread("w", x.t() @ dz, q), _spread("w", h.t() @ g, q, z_ax),
            _spread_bias(dz.sum(0), q), _spread_bias(g.sum(0), q))
