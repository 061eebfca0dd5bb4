"""The work a program has this framework do, as timed cases.

A case is one layer of a task chain (a contraction with its epilogue kernels),
one point cloud, or one whole frame through the launch gate.  Layers go
through the C-ABI's direct launch (``ug_kernel_launch``) with descriptors
marshalled once, as a program keeps them; the frame goes through a started
gate.  Sizes are those of the repository's workload configurations, tests and
benchmark: GEMMs of 256 to 4096 a side, 3x3 convolutions of 16 to 256 channels
on images of 32 to 336 pixels a side, row kernels that follow them, clouds of
20 thousand to 8 million points, FP8 products of the best-effort load.
"""

import ctypes

import torch
import torch.nn.functional as F

from paper_2509_12207_amd import capi

DEV = "cuda"
GRID = (512, 512)                       # bird's-eye-view cells
GRID_PARAM = (-51.2, -51.2, 5.0)        # xmin, ymin, cells per metre


def listed():
    return [
        # the smallest call: one frame of configuration 0's chain (three tasks
        # of GEMM, bias+ReLU, 3x3 convolution, row sum) through the gate,
        # where launches, events and decisions are the time
        {"name": "frame_cfg0", "kind": "frame", "tasks": 3, "dim": 128, "ch": 16, "img": 64},
        # the smallest dense layer the chains draw
        {"name": "dense_f32_256", "kind": "dense", "dtype": "f32", "m": 256, "n": 256, "k": 256,
         "softmax": False, "rowsum": False},
        # an ordinary dense layer of a text or detection task, every epilogue
        {"name": "dense_f32_1280x2048x1024", "kind": "dense", "dtype": "f32", "m": 1280,
         "n": 2048, "k": 1024, "softmax": True, "rowsum": True},
        # a frame-sized, odd product: no side a multiple of four
        {"name": "dense_f32_1003x2050x1021", "kind": "dense", "dtype": "f32", "m": 1003,
         "n": 2050, "k": 1021, "softmax": True, "rowsum": False},
        # the largest FP32 layer of the chains
        {"name": "dense_f32_4096", "kind": "dense", "dtype": "f32", "m": 4096, "n": 4096,
         "k": 4096, "softmax": True, "rowsum": True},
        # an ordinary camera layer
        {"name": "conv_f32_c128_128", "kind": "conv", "dtype": "f32", "c": 128, "h": 128,
         "w": 128, "rowsum": True},
        # a serving layer at a frame's own image size
        {"name": "conv_f32_c64_84", "kind": "conv", "dtype": "f32", "c": 64, "h": 84, "w": 84,
         "rowsum": False},
        # an ordinary dense layer of the BF16 chains
        {"name": "dense_bf16_1280x1792x768", "kind": "dense", "dtype": "bf16", "m": 1280,
         "n": 1792, "k": 768, "softmax": True, "rowsum": False},
        # an ordinary camera layer of the BF16 chains
        {"name": "conv_bf16_c64_128", "kind": "conv", "dtype": "bf16", "c": 64, "h": 128,
         "w": 128, "rowsum": True},
        # the best-effort load of an overloaded GPU: a row band of its FP8 product
        {"name": "gemm_fp8_2048x8192x8192", "kind": "dense", "dtype": "fp8", "m": 2048,
         "n": 8192, "k": 8192, "softmax": False, "rowsum": False},
        # one LiDAR frame
        {"name": "voxel_100k", "kind": "voxel", "points": 100_000},
        # an accumulated map cloud, past the size where points are binned first
        {"name": "voxel_8M", "kind": "voxel", "points": 8_000_000},
    ]


def _log_int(rng, lo, hi, step=1):
    v = lo * (hi / lo) ** rng.random()
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["frame", "dense", "dense", "dense", "dense", "conv", "conv", "conv",
                       "voxel"])
    if kind == "frame":
        return {"kind": kind, "tasks": rng.randint(2, 6), "dim": _log_int(rng, 64, 512, 4),
                "ch": 16 * rng.randint(1, 4), "img": _log_int(rng, 32, 128)}
    if kind == "voxel":
        return {"kind": kind, "points": _log_int(rng, 20_000, 8_000_000)}
    if kind == "conv":
        dtype = rng.choice(["f32", "bf16"])
        c = _log_int(rng, 32, 256, 32) if dtype == "bf16" else _log_int(rng, 16, 256, 4)
        h = _log_int(rng, 32, 336 if c <= 64 else 256)
        # most images are square; some are not
        w = h if rng.random() < 0.7 else _log_int(rng, 32, 256)
        return {"kind": kind, "dtype": dtype, "c": c, "h": h, "w": w,
                "rowsum": rng.random() < 0.3}
    dtype = rng.choice(["f32", "f32", "bf16", "fp8"])
    # the chains' layers are multiples of 256; a serving frame's rows, and a
    # program's own layers, are any size
    if rng.random() < 0.5:
        m, n, k = (_log_int(rng, 256, 4096, 256) for _ in range(3))
    else:
        m, n, k = (_log_int(rng, 128, 3000) for _ in range(3))
        k = {"f32": k, "bf16": k // 32 * 32, "fp8": k // 16 * 16}[dtype]
    soft = dtype != "fp8" and rng.random() < 0.4
    return {"kind": kind, "dtype": dtype, "m": m, "n": n, "k": k, "softmax": soft,
            "rowsum": dtype != "fp8" and rng.random() < 0.3}


# ---------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(g, *shape, lo=-1.0, hi=1.0):
    return torch.rand(*shape, generator=g, device=DEV) * (hi - lo) + lo


def _e4m3(g, *shape):
    """Finite FP8 E4M3 codes: random sign and mantissa, exponent field 4..9."""
    sign = torch.randint(0, 2, shape, generator=g, device=DEV, dtype=torch.uint8) << 7
    expo = torch.randint(4, 10, shape, generator=g, device=DEV, dtype=torch.uint8) << 3
    return sign | expo | torch.randint(0, 8, shape, generator=g, device=DEV, dtype=torch.uint8)


def _dense_inputs(case, seed):
    """A [M, K]; B as the type's layout has it ([K, N] FP32, else [N, K]); bias [N]."""
    g = _generator(seed)
    m, n, k = case["m"], case["n"], case["k"]
    if case["dtype"] == "f32":
        return _uniform(g, m, k), _uniform(g, k, n), _uniform(g, n)
    if case["dtype"] == "bf16":
        return (_uniform(g, m, k).bfloat16(), _uniform(g, n, k).bfloat16(), _uniform(g, n))
    return _e4m3(g, m, k), _e4m3(g, n, k), None


def _conv_inputs(case, seed):
    """X and W (FP32: [C, H, W] and [C, C, 3, 3]; BF16: [H, W, C] and
    [C, 3, 3, C]) and a bias per channel."""
    g = _generator(seed)
    c, h, w = case["c"], case["h"], case["w"]
    if case["dtype"] == "f32":
        return _uniform(g, c, h, w), _uniform(g, c, c, 3, 3), _uniform(g, c)
    return (_uniform(g, h, w, c).bfloat16(), _uniform(g, c, 3, 3, c).bfloat16(), _uniform(g, c))


def _cloud(case, seed):
    g = _generator(seed)
    n = case["points"]
    pts = torch.empty(n, 4, device=DEV)
    pts[:, :3] = torch.randn(n, 3, generator=g, device=DEV) * 20.0
    pts[:, 3] = torch.rand(n, generator=g, device=DEV)
    return pts


def _frame_inputs(case, seed):
    g = _generator(seed)
    d, c, s = case["dim"], case["ch"], case["img"]
    return [(_uniform(g, d, d), _uniform(g, d, d), _uniform(g, d), _uniform(g, c, s, s),
             _uniform(g, c, c, 3, 3)) for _ in range(case["tasks"])]


# ---------------------------------------------------------------- states
class _Layer:
    """Descriptors marshalled once, and the tensors they point to."""

    def __init__(self):
        self.calls = []
        self.keep = []

    def add(self, op, shape, ins, outs, fparam=()):
        tensors = list(ins) + list(outs)
        n_in = len(ins)
        desc = {"op": op, "shape": shape, "in": tuple(range(n_in)),
                "out": tuple(range(n_in, len(tensors))), "fparam": fparam}
        self.calls.append((capi.kernel_struct(desc),
                           capi.pointer_array([t.data_ptr() for t in tensors]), len(tensors)))
        self.keep.append(tensors)

    def launch(self):
        launch = capi.lib().ug_kernel_launch
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        for ks, ptrs, n in self.calls:
            status = launch(ctypes.byref(ks), ptrs, n, stream)
            if status != capi.OK:
                raise capi.UgError(status, "ug_kernel_launch")


def _prepare_dense(case, seed):
    a, b, bias = _dense_inputs(case, seed)
    m, n, k = case["m"], case["n"], case["k"]
    layer = _Layer()
    c = torch.empty(m, n, device=DEV)
    outs = [c]
    layer.add({"f32": "gemm", "bf16": "gemm_bf16", "fp8": "gemm_fp8"}[case["dtype"]], (m, n, k),
              [a, b], [c])
    if bias is not None:
        layer.add("bias_relu", (m, n, 0), [c, bias], [c])
    if case["softmax"]:
        outs.append(torch.empty(m, n, device=DEV))
        layer.add("softmax", (m, n), [c], [outs[-1]])
    if case["rowsum"]:
        outs.append(torch.empty(m, device=DEV))
        layer.add("rowsum", (m, n), [c], [outs[-1]])
    return layer, outs


def _prepare_conv(case, seed):
    x, wt, bias = _conv_inputs(case, seed)
    c, h, w = case["c"], case["h"], case["w"]
    layer = _Layer()
    y = torch.empty(c, h, w, device=DEV)
    outs = [y]
    layer.add("conv3x3" if case["dtype"] == "f32" else "conv3x3_bf16", (1, c, h, w), [x, wt], [y])
    layer.add("bias_relu", (c, h * w, 1), [y, bias], [y])
    if case["rowsum"]:
        outs.append(torch.empty(c, device=DEV))
        layer.add("rowsum", (c, h * w), [y], [outs[-1]])
    return layer, outs


def _prepare_voxel(case, seed):
    pts = _cloud(case, seed)
    n, cells = case["points"], GRID[0] * GRID[1]
    layer = _Layer()
    outs = [torch.empty(n, dtype=torch.int32, device=DEV),
            torch.empty(cells, dtype=torch.int32, device=DEV), torch.empty(cells, device=DEV),
            torch.empty(cells, dtype=torch.int32, device=DEV)]
    layer.add("voxel", (n, *GRID), [pts], outs, GRID_PARAM)
    return layer, outs


class _Frame:
    """A started gate with one chain, and the buffers of its frames."""

    def __init__(self, case, seed):
        d, c, s = case["dim"], case["ch"], case["img"]
        slots, tasks = [], []
        self.outs = []
        for a, b, bias, x, wt in _frame_inputs(case, seed):
            o = len(slots)
            outs = [torch.empty(d, d, device=DEV), torch.empty(c, s, s, device=DEV),
                    torch.empty(c * s, device=DEV)]
            slots += [a, b, bias, x, wt] + outs
            self.outs += outs
            tasks.append({"cpu_ns": 0, "kernels": [
                {"op": "gemm", "shape": (d, d, d), "in": (o, o + 1), "out": (o + 5,)},
                {"op": "bias_relu", "shape": (d, d, 0), "in": (o + 5, o + 2), "out": (o + 5,)},
                {"op": "conv3x3", "shape": (1, c, s, s), "in": (o + 3, o + 4), "out": (o + 6,)},
                {"op": "rowsum", "shape": (c * s, s), "in": (o + 6,), "out": (o + 7,)}]})
        self.slots = slots
        self.ptrs = [t.data_ptr() for t in slots]
        torch.cuda.synchronize()
        self.gate = capi.Gate(policy="urgency", own_streams=1)
        self.chain = self.gate.register_chain(100_000_000, 100_000_000, tasks, len(slots))
        self.gate.profile(self.chain, self.ptrs, warmup=1, reps=3)
        self.gate.start()

    def run(self):
        # a frame's buffers are in place when it is submitted: the gate's
        # streams are not ordered after the program's
        torch.cuda.current_stream().synchronize()
        if self.gate.submit(self.chain, -1, self.ptrs) is None:
            raise RuntimeError("submission queue full")
        self.gate.drain(20.0)
        self.gate.poll(16)
        return self.outs

    def __del__(self):
        # the gate ends before the buffers its frames used are given back
        if hasattr(self, "gate"):
            self.gate.close()


def prepare(case, seed):
    if case["kind"] == "frame":
        return _Frame(case, seed)
    return {"dense": _prepare_dense, "conv": _prepare_conv,
            "voxel": _prepare_voxel}[case["kind"]](case, seed)


def run(state):
    if isinstance(state, _Frame):
        return state.run()
    layer, outs = state
    layer.launch()
    return outs


# ---------------------------------------------------------------- work
def _conv_work(c, h, w, in_bytes):
    return (in_bytes * (c * h * w + 9 * c * c) + 4 * c * h * w, 18 * c * c * h * w)


def work(case):
    if case["kind"] == "frame":
        d, c, s, t = case["dim"], case["ch"], case["img"], case["tasks"]
        conv_bytes, conv_flops = _conv_work(c, s, s, 4)
        return {"bytes": t * (4 * (3 * d * d + d) + conv_bytes + 4 * c * s),
                "flops": t * (2 * d ** 3 + 2 * d * d + conv_flops + c * s * s)}
    if case["kind"] == "voxel":
        # 16 bytes a point in, its cell out, three words a cell out
        return {"bytes": 20 * case["points"] + 12 * GRID[0] * GRID[1],
                "flops": 4 * case["points"]}
    if case["kind"] == "conv":
        c, h, w = case["c"], case["h"], case["w"]
        nbytes, flops = _conv_work(c, h, w, 4 if case["dtype"] == "f32" else 2)
        flops += (3 if case["rowsum"] else 2) * c * h * w
        return {"bytes": nbytes + 4 * c + (4 * c if case["rowsum"] else 0), "flops": flops}
    m, n, k = case["m"], case["n"], case["k"]
    size = {"f32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
    nbytes, flops = size * (m * k + k * n) + 4 * m * n, 2 * m * n * k
    if case["dtype"] != "fp8":
        nbytes, flops = nbytes + 4 * n, flops + 2 * m * n
    if case["softmax"]:
        nbytes, flops = nbytes + 4 * m * n, flops + 5 * m * n
    if case["rowsum"]:
        nbytes, flops = nbytes + 4 * m, flops + m * n
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- 64 bits
def _conv64(x, w):
    """3x3 cross-correlation with zero padding of x [C, H, W] with w
    [O, C, 3, 3] in float64: nine products of channel matrices."""
    c, h, wd = x.shape
    xp = F.pad(x.double(), (1, 1, 1, 1))
    y = torch.zeros(w.shape[0], h * wd, dtype=torch.float64, device=x.device)
    for dy in range(3):
        for dx in range(3):
            y += w[:, :, dy, dx].double() @ xp[:, dy:dy + h, dx:dx + wd].reshape(c, h * wd)
    return y.reshape(w.shape[0], h, wd)


def _voxel64(pts):
    n, cells = pts.shape[0], GRID[0] * GRID[1]
    # a point's cell is defined by two single-precision operations a side
    fx = (pts[:, 0] - GRID_PARAM[0]) * GRID_PARAM[2]
    fy = (pts[:, 1] - GRID_PARAM[1]) * GRID_PARAM[2]
    inside = (fx >= 0) & (fx < GRID[0]) & (fy >= 0) & (fy < GRID[1])
    cell = torch.where(inside, fy.floor().long() * GRID[0] + fx.floor().long(), -1)
    idx = inside.nonzero().flatten()
    hit = cell[idx]
    count = torch.bincount(hit, minlength=cells)
    zmax = torch.full((cells,), float("-inf"), dtype=torch.float64, device=pts.device)
    zmax.scatter_reduce_(0, hit, pts[idx, 2].double(), "amax")
    first = torch.full((cells,), n, device=pts.device)
    first.scatter_reduce_(0, hit, idx, "amin")
    first[count == 0] = -1
    return [cell.int(), count.int(), zmax, first.int()]


def exact(case, seed):
    if case["kind"] == "voxel":
        return _voxel64(_cloud(case, seed))
    if case["kind"] == "frame":
        outs = []
        for a, b, bias, x, wt in _frame_inputs(case, seed):
            z = _conv64(x, wt)
            outs += [torch.relu(a.double() @ b.double() + bias.double()), z,
                     z.reshape(-1, case["img"]).sum(1)]
        return outs
    if case["kind"] == "conv":
        x, wt, bias = _conv_inputs(case, seed)
        if case["dtype"] == "bf16":
            x, wt = x.permute(2, 0, 1), wt.permute(0, 3, 1, 2)
        y = torch.relu(_conv64(x, wt) + bias.double()[:, None, None])
        return [y] + ([y.flatten(1).sum(1)] if case["rowsum"] else [])
    a, b, bias = _dense_inputs(case, seed)
    if case["dtype"] == "fp8":
        a, b = a.view(torch.float8_e4m3fn), b.view(torch.float8_e4m3fn)
    b = b.double() if case["dtype"] == "f32" else b.double().t()
    y = a.double() @ b
    if bias is not None:
        y = torch.relu(y + bias.double())
    outs = [y]
    if case["softmax"]:
        outs.append(torch.softmax(y, 1))
    if case["rowsum"]:
        outs.append(y.sum(1))
    return outs
