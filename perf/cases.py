"""The calls a user of this package makes, as cases that can be timed and compared: `listed()` names twelve of them,
`draw()` gives more of the same ranges, `prepare()` makes what a program holds before the call and `run()` is one pass.

Four kinds of pass, each through the package's public entry points:
  encode   one batch through the encoding and its gradient back into the tables (HashGrid.encode_fwd, encode_bwd): what
           a program does around a network of its own
  train    one iteration of the whole model (HashGridModel.step): encoding, network, loss, both backward passes, Adam
  infer    the model's output at a batch of points (HashGridModel.infer)
  normals  the output's gradient with respect to the position (HashGridModel.input_gradient)

Points are spread as in the method's applications: "uniform" (pixels of an image drawn at random), "surface" (four in
five near a surface, the rest anywhere, as signed distances are trained), "rays" (256 samples along each ray, ray after
ray) and "raster" (the pixels of an image row by row, as it is drawn).
"""
import math

import torch

from paper_2201_05989_amd import HashGrid, HashGridModel

BELOW_ONE = 1.0 - 2.0 ** -24
SAMPLES_PER_RAY = 256
HIDDEN = 64
DTYPES = {"f16": torch.float16, "f32": torch.float32}


def encode(name, d, L, F, T, N_min, N_max, B, points, params="f16", io="f16", grad="f32", smooth=False, count=True, add=False):
    """count: the forward call also counts for the backward pass; add: the gradient grows by this batch's, else it is replaced."""
    return {"name": name, "kind": "encode", "d": d, "L": L, "F": F, "T": T, "N_min": N_min, "N_max": N_max, "B": B, "points": points,
            "params": params, "io": io, "grad": grad, "smooth": smooth, "count": count, "add": add}


def model(name, kind, d, L, F, T, N_min, N_max, B, points, n_out, loss="l2", smooth=False):
    return {"name": name, "kind": kind, "d": d, "L": L, "F": F, "T": T, "N_min": N_min, "N_max": N_max, "B": B, "points": points,
            "n_out": n_out, "loss": loss, "smooth": smooth}


def listed():
    return [
        # one ray's samples through a trained model: the smallest call, all latency
        model("infer_one_ray", "infer", 3, 16, 2, 1 << 19, 16, 2048, 256, "rays", 4),
        # the small reference configuration in single precision: a few launches on little data
        encode("encode_tiny2d", 2, 4, 2, 1 << 10, 4, 32, 4096, "uniform", "f32", "f32", add=True),
        # learning a small colour image
        model("train_image_small", "train", 2, 16, 2, 1 << 17, 16, 1024, 1 << 14, "uniform", 3),
        # a batch of a training loop that keeps half-precision gradients, eight features an entry, an odd number of points
        encode("encode_wide_half_grad", 3, 8, 8, 1 << 17, 16, 512, 30011, "surface", grad="f16"),
        # single-precision tables of a size that is no power of two
        encode("encode_single_any_size", 3, 16, 2, 1000003, 16, 2048, 100003, "uniform", "f32", "f32"),
        # normals of a signed distance function with the smoothstep variant, as a renderer asks for them
        model("normals_smoothstep", "normals", 3, 8, 4, 1 << 15, 4, 64, 76801, "surface", 1, smooth=True),
        # gigapixel image fitting: a large table in two dimensions
        encode("encode_image2d", 2, 16, 2, 1 << 22, 16, 32768, 1 << 18, "uniform"),
        # signed distance training at the paper's size: the benchmark's own step
        encode("encode_sdf3d", 3, 16, 2, 1 << 19, 16, 2048, 1 << 18, "surface", add=True),
        # the whole model on that batch
        model("train_sdf3d", "train", 3, 16, 2, 1 << 19, 16, 2048, 1 << 18, "surface", 1, "mape"),
        # drawing a learned image, 1920 x 1080 pixels row by row
        model("infer_frame", "infer", 2, 16, 2, 1 << 22, 16, 32768, 1920 * 1080, "raster", 3),
        # radiance-field training: 4096 rays of 256 samples in ray order
        model("train_nerf3d", "train", 3, 16, 2, 1 << 19, 16, 2048, 1 << 20, "rays", 4),
        # tables far larger than the caches
        encode("encode_large3d", 3, 16, 2, 1 << 24, 16, 1 << 19, 1 << 21, "uniform"),
    ]


def draw(rng):
    kind = rng.choice(("encode", "encode", "encode", "train", "train", "infer", "normals"))
    d = rng.choice((2, 3))
    L, F = rng.choice(((16, 2), (16, 2), (16, 2), (16, 1), (16, 4), (8, 4), (8, 8), (12, 2)))
    log2_T = rng.randint(14, 22)
    T = 1 << log2_T
    N_min = rng.choice((4, 16, 16))
    N_max = int(round(2.0 ** rng.uniform(6, 15 if d == 2 else 12)))
    # no more scalars than 2^20 points read on 16 levels of 8 corners and 2 features
    B = min(int(round(2.0 ** rng.uniform(8, 20))), (1 << 28) // (L * F << d))
    points = rng.choice(("uniform", "rays") if d == 2 else ("uniform", "surface", "rays"))
    smooth = rng.random() < 0.2
    if kind != "encode":
        n_out = 1 if kind == "normals" else rng.choice((1, 3, 4, 16))
        if kind == "infer" and d == 2:
            points = "raster"
        c = model("", kind, d, L, F, T, N_min, N_max, B, points, n_out, rng.choice(("l2", "mape")), smooth)
    else:
        if rng.random() < 0.2:
            T = rng.randint(T // 2 + 1, T - 1)  # any size: not a power of two
        params, io, grad = rng.choice((("f16", "f16", "f32"),) * 3 + (("f32", "f32", "f32"), ("f16", "f16", "f16")))
        c = encode("", d, L, F, T, N_min, N_max, B, points, params, io, grad, smooth, points != "rays", rng.random() < 0.3)
    del c["name"]
    return c


# ---- inputs ----

def unit_vectors(n, d, gen):
    v = torch.randn((n, d), device="cuda", generator=gen)
    return v / torch.linalg.norm(v, dim=1, keepdim=True)


def make_points(how, B, d, gen):
    if how == "uniform":
        x = torch.rand((B, d), device="cuda", generator=gen)
    elif how == "surface":
        near = 0.5 + 0.3 * unit_vectors(B * 4 // 5, d, gen)
        near += 0.01 * torch.randn(near.shape, device="cuda", generator=gen)
        x = torch.cat([near, torch.rand((B - near.shape[0], d), device="cuda", generator=gen)])
        x = x[torch.randperm(B, device="cuda", generator=gen)]
    elif how == "rays":
        n = -(-B // SAMPLES_PER_RAY)
        o = 0.5 + 1.5 * unit_vectors(n, d, gen)
        to = torch.rand((n, d), device="cuda", generator=gen) * 0.5 + 0.25 - o
        to /= torch.linalg.norm(to, dim=1, keepdim=True)
        a, b = (0.0 - o) / to, (1.0 - o) / to
        near, far = torch.minimum(a, b).amax(dim=1), torch.maximum(a, b).amin(dim=1)
        k = torch.arange(SAMPLES_PER_RAY, device="cuda") + torch.rand((n, SAMPLES_PER_RAY), device="cuda", generator=gen)
        t = near[:, None] + k / SAMPLES_PER_RAY * (far - near)[:, None]
        x = (o[:, None, :] + t[:, :, None] * to[:, None, :]).reshape(-1, d)[:B]
    else:  # raster: pixel centres of a 16 : 9 picture, the view moved a little from picture to picture
        width = max(1, math.ceil(math.sqrt(B * 16 / 9)))
        height = -(-B // width)
        i = torch.arange(B, device="cuda")
        x = torch.stack([(i % width + 0.5) / width, (i // width + 0.5) / height], dim=1)
        x = 0.05 + 0.9 * x + 0.05 * torch.rand((1, d), device="cuda", generator=gen)
    return x.float().clamp(0.0, BELOW_ONE).contiguous()


def targets(x, n_out):
    """What a model learns here: a distance-like field and some smooth channels."""
    r = torch.linalg.norm(x - 0.5, dim=1, keepdim=True) - 0.3
    k = torch.arange(n_out, device="cuda")
    return torch.cos(k * (3.0 + 20.0 * x.sum(dim=1, keepdim=True))).mul_(r).contiguous()


def make_grid(c):
    return HashGrid(c["d"], c["L"], c["F"], c["T"], c["N_min"], c["N_max"], c["params"], c["io"], int(c["smooth"]), c["grad"])


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = make_points(c["points"], c["B"], c["d"], gen)
    if c["kind"] == "encode":
        grid = make_grid(c)
        rows = (c["B"], c["L"] * c["F"])
        # features as they are after some training
        tables = torch.randn((grid.n_entries, c["F"]), device="cuda", generator=gen, dtype=DTYPES[c["params"]]).mul_(0.1)
        dy = torch.randn(rows, device="cuda", generator=gen, dtype=DTYPES[c["io"]]).mul_(0.1)
        y = torch.empty(rows, device="cuda", dtype=DTYPES[c["io"]])
        grad = torch.zeros((grid.n_entries, c["F"]), device="cuda", dtype=DTYPES[c["grad"]])
        return {"case": c, "grid": grid, "x": x, "tables": tables, "dy": dy, "y": y, "grad": grad}
    m = HashGridModel(c["d"], c["n_out"], L=c["L"], F=c["F"], T=c["T"], N_min=c["N_min"], N_max=c["N_max"], loss=c["loss"],
                      lr=1e-4 if c["loss"] == "mape" else 1e-2, seed=seed, interp=int(c["smooth"]))
    state = {"case": c, "model": m, "x": x}
    # features as they are after some training
    m.tables.copy_(torch.randn(m.tables.shape, device="cuda", generator=gen).mul_(0.1))
    m.tables_half.copy_(m.tables)
    if c["kind"] == "train":
        # in the middle of training: the optimiser's moments are not zero any more
        for _ in range(2):
            xp = make_points(c["points"], c["B"], c["d"], gen)
            m.step(xp, targets(xp, c["n_out"]))
        state["target"] = targets(x, c["n_out"])
    return state


# ---- one pass ----

def run(state):
    c = state["case"]
    if c["kind"] == "encode":
        y = state["grid"].encode_fwd(state["x"], state["tables"], state["y"], count_for_bwd=c["count"])
        grad = state["grid"].encode_bwd(state["x"], state["dy"], state["grad"], overwrite=not c["add"])
        return {"y": y, "grad": grad}
    m = state["model"]
    if c["kind"] == "train":
        m.step(state["x"], state["target"])
        return {"tables": m.tables, "tables_half": m.tables_half, "weights": m.weights, "weights_half": m.weights_half}
    if c["kind"] == "infer":
        return m.infer(state["x"])
    return m.input_gradient(state["x"])


# ---- what a pass cannot do without ----

def level_entries(c):
    """Entries of each level: (N + 1)^d vertices (one more a side with the smoothstep variant), T at the most."""
    L, lo, hi = c["L"], c["N_min"], c["N_max"]
    b = math.exp((math.log(hi) - math.log(lo)) / (L - 1)) if L > 1 else 1.0
    return [min(c["T"], (int(lo * b ** l + 1e-6) + (2 if c["smooth"] else 1)) ** c["d"]) for l in range(L)]


def work(case):
    c = case
    B, d, F, n_in = c["B"], c["d"], c["F"], c["L"] * c["F"]
    entries = level_entries(c)
    # entries that at least one of the batch's corners falls on, corners taken as evenly spread
    touched = sum(n * -math.expm1(-(B << d) / n) for n in entries) * F
    blend = 2.0 * B * n_in * (1 << d)  # one multiply-add for every feature of every corner
    if c["kind"] == "encode":
        s_io, s_par, s_grad = (2 if c[k] == "f16" else 4 for k in ("io", "params", "grad"))
        gradient = 2 * touched * s_grad if c["add"] else sum(entries) * F * s_grad
        return {"bytes": 4 * B * d + touched * s_par + 2 * B * n_in * s_io + gradient, "flops": 2 * blend}
    weights = HIDDEN * (n_in + HIDDEN + c["n_out"])
    net = 2.0 * B * weights
    if c["kind"] == "train":  # master copy and both moments read and written, the half-precision copy read and written
        return {"bytes": 4 * B * (d + c["n_out"]) + (touched + weights) * (24 + 4), "flops": 2 * blend + 3 * net}
    inputs = 4 * B * d + 2 * (touched + weights)
    if c["kind"] == "infer":
        return {"bytes": inputs + 4 * B * c["n_out"], "flops": blend + net}
    return {"bytes": inputs + 4 * B * d, "flops": (1 + d) * blend + 2 * net}


def tolerance(case):
    c = case
    if c["kind"] == "encode":
        if c["grad"] == "f16":  # sums of half-precision summands, each rounded on its way in where the sums are atomic
            return {"rel": 5e-3, "max": 0.2}
        if c["io"] == "f32":
            return {"rel": 1e-5, "max": 1e-4}
        # single-precision sums; y is rounded to half once, and sums that differ in their last bits round apart now and then
        return {"rel": 5e-5, "max": 2e-3}
    # half-precision activations, weights and hidden gradients (2^-11 each time they are stored); a hidden neuron whose
    # sum is next to zero passes a point's gradient in one implementation and stops it in another
    if c["kind"] == "infer":
        return {"rel": 1e-3, "max": 0.05}
    if c["kind"] == "normals":
        return {"rel": 2e-3, "max": 0.5}
    # an iteration moves features of size 0.1 by the learning rate; a scalar whose gradient nearly cancels may take
    # another step, since the optimiser divides by the gradient's own size, and a half-precision copy may round apart
    return {"rel": 1e-4, "max": 0.02} if c["loss"] == "mape" else {"rel": 1e-3, "max": 0.5}
