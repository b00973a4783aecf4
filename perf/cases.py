"""The work that users of this library have it do, as cases that can be timed and compared.

Every case is one pass through the C ABI as an application makes it: the cell lists of the current positions, then the
forward pass (a property prediction), the forward and backward passes (a force evaluation, or a training step with the
gradients of all weights), or a stand-alone tensor product.  Sizes, model shapes and position statistics are those of
workloads.py and of the benchmark; positions, features and weights are drawn on the GPU from the seed alone.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what an application holds before the call: inputs, weights, context, workspaces
  run(state)           one pass, its outputs in full
  work(case)           bytes and operations that the pass cannot do without
  tolerance(case)      how far another correct implementation of the same precision may be off
"""
import math
import random
import weakref

import numpy as np
import torch

from paper_2601_16622_amd import binding as B
from paper_2601_16622_amd import workloads as W

DENSITY = 0.1      # atoms per cubic Angstrom
MIN_SEP = 0.9      # Angstrom
FCC_A = 3.8        # lattice constant of the FCC recipe
MODELS = {         # model shapes: L_max, channels, heads, filter degree, cutoff, feature type
    "tiny": dict(L=1, C=16, H=2, lf=1, cutoff=5.0, dtype="f32"),
    "small": dict(L=2, C=128, H=8, lf=1, cutoff=5.0, dtype="f32"),
    "base": dict(L=4, C=128, H=8, lf=1, cutoff=6.0, dtype="bf16"),
    "wide": dict(L=4, C=256, H=16, lf=1, cutoff=6.0, dtype="bf16"),
    "narrow": dict(L=3, C=64, H=4, lf=1, cutoff=6.0, dtype="bf16"),
}
N_RBF = 8


def listed():
    return [
        # one small system in single precision, the smallest call: bound by launches
        dict(name="tiny_forward", kind="forward", model="tiny", system="box", systems=1, lo=64, hi=64),
        # a batch of small organic molecules in single precision: inference ...
        dict(name="small_forward", kind="forward", model="small", system="molecules", systems=64, lo=10, hi=60),
        # ... and a training step, every gradient asked for
        dict(name="small_train", kind="train", model="small", system="molecules", systems=64, lo=10, hi=60),
        # a batch of larger molecules: inference and a training step
        dict(name="large_forward", kind="forward", model="base", system="box", systems=16, lo=150, hi=350),
        dict(name="large_train", kind="train", model="base", system="box", systems=16, lo=150, hi=350),
        # the scaling point, one open box of 10 000 atoms: the benchmark's step
        dict(name="box10k_forward", kind="forward", model="base", system="box", systems=1, lo=10000, hi=10000),
        # molecular dynamics of a bulk cell: energies and forces under periodic boundaries, new cell lists every step
        dict(name="bulk10k_force", kind="force", model="base", system="bulk", systems=1, lo=9973, hi=9973),
        # the largest system of the scaling runs
        dict(name="box100k_forward", kind="forward", model="base", system="box", systems=1, lo=100000, hi=100000),
        # the lattice recipe of the inference-scaling experiment with the model table's cap of 32 neighbours
        dict(name="fcc50k_capped", kind="capped", model="base", system="fcc", systems=1, lo=50000, hi=50000),
        # the channel count of the model table, forces for a batch of larger molecules
        dict(name="wide_force", kind="force", model="wide", system="box", systems=16, lo=150, hi=350),
        # the scoring form of the model table (non-linear pair feature) on the same kind of batch
        dict(name="large_nonlinear", kind="nonlinear", model="base", system="box", systems=16, lo=150, hi=350),
        # the stand-alone product (128x0e+128x1e+128x2e) x 1x2e of the tensor-product timing table, its largest size
        dict(name="product32k", kind="product", model="product", system="pairs", systems=1, lo=32000, hi=32000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "force", "force", "train", "capped", "nonlinear", "product"])
    if kind == "product":
        return dict(kind=kind, model="product", system="pairs", systems=1, lo=(n := _log_int(rng, 1000, 32000)), hi=n)
    if kind == "forward" and rng.random() < 0.15:
        return dict(kind=kind, model="tiny", system="box", systems=1, lo=(n := _log_int(rng, 64, 2000)), hi=n)
    if kind in ("forward", "train") and rng.random() < 0.35:
        lo = rng.randint(5, 30)
        return dict(kind=kind, model="small", system="molecules", systems=_log_int(rng, 8, 64), lo=lo, hi=lo + rng.randint(0, 30))
    model = rng.choice(["base", "base", "base", "wide", "narrow"])
    if kind in ("capped", "nonlinear"):
        model = rng.choice(["base", "base", "narrow"])
    most = {"forward": 100000, "capped": 50000, "force": 10000, "train": 6000, "nonlinear": 4000}[kind]
    if model == "wide":
        most = min(most, 20000 if kind == "forward" else 4000)
    system = rng.choice(["batch", "box", "bulk"] if kind in ("force", "nonlinear", "train") else ["batch", "box", "bulk", "fcc"])
    if system == "batch":
        lo = rng.randint(100, 300)
        hi = lo + rng.randint(0, 200)
        return dict(kind=kind, model=model, system="box", systems=max(1, min(_log_int(rng, 2, 32), 2 * most // (lo + hi))), lo=lo, hi=hi)
    n = _log_int(rng, 900, most)
    return dict(kind=kind, model=model, system=system, systems=1, lo=n, hi=n)


def _sizes(case):
    """Atoms of every system of the case: a fact of the case, the same for every seed."""
    r = random.Random(case["systems"] * 1000003 + case["lo"] * 1009 + case["hi"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["systems"])]


def _separated(gen, n, lens, periodic):
    """n points uniform in a box, none closer than MIN_SEP to another (hard-core thinning of a denser throw: a point
    stays if no earlier point is within reach), all on the GPU.  lens: edges of the box."""
    dev = gen.device
    L = torch.tensor(lens, dtype=torch.float64, device=dev)
    raw = int(1.28 * n + 8 * math.sqrt(n) + 16)
    p = torch.rand((raw, 3), dtype=torch.float64, device=dev, generator=gen) * L
    dims = [max(1, int(x / 2.5)) for x in lens]
    D = torch.tensor(dims, device=dev)
    c = torch.minimum((p / L * D).long(), D - 1)
    cell = (c[:, 2] * dims[1] + c[:, 1]) * dims[0] + c[:, 0]
    order = torch.argsort(cell, stable=True)
    counts = torch.bincount(cell, minlength=dims[0] * dims[1] * dims[2])
    depth = int(counts.max())
    rank = torch.empty_like(order)
    rank[order] = torch.arange(raw, device=dev) - (torch.cumsum(counts, 0) - counts)[cell[order]]
    table = torch.full((counts.numel(), depth), -1, dtype=torch.long, device=dev)
    table[cell, rank] = torch.arange(raw, device=dev)
    keep = torch.ones(raw, dtype=torch.bool, device=dev)
    me = torch.arange(raw, device=dev)[:, None]
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dz in (-1, 0, 1):
                o = c + torch.tensor([dx, dy, dz], device=dev)
                inside = torch.ones(raw, dtype=torch.bool, device=dev) if periodic else ((o >= 0) & (o < D)).all(1)
                o = torch.remainder(o, D)
                other = table[(o[:, 2] * dims[1] + o[:, 1]) * dims[0] + o[:, 0]]
                d = p[:, None] - p[other.clamp(min=0)]
                if periodic:
                    d = d - L * torch.round(d / L)
                near = ((d * d).sum(-1) < MIN_SEP ** 2) & (other >= 0) & (other < me) & inside[:, None]
                keep &= ~near.any(1)
    kept = p[keep][:n]
    assert kept.shape[0] == n
    return kept


def _bulk_lens(n, cutoff):
    base = (n / DENSITY / (1.1 * 0.95)) ** (1.0 / 3.0)
    return [float(np.float32(max(x * base, 3.0 * cutoff * 1.001))) for x in (1.0, 1.1, 0.95)]


def _positions(case, cutoff, gen, seed):
    """(positions float32 [N][3] on the GPU, host box lengths [S][3] or None)"""
    sizes, dev = _sizes(case), gen.device
    if case["system"] == "molecules":
        rng = np.random.default_rng(seed)
        mols = [W.bonded_cluster(rng, s) + rng.uniform(-20, 20, size=3).astype(np.float32) for s in sizes]
        return torch.from_numpy(np.concatenate(mols).astype(np.float32)).to(dev), None
    if case["system"] == "fcc":
        n = sizes[0]
        nc = 1
        while 4 * nc ** 3 < n:
            nc += 1
        g = torch.arange(nc, dtype=torch.float64, device=dev)
        cell = torch.stack(torch.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 1, 3)
        basis = torch.tensor([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]], dtype=torch.float64, device=dev)
        sites = ((cell + basis) * FCC_A).reshape(-1, 3)
        keep = torch.randperm(sites.shape[0], device=dev, generator=gen)[:n].sort().values
        return sites[keep].float(), None
    if case["system"] == "bulk":
        lens = _bulk_lens(sizes[0], cutoff)
        p = _separated(gen, sizes[0], lens, True)
        # a tenth of the atoms displaced by whole box lengths, as coordinates of a running simulation are
        hop = torch.randint(-2, 3, p.shape, device=dev, generator=gen) * torch.tensor(lens, dtype=torch.float64, device=dev)
        moved = torch.rand((p.shape[0], 1), device=dev, generator=gen) < 0.1
        return (p + torch.where(moved, hop, torch.zeros_like(hop))).float(), np.asarray([lens], dtype=np.float32)
    # one system to a box; the first "tiny" system is denser, as the Tiny configuration is
    parts = []
    for n in sizes:
        side = (n / (DENSITY if case["model"] != "tiny" else 0.125)) ** (1.0 / 3.0)
        origin = (torch.rand(3, dtype=torch.float64, device=dev, generator=gen) - 0.5) * 60.0
        parts.append(_separated(gen, n, [side] * 3, False) + origin)
    return torch.cat(parts).float(), None


class State:
    """What an application keeps between calls: the context, inputs, weights, workspaces and result buffers."""

    def __init__(self, case, ctx):
        self.kind, self.ctx, self.cells = case["kind"], ctx, []
        weakref.finalize(self, _release, ctx, self.cells)


def _release(ctx, cells):
    while cells:
        B.e2f_cells_destroy(cells.pop())
    B.e2f_destroy(ctx)


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, dtype=torch.float32, device=dev, generator=gen)

    if case["kind"] == "product":
        T = case["lo"]
        s = State(case, B.e2f_create(2, 128, 1, 1, 2, 1.0, "f32"))
        s.h, s.r = normal(T, 9, 128), normal(T, 3)
        s.w_path = torch.rand((3, 3), device=dev, generator=gen) + 0.5
        s.out = torch.empty_like(s.h)
        return s

    m = MODELS[case["model"]]
    L, C, H = m["L"], m["C"], m["H"]
    n = (L + 1) ** 2
    fdt = torch.bfloat16 if m["dtype"] == "bf16" else torch.float32
    s = State(case, B.e2f_create(L, C, H, N_RBF, m["lf"], m["cutoff"], m["dtype"]))
    s.pos, s.box = _positions(case, m["cutoff"], gen, seed)
    sizes = _sizes(case)
    N, S = sum(sizes), len(sizes)
    s.seg = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int32, device=dev)
    h = normal(N, n, C)
    if case["model"] != "tiny":   # degree 0 holds the embedding of the atom's element
        el = torch.multinomial(torch.tensor(W.ELEMENT_PROBS, device=dev), N, replacement=True, generator=gen)
        h[:, 0] = normal(len(W.ELEMENT_PROBS), C)[el]
    s.h = h.to(fdt)
    lim = math.sqrt(6.0 / (2 * C))
    s.weights = {k: ((torch.rand((L + 1, C, C), device=dev, generator=gen) * 2 - 1) * lim).to(fdt)
                 for k in ("WQ1", "WQ2", "WK1", "WK2", "WV")}
    s.weights["Wb"] = normal(H, N_RBF) / math.sqrt(N_RBF)
    s.weights["w_path"] = torch.rand((L + 1, L + 1), device=dev, generator=gen) + 0.5
    s.out = torch.empty((N, n, C), dtype=torch.float32, device=dev)
    need = {"forward": B.e2f_attn_workspace_bytes, "capped": B.e2f_attn_capped_workspace_bytes,
            "nonlinear": B.e2f_attn_nonlinear_workspace_bytes, "force": B.e2f_attn_backward_workspace_bytes,
            "train": B.e2f_attn_backward_weights_workspace_bytes}[case["kind"]](s.ctx, N)
    s.ws = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
    s.cells_ws = torch.empty(B.e2f_cells_workspace_bytes(s.ctx, N, S), dtype=torch.uint8, device=dev)
    if case["kind"] in ("force", "train"):
        s.grad_out = normal(N, n, C)
        s.grads = [torch.empty(shape, dtype=torch.float32, device=dev)
                   for shape in ((N, 3), (N, L + 1, C), (N, L + 1, C), (N, n, C), (N, n, C))]
        s.wgrads = [None] * 3
        if case["kind"] == "train":
            s.wgrads = [torch.empty(shape, dtype=torch.float32, device=dev)
                        for shape in ((H, N_RBF), (L + 1, L + 1), (5, L + 1, C, C))]
    return s


def run(s):
    if s.kind == "product":
        B.e2f_eaas_tensor_product(s.ctx, s.h, s.r, s.w_path, s.out)
        return s.out
    while s.cells:   # the lists of the last step's positions
        B.e2f_cells_destroy(s.cells.pop())
    if s.box is not None:
        s.cells.append(B.e2f_build_cells_periodic(s.ctx, s.pos, s.seg, s.box, s.cells_ws))
    else:
        s.cells.append(B.e2f_build_cells(s.ctx, s.pos, s.seg, s.cells_ws))
    args = (s.ctx, s.cells[0], s.pos, s.h, s.seg, s.weights)
    if s.kind == "capped":
        B.e2f_attn_forward_capped(*args, 32, s.out, s.ws)
    elif s.kind == "nonlinear":
        B.e2f_attn_forward_nonlinear(*args, s.out, s.ws)
    else:
        B.e2f_attn_forward(*args, s.out, s.ws)
    if s.kind not in ("force", "train"):
        return s.out
    B.e2f_attn_backward_after_forward(*args, s.out, s.grad_out, *s.grads, s.ws, *s.wgrads)
    return [s.out] + s.grads + [g for g in s.wgrads if g is not None]


def _pairs(case, cutoff):
    """Expected number of directed pairs inside the cutoff."""
    total = 0.0
    for n in _sizes(case):
        if case["system"] == "molecules":   # bonded clusters of up to 60 atoms: counted on samples
            total += 0.85 * n * (n - 1)
        elif case["system"] == "fcc":       # 54 sites in reach, thinned to the occupied share, fewer at the surface
            nc = 1
            while 4 * nc ** 3 < n:
                nc += 1
            total += n * 54.0 * n / (4 * nc ** 3) * max(0.0, 1.0 - 9.0 * cutoff / (8.0 * nc * FCC_A))
        else:
            rho = DENSITY if case["model"] != "tiny" else 0.125
            full = 4.0 / 3.0 * math.pi * (cutoff ** 3 - MIN_SEP ** 3)
            if case["system"] == "bulk":
                lens = _bulk_lens(n, cutoff)
                total += n * n / (lens[0] * lens[1] * lens[2]) * full
                continue
            a = (n / rho) ** (1.0 / 3.0)    # integral of the box's self-overlap over the ball
            r = cutoff
            total += n * rho * max(0.2 * full, full - 3 * math.pi * r ** 4 / (2 * a) + 3 * 8 * r ** 5 / (15 * a * a) - r ** 6 / (6 * a ** 3))
    return total


def work(case):
    """Each input read once, each output written once; products of the l-wise maps, the logits and the aggregation with
    the degree-1 filter taken through its linearity (three weighted sums of value rows per target)."""
    if case["kind"] == "product":
        T = case["lo"]
        # per product and channel: rotate in, re-index (19 entries at degrees 2 x 2), rotate back
        return {"bytes": T * (2.0 * 9 * 128 * 4 + 12), "flops": T * 128.0 * 2 * (35 + 19 + 35)}
    m = MODELS[case["model"]]
    n, C, L1 = (m["L"] + 1) ** 2, m["C"], m["L"] + 1
    N = float(sum(_sizes(case)))
    E = _pairs(case, m["cutoff"])
    esz = 2 if m["dtype"] == "bf16" else 4
    weights = 5.0 * L1 * C * C * esz
    rows = N * n * C
    bytes_ = N * 12 + rows * esz + weights + rows * 4
    flops = N * (10.0 * n * C * C + 4 * n * C) + E * (2.0 * L1 * C + 6 * n * C)
    if case["kind"] == "capped":
        flops = N * (10.0 * n * C * C + 4 * n * C) + min(E, 32.0 * N) * (2.0 * L1 * C + 6 * n * C)
    if case["kind"] == "nonlinear":
        flops += E * (4.0 * n * C + 8.0 * L1 * C)
    if case["kind"] in ("force", "train"):
        # out and its gradient read, the gradients of positions, q, k, v and h written; per pair the logits again, the
        # products for dq, dk and three each for the weights' gradient and for dv; per atom the transposed maps
        bytes_ += rows * 4 + N * 12 + 2 * N * L1 * C * 4 + 2 * rows * 4
        flops += E * (6.0 * L1 * C + 12 * n * C) + N * 10.0 * n * C * C
        if case["kind"] == "train":
            bytes_ += 5.0 * L1 * C * C * 4
            flops += N * 10.0 * n * C * C
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times the distance between this path and the operator in 64 bits, at the sizes that take it there
    in seconds: single precision 8e-7 (forward), 2e-6 (gradients), 1.4e-7 (product), largest element 2e-5 and 2e-6 of
    the rms; bf16 features 3e-3 (forward), 4.6e-3 (non-linear logit) and 8e-3 to 1.3e-2 (gradients of q, k, h and the
    weights, which are small differences of large terms), largest element 0.03, 0.13 and 0.29 of the rms."""
    if case["kind"] == "product":
        return {"rel": 1e-6, "max": 2e-5}
    if MODELS[case["model"]]["dtype"] == "f32":
        return {"rel": 8e-6, "max": 1e-4}
    if case["kind"] in ("force", "train"):
        return {"rel": 3e-2, "max": 0.9}
    if case["kind"] == "nonlinear":
        return {"rel": 1.8e-2, "max": 0.5}
    return {"rel": 1e-2, "max": 0.15}
