"""The work a user of this library has it do, as timed cases: whole merge schedules
(insertions, map composition, gather back to the grid), the same through the
allocating one-call API, insertions on ragged packed rows with a class token in the
gather, the windowed schedule, the nearest-neighbour query with its cosines, and the
padded layout around batched attention.

Inputs are drawn on the GPU from the seed alone, with the distributions of the
package's synthetic token grids: piecewise constant regions plus noise (optionally a
smooth gradient), or independent tokens some of whose images are exact 2x2
duplicates.
"""
import math

import torch

import paper_2604_05718_amd as mpm
from paper_2604_05718_amd import api

DEV = "cuda"
_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_BYTES = {"bf16": 2, "f32": 4}
SURVIVORS = 0.85  # share of an image's tokens left after an insertion on these inputs


def listed():
    return [
        # A first call on one 224x224 image (14x14 patches) at ViT-S width, through the
        # allocating API: nothing but latency and launches.
        dict(name="one_image_224", kind="chain", B=1, gh=14, gw=14, D=384, dtype="bf16", data="voronoi",
             regions=10, sigma=0.25, gradient=0.0, insertions=2, window=-1),
        # ViT-Ti/16 at 512x512, one float32 image, one insertion (interactive use).
        dict(name="vit_ti_512", kind="schedule", B=1, gh=32, gw=32, D=192, dtype="f32", data="voronoi",
             regions=12, sigma=0.3, gradient=0.0, insertions=1, window=-1),
        # ViT-S/16 at 512x512, a serving batch.
        dict(name="vit_s_512", kind="schedule", B=32, gh=32, gw=32, D=384, dtype="bf16", data="voronoi",
             regions=20, sigma=0.25, gradient=0.0, insertions=2, window=-1),
        # ViT-B/16 at 512x512, the headline workload of the benchmark.
        dict(name="vit_b_512", kind="schedule", B=64, gh=32, gw=32, D=768, dtype="bf16", data="voronoi",
             regions=30, sigma=0.2, gradient=0.05, insertions=2, window=-1),
        # ViT-L/16 at 1024x1024: the largest, 4096 tokens an image.
        dict(name="vit_l_1024", kind="schedule", B=16, gh=64, gw=64, D=1024, dtype="bf16", data="voronoi",
             regions=60, sigma=0.2, gradient=0.0, insertions=2, window=-1),
        # 768x768 low-affinity tokens, every tenth image with exactly duplicated patches.
        dict(name="stress_768", kind="schedule", B=32, gh=48, gw=48, D=768, dtype="bf16", data="iid_dup",
             regions=0, sigma=0.0, gradient=0.0, insertions=2, window=-1),
        # ViT-B/16 at 480x480 (900 tokens, no multiple of a tile), through the allocating API.
        dict(name="vit_b_480", kind="chain", B=32, gh=30, gw=30, D=768, dtype="bf16", data="voronoi",
             regions=30, sigma=0.2, gradient=0.05, insertions=2, window=-1),
        # The float32 batch of the paper's speed tables (ViT-Ti/16 at 512x512, B=32).
        dict(name="vit_ti_512_b32", kind="schedule", B=32, gh=32, gw=32, D=192, dtype="f32", data="voronoi",
             regions=12, sigma=0.3, gradient=0.0, insertions=2, window=-1),
        # The locality constraint on the benchmark's grid.
        dict(name="vit_b_512_window3", kind="schedule", B=64, gh=32, gw=32, D=768, dtype="bf16", data="voronoi",
             regions=30, sigma=0.2, gradient=0.05, insertions=2, window=3),
        # Ragged packed images of a width that is no whole number of cache lines, one class
        # token in front of the rebuilt grid.
        dict(name="packed_d200", kind="packed", B=24, gh=30, gw=33, D=200, dtype="bf16", data="voronoi",
             regions=20, sigma=0.25, gradient=0.0, E=1),
        # Nearest neighbours and their cosines (affinity statistics), no merge.
        dict(name="neighbours_s_512", kind="argmax", B=16, gh=32, gw=32, D=384, dtype="bf16", data="voronoi",
             regions=20, sigma=0.25, gradient=0.0),
        # The packed queries, keys and values of a ViT-B block padded for batched attention,
        # and its output back to packed rows.
        dict(name="pad_qkv_b_512", kind="pad", B=64, gh=32, gw=32, D=768, dtype="bf16"),
    ]


def _largest():
    return next(c for c in listed() if c["name"] == "vit_l_1024")


def _cost(case):
    """A case's weight against the largest listed one's (float32 pairs cost eight times as much)."""
    w = work(case)
    return w["bytes"] / 3e12 + w["flops"] * (8 if case["dtype"] == "f32" else 1) / 6e14 + 2e-5


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["schedule", "schedule", "schedule", "chain", "chain", "packed", "argmax", "pad"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        gh = log_int(10, 64)
        gw = max(7, min(64, gh + rng.randint(-4, 4)))
        B = log_int(1, 64)
        # Widths of the ViT family, and any other whole number of 16-byte pieces.
        D = rng.choice([192, 384, 768, 1024]) if rng.random() < 0.6 else 8 * log_int(6, 128)
        case = dict(kind=kind, B=B, gh=gh, gw=gw, D=D, dtype=dtype)
        if kind != "pad":
            dup = rng.random() < 0.2 and gh % 2 == 0 and gw % 2 == 0
            case.update(data="iid_dup" if dup else "voronoi", regions=0 if dup else rng.randint(8, 60),
                        sigma=0.0 if dup else round(rng.uniform(0.15 if dtype == "bf16" else 0.25, 0.35), 3),
                        gradient=0.0 if dup else rng.choice([0.0, 0.0, 0.05]))
        if kind in ("schedule", "chain"):
            case.update(insertions=rng.choice([1, 2, 2, 2, 3]), window=rng.choice([-1, -1, -1, 2, 3, 5]))
        if kind == "packed":
            case.update(E=rng.choice([0, 1]))
        if _cost(case) <= _cost(_largest()):
            return case


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _tokens(case, g):
    """[B, N, D] tokens in the storage type."""
    B, gh, gw, D = case["B"], case["gh"], case["gw"], case["D"]
    N = gh * gw
    if case["data"] == "iid_dup":
        x = torch.randn((B, gh, gw, D), generator=g, device=DEV)
        if B > 5:
            d = x[5::10, ::2, ::2]
            x[5::10] = d.repeat_interleave(2, dim=1).repeat_interleave(2, dim=2)
        return x.view(B, N, D).to(_DT[case["dtype"]]).contiguous()
    R = case["regions"]
    sites = torch.rand((B, R, 2), generator=g, device=DEV) * torch.tensor([gh, gw], device=DEV, dtype=torch.float32)
    centroids = torch.randn((B, R, D), generator=g, device=DEV)
    cell = torch.arange(N, device=DEV)
    rows, cols = cell // gw, cell % gw
    at = torch.stack([rows + 0.5, cols + 0.5], dim=1)
    label = ((at[None, :, None, :] - sites[:, None, :, :]) ** 2).sum(-1).argmin(-1)  # [B, N]
    x = torch.randn((B, N, D), generator=g, device=DEV).mul_(case["sigma"])
    x += torch.gather(centroids, 1, label[:, :, None].expand(B, N, D))
    if case["gradient"]:
        d = torch.randn((B, 2, D), generator=g, device=DEV) * case["gradient"]
        x += rows[None, :, None] * d[:, :1] + cols[None, :, None] * d[:, 1:]
    return x.to(_DT[case["dtype"]]).contiguous()


def _counts(case, seed):
    """Ragged tokens per image, as merges leave them or crops of several sizes bring them:
    the same spread of lengths for every seed, dealt to the images in another order."""
    B, N = case["B"], case["gh"] * case["gw"]
    g = torch.Generator().manual_seed(int(seed) * 104729 + 7)
    lo, hi = (0.70, 0.90) if case["kind"] == "pad" else (0.35, 1.0)
    n = (torch.linspace(lo, hi, B) * N).long().clamp(1, N)
    return n[torch.randperm(B, generator=g)]


def prepare(case, seed):
    g = _generator(seed)
    kind, B, D, N = case["kind"], case["B"], case["D"], case["gh"] * case["gw"]
    state = {"case": case}
    if kind == "pad":
        n = _counts(case, seed)
        off = torch.zeros(B + 1, dtype=torch.int32)
        off[1:] = n.cumsum(0)
        R = int(off[-1])
        state.update(off=off.to(DEV), P=int(n.max()), R=R,
                     qkv=torch.randn((R, 3 * D), generator=g, device=DEV).to(_DT[case["dtype"]]),
                     o=torch.randn((B, int(n.max()), D), generator=g, device=DEV).to(_DT[case["dtype"]]))
        return state
    x = _tokens(case, g)
    if kind == "packed":
        n = _counts(case, seed)
        off = torch.zeros(B + 1, dtype=torch.int32)
        off[1:] = n.cumsum(0)
        keep = torch.arange(N)[None, :] < n[:, None]
        state.update(x=x[keep.to(DEV)].contiguous(), off=off.to(DEV), N=N, n=n,
                     spec=torch.randn((B, 1, D), generator=g, device=DEV).to(x.dtype) if case["E"] else None)
        return state
    state["x"] = x
    if kind == "schedule":
        local = dict(grid_w=case["gw"], window=case["window"]) if case["window"] >= 0 else {}
        state["plan"] = api.Schedule(B, N, D, x.dtype, insertions=case["insertions"], device=DEV, **local)
    return state


def run(state):
    """One pass. The rebuilt grid (what the decoder reads), the neighbours with their
    cosines, or the padded and the unpadded rows."""
    case = state["case"]
    kind = case["kind"]
    if kind == "schedule":
        return state["plan"].run(state["x"])
    if kind == "chain":
        local = dict(grid_w=case["gw"], window=case["window"]) if case["window"] >= 0 else {}
        return mpm.run_schedule(state["x"], insertions=case["insertions"], **local).out
    if kind == "packed":
        m = mpm.merge(state["x"], state["off"], N=state["N"])
        return mpm.unmerge(m.y, m.y_off, m.map, z_spec=state["spec"])
    if kind == "argmax":
        return mpm.argmax(state["x"], with_best=True)
    return api.pad(state["qkv"], state["off"], state["P"]), api.unpad(state["o"], state["off"], rows=state["R"])


def _window_pairs(gh, gw, w):
    """Unordered pairs of cells within w rows and columns of each other."""
    def ordered(n):
        return sum(min(n - 1, i + w) - max(0, i - w) + 1 for i in range(n))

    return (ordered(gh) * ordered(gw) - gh * gw) / 2


def work(case):
    """Tokens read once and the grid written once; two flops a channel for every pair of
    tokens (each pair once: the affinity is symmetric), later insertions on the tokens
    that typically survive."""
    B, D, N, s = case["B"], case["D"], case["gh"] * case["gw"], _BYTES[case["dtype"]]
    if case["kind"] == "pad":
        real = 0.80 * N
        return {"bytes": B * s * D * (real * 3 + 0.9 * N * 3 + real + real), "flops": 0.0}
    if case["kind"] == "packed":
        n = 0.675 * N
        return {"bytes": B * s * D * (n + N + 2 * case["E"]), "flops": B * 2.0 * D * n * n / 2}
    if case["kind"] == "argmax":
        return {"bytes": B * N * (s * D + 8), "flops": B * 2.0 * D * N * (N - 1) / 2}
    flops = 0.0
    for k in range(case["insertions"]):
        f = SURVIVORS ** k
        pairs = _window_pairs(case["gh"], case["gw"], case["window"]) * f if case["window"] >= 0 else (N * f) ** 2 / 2
        flops += B * 2.0 * D * pairs
    return {"bytes": 2.0 * B * N * D * s, "flops": flops}


def tolerance(case):
    """Copies are bit for bit. A merged row is the mean of two rows rounded once, so
    grids agree bit for bit but where two candidates' cosines differ by less than their
    float32 rounding: there another summation order picks the other token, which changes
    the few rows of the grid that the two pairs cover."""
    if case["kind"] == "pad":
        return "exact"
    if case["kind"] == "argmax":
        return {"rel": 2e-6, "max": 2e-5, "differ": 2e-3}
    return {"rel": 1e-2, "max": 0.99}


def _nearest(x64, pos, gw, window):
    """Nearest other row by cosine in float64, the lowest index among equal ones (cosines
    closer than 1e-12 count as equal), -1 where the window holds none; and the cosine."""
    n = x64.shape[0]
    u = x64 / x64.norm(dim=1, keepdim=True).clamp_min(1e-12)
    s = torch.mm(u, u.t())
    s.fill_diagonal_(-math.inf)
    if window >= 0:
        r, c = pos // gw, pos % gw
        out = ((r[:, None] - r[None, :]).abs() > window) | ((c[:, None] - c[None, :]).abs() > window)
        s.masked_fill_(out, -math.inf)
    best = s.max(dim=1).values
    at = torch.arange(n, device=x64.device)
    first = torch.where(s >= best[:, None] - 1e-12, at[None, :], n).amin(dim=1)
    return torch.where(torch.isfinite(best), first, -1), best


def _insert(x, pos, gw, window):
    """One insertion on [n, D] rows in the storage type: (merged rows, map, positions)."""
    n = x.shape[0]
    nb, _ = _nearest(x.double(), pos, gw, window)
    at = torch.arange(n, device=x.device)
    mutual = (nb >= 0) & (nb[nb.clamp_min(0)] == at)
    rep = ~mutual | (at < nb)
    ids = rep.long().cumsum(0) - 1
    a = at[rep]
    b = torch.where(mutual[rep], nb[rep], a)
    y = ((x[a].double() + x[b].double()) * 0.5).to(x.dtype)
    y[a == b] = x[a[a == b]]
    m = torch.where(rep, ids, ids[nb.clamp_min(0)])
    return y, m, pos[a]


def exact(case, seed):
    """float64 similarities; merged rows rounded once to the storage type, as they are stored."""
    state = prepare(case, seed)
    kind, B, N, D = case["kind"], case["B"], case["gh"] * case["gw"], case["D"]
    if kind == "pad":
        off, P = state["off"].tolist(), state["P"]
        padded = torch.zeros((B, P, 3 * D), dtype=torch.float64, device=DEV)
        rows = torch.zeros((state["R"], D), dtype=torch.float64, device=DEV)
        for b in range(B):
            n = off[b + 1] - off[b]
            padded[b, :n] = state["qkv"][off[b]:off[b + 1]].double()
            rows[off[b]:off[b + 1]] = state["o"][b, :n].double()
        return padded, rows
    if kind == "argmax":
        nb, best = zip(*(_nearest(state["x"][b].double(), None, 1, -1) for b in range(B)))
        return torch.stack(nb).int(), torch.stack(best)
    E = case.get("E", 0)
    out = torch.zeros((B, E + N, D), dtype=torch.float64, device=DEV)
    off = state["off"].tolist() if kind == "packed" else None
    for b in range(B):
        x = state["x"][off[b]:off[b + 1]] if off else state["x"][b]
        n = x.shape[0]
        pos = torch.arange(n, device=DEV)
        r = pos
        for _ in range(case.get("insertions", 1)):
            x, m, pos = _insert(x, pos, case["gw"], case.get("window", -1))
            r = m[r]
        if E:
            out[b, :E] = state["spec"][b].double()
        out[b, E:E + n] = x[r].double()
    return out
