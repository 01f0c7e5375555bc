"""Performance cases of the per-ROI texture library: what its users have it do.

A case is one pass through a public call of ``paper_2603_12016_amd.nyx`` on
images that are already on the GPU.  ``listed`` names the cases, ``draw`` gives
more of the same ranges, ``prepare`` makes a case's inputs (and the plan and
the output table a program keeps between passes), ``run`` makes one pass,
``work`` counts the bytes and operations the pass cannot do without, and
``exact`` gives the same outputs in 64 bits from plain torch.

The images follow the recipes of the repository's benchmark workloads, made on
the GPU: smooth positive fields with counting noise for the intensities;
ellipses (ellipsoids in a volume) of random size for the labels, which touch
and clip each other as cells of a tissue do.

Fields of a case: ``call`` (plan: a replayed plan; oneshot: the whole path in
one call; noalloc: the same without device allocation; intensity and
neighbourhood: the other feature families; counts: ROI table, level image,
co-occurrence counts and the features from them), ``images`` of ``nz`` x ``ny``
x ``nx`` voxels, ``rois`` per image with sizes of law ``law`` (loguniform on
[lo, hi], lognormal of median lo and log-deviation hi, one: the image is one
ROI), ``giant`` (a further ROI over every free pixel of the upper 90 % of the
rows), ``bins`` grey levels, ``reach`` (offsets up to that distance: 4 per
distance in the plane, 13 in a volume), ``fp64`` output, ``symmetric``,
``merged`` (one matrix per ROI) and ``alpha`` (neighbourhood only).
"""
import math

import torch

from paper_2603_12016_amd import nyx

_BASE = {"call": "plan", "images": 1, "nz": 1, "ny": 512, "nx": 512, "rois": 100, "law": "lognormal", "lo": 800.0,
         "hi": 1.0, "giant": False, "bins": 64, "reach": 1, "fp64": False, "symmetric": True, "merged": False, "alpha": 0}


def _case(name, **kw):
    return dict(_BASE, name=name, **kw)


def listed():
    return [
        # The smallest pass: one 64 x 64 patch of noise as one ROI, few levels,
        # double precision; a patch-wise loop, where launches count.
        _case("patch_plan", ny=64, nx=64, rois=1, law="one", bins=8, fp64=True),
        # An interactive call on a field of view: no plan, no known ROI count.
        _case("view_oneshot", call="oneshot", ny=384, nx=517, rois=80),
        # A microscope image of about 2000 cells at 256 grey levels.
        _case("cells_plan", ny=2048, nx=2048, rois=2000, law="loguniform", lo=100.0, hi=5000.0, bins=256),
        # A plate of 64 images, about 150000 cells in one pass.
        _case("plate_plan", images=64, ny=2048, nx=2048, rois=2344),
        # A volume with about 500 organs-sized regions, 13 offsets.
        _case("volume_plan", nz=256, ny=512, nx=512, rois=500, law="loguniform", lo=1e3, hi=216e3),
        # A slide tile: one region over most of it next to 10000 tiny ones, 1024 levels.
        _case("tile_plan", ny=8192, nx=8192, rois=10000, law="loguniform", lo=30.0, hi=300.0, giant=True, bins=1024),
        # A tuning sweep's larger settings: 8 offsets at two distances, 128 levels, odd image sizes.
        _case("distances_plan", images=4, ny=1361, nx=1531, rois=1100, bins=128, reach=2),
        # Ordered (non-symmetric) matrices in double precision.
        _case("ordered_plan", images=4, ny=1024, nx=1024, rois=500, fp64=True, symmetric=False),
        # One merged matrix per region of a ragged volume, in one call.
        _case("merged_volume_oneshot", call="oneshot", nz=77, ny=203, nx=181, rois=60, law="loguniform", lo=500.0,
              hi=50e3, bins=32, merged=True),
        # First-order intensity features of every cell of 8 images.
        _case("intensity_batch", call="intensity", images=8, ny=2048, nx=2048, rois=2344),
        # Neighbourhood matrices of the regions of a volume.
        _case("neighbourhood_volume", call="neighbourhood", nz=128, ny=256, nx=256, rois=60, law="loguniform", lo=1e3,
              hi=216e3, bins=32),
        # The step-by-step calls: ROI table and levels, exported counts, features from the counts.
        _case("counts_export", call="counts", ny=1031, nx=1024, rois=500),
    ]


def _log(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def draw(rng):
    """A case of the same ranges: every call, in the plane and in volumes,
    sizes spread over their logarithm, odd ones among them."""
    call = rng.choice(["plan", "plan", "plan", "plan", "oneshot", "oneshot", "noalloc", "intensity", "neighbourhood", "counts"])
    volume = rng.random() < (0.15 if call == "counts" else 0.3)
    c = dict(_BASE, call=call)
    top = {"plan": 3e7, "oneshot": 1.6e7, "noalloc": 4e6, "intensity": 1.6e7, "neighbourhood": 8e6, "counts": 2e6}[call]
    if volume:
        vox = _log(rng, 3e4, top)
        nz = max(5, int(_log(rng, 0.1, 0.8) * vox ** (1 / 3)))
        nx = max(24, int((vox / nz) ** 0.5 * rng.uniform(0.7, 1.3)))
        c.update(images=1, nz=nz, ny=max(24, int(vox / nz / nx)), nx=nx, law="loguniform")
        small = min(nz * c["ny"] * nx / 8, _log(rng, 200, 2000))
        c.update(lo=small, hi=small * _log(rng, 3, 200))
        c["bins"] = rng.choice([16, 32, 50, 64])
    else:
        vox = _log(rng, 4e3, top)
        images = max(1, min(int(vox / 4096), int(_log(rng, 1, 24))))
        nx = max(48, int((vox / images) ** 0.5 * rng.uniform(0.7, 1.4)))
        c.update(images=images, ny=max(48, int(vox / images / nx)), nx=nx)
        if rng.random() < 0.5:
            c.update(law="loguniform", lo=_log(rng, 30, 200))
            c["hi"] = c["lo"] * _log(rng, 5, 60)
        else:
            c.update(lo=_log(rng, 200, 2000), hi=rng.uniform(0.4, 1.1))
        c["bins"] = rng.choice([8, 16, 32, 64, 64, 100, 128, 256])
        c["giant"] = call in ("plan", "oneshot") and rng.random() < 0.1
        c["reach"] = 2 if rng.random() < 0.15 else 1
    mean = (c["hi"] - c["lo"]) / math.log(c["hi"] / c["lo"]) if c["law"] == "loguniform" else c["lo"] * math.exp(c["hi"] ** 2 / 2)
    c["rois"] = max(1, int(rng.uniform(0.3, 0.8) * c["nz"] * c["ny"] * c["nx"] / mean))
    if c["bins"] >= 128:  # many levels: at most about 12000 regions
        c["rois"] = min(c["rois"], max(1, 12000 // c["images"]))
    c["fp64"] = rng.random() < 0.25
    if call in ("plan", "oneshot", "noalloc", "counts"):
        c["symmetric"] = rng.random() < 0.85 or c["bins"] > 128
        c["merged"] = call != "counts" and c["bins"] <= 64 and rng.random() < 0.15
    if call == "neighbourhood":
        c["alpha"] = rng.choice([0, 0, 0, 1])
    return c


# ------------------------------------------------------------------ inputs
def _field(g, dims, spacing):
    """Smooth random field: values on a coarse grid, interpolated."""
    shape = [max(2, int(n / spacing) + 2) for n in dims]
    v = torch.randn([1, 1] + shape, generator=g, device="cuda")
    kind = "bicubic" if len(dims) == 2 else "trilinear"
    return torch.nn.functional.interpolate(v, size=list(dims), mode=kind, align_corners=False)[0, 0]


def _intensity(case, g):
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    if case["law"] == "one":
        return torch.randint(0, 4096, (nz, ny, nx), generator=g, device="cuda").to(torch.int16)
    if nz > 1:
        f = 1000.0 + 250.0 * _field(g, (nz, ny, nx), 7.0) + 20.0 * torch.randn((nz, ny, nx), generator=g, device="cuda")
    else:
        f = _field(g, (ny, nx), 9.0).abs() * 350.0 + _field(g, (ny, nx), 31.0).square_() * 400.0 + 100.0
        f = f + f.clamp(min=1.0).sqrt() * torch.randn((ny, nx), generator=g, device="cuda")
        f = f.reshape(1, ny, nx)
    return f.round().clamp_(0, 32000).to(torch.int16)


def _sizes(case, n, g):
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    if case["law"] == "loguniform":
        return case["lo"] * (case["hi"] / case["lo"]) ** u
    s = case["lo"] * torch.exp(case["hi"] * torch.randn(n, generator=g, device="cuda", dtype=torch.float64))
    return s.clamp(20.0, 200000.0)


def _labels(case, g):
    """Ellipses or ellipsoids at random places; a pixel under several belongs
    to the one whose centre is nearest in units of its axes.  The first
    case["rois"] of them that keep a pixel are the image's regions."""
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    if case["law"] == "one":
        return torch.ones((nz, ny, nx), dtype=torch.int32, device="cuda")
    n = case["rois"] + case["rois"] // 5 + 8
    size = _sizes(case, n, g)
    ratio = 1.0 + torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (2.0 if nz == 1 else 1.0)
    place = torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float64)
    turn = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * math.pi
    if nz == 1:
        a = (size / math.pi * ratio).sqrt()
        b = a / ratio
        rz = torch.ones_like(a)
    else:
        a = (size * 0.75 / math.pi * ratio).pow(1 / 3)
        b = a / ratio.sqrt()
        rz = b
    co, si = turn.cos(), turn.sin()
    ex, ey = ((a * co) ** 2 + (b * si) ** 2).sqrt(), ((a * si) ** 2 + (b * co) ** 2).sqrt()
    ez = rz if nz > 1 else torch.zeros_like(a)
    dims = torch.tensor([nz, ny, nx], device="cuda", dtype=torch.float64)
    mid = place * (dims - 1)
    half = torch.stack([ez, ey, ex], 1)
    low = (mid - half).floor().clamp(min=0).long()
    high = torch.minimum((mid + half).ceil(), dims - 1).long()
    ext = high - low + 1
    count = ext.prod(1)
    best = torch.full((nz * ny * nx,), 2 ** 62, dtype=torch.int64, device="cuda")
    ends = count.cumsum(0)
    first = 0
    while first < n:  # boxes in groups of bounded size
        start = int(ends[first - 1]) if first else 0
        last = max(first + 1, int(torch.searchsorted(ends, start + (1 << 25), right=True)))
        k = torch.repeat_interleave(torch.arange(first, last, device="cuda"), count[first:last])
        o = torch.arange(k.numel(), device="cuda") - (ends[k] - count[k] - start)
        w, h = ext[k, 2], ext[k, 1]
        x, y, z = o % w + low[k, 2], o // w % h + low[k, 1], o // (w * h) + low[k, 0]
        dx, dy, dz = x - mid[k, 2], y - mid[k, 1], z - mid[k, 0]
        d = ((dx * co[k] + dy * si[k]) / a[k]) ** 2 + ((dy * co[k] - dx * si[k]) / b[k]) ** 2
        if nz > 1:
            d = d + (dz / rz[k]) ** 2
        keep = d <= 1.0
        key = ((d[keep] * (1 << 20)).long() << 32) | (k[keep] + 1)
        best.scatter_reduce_(0, ((z * ny + y) * nx + x)[keep], key, "amin")
        first = last
    lab = torch.where(best < 2 ** 62, best & 0xFFFFFFFF, torch.zeros_like(best))
    seen = torch.bincount(lab, minlength=n + 1) > 0
    seen[0] = False
    rank = seen.cumsum(0) * seen
    lab = torch.where(rank > case["rois"], torch.zeros_like(rank), rank)[lab]
    missing = case["rois"] - min(case["rois"], int(seen.sum()))
    if missing:  # (a very crowded image: the rest are single pixels)
        free = (lab == 0).nonzero()[:missing, 0]
        lab[free] = torch.arange(case["rois"] - missing + 1, case["rois"] - missing + 1 + free.numel(), device="cuda")
    lab = lab.to(torch.int32).reshape(nz, ny, nx)
    if case["giant"]:
        rows = lab[:, : int(0.9 * ny)]
        rows[rows == 0] = case["rois"] + 1
    return lab


def _images(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    out = []
    for _ in range(case["images"]):
        im, lab = _intensity(case, g), _labels(case, g)
        out.append((im, lab) if case["nz"] > 1 else (im[0], lab[0]))
    return out


def _offsets(case):
    return [o for d in range(1, case["reach"] + 1) for o in nyx.nyx_offsets_default(2 if case["nz"] == 1 else 3, d)]


def _cells(case):
    """Most nonzero cells the matrices of a case can have."""
    vox, K = case["images"] * case["nz"] * case["ny"] * case["nx"], len(_offsets(case))
    cells = case["bins"] * (case["bins"] + 1) // 2 if case["symmetric"] else case["bins"] ** 2
    return K * min(vox, case["images"] * case["rois"] * cells)


# ------------------------------------------------------------------ passes
def prepare(case, seed):
    images, ctx = _images(case, seed), nyx.nyx_create(0)
    torch.cuda.synchronize()
    s = {"case": case, "images": images, "ctx": ctx, "offsets": _offsets(case),
         "prec": nyx.NYX_FP64 if case["fp64"] else nyx.NYX_FP32,
         "agg": nyx.NYX_AGG_MERGED if case["merged"] else nyx.NYX_AGG_PER_OFFSET}
    if case["call"] == "plan":
        s["plan"] = nyx.nyx_plan_create(ctx, images, case["bins"], s["offsets"], s["prec"], aggregate=s["agg"],
                                        symmetric=case["symmetric"])
        s["table"] = nyx.new_table(s["plan"], len(s["offsets"]), s["prec"], aggregate=s["agg"])
        s["rois"] = nyx.RoiTable(s["plan"].n_rois, s["table"].device)
    elif case["call"] == "counts":
        # the program's own arrays for the exported counts
        s["key"], s["count"] = (torch.zeros(_cells(case), dtype=torch.int64, device="cuda") for _ in range(2))
    elif case["call"] == "noalloc":
        n = case["images"] * (case["rois"] + 1)
        s["rois"] = nyx.RoiTable(n, images[0][0].device)
        s["table"] = torch.zeros((n, nyx.table_blocks(len(s["offsets"]), s["agg"]), 30), device="cuda",
                                 dtype=torch.float64 if case["fp64"] else torch.float32)
    return s


def _rois(r, n):
    return {"label": r.label[:n], "image": r.image[:n], "n_vox": r.n_vox[:n], "vmin": r.vmin[:n], "vmax": r.vmax[:n],
            "bbox": r.bbox[:n]}


def run(s):
    c, ctx, images, offsets = s["case"], s["ctx"], s["images"], s["offsets"]
    if c["call"] == "plan":
        nyx.nyx_plan_execute(s["plan"], s["table"], s["rois"])
        n = s["plan"].n_rois
        return {"table": s["table"][:n], **_rois(s["rois"], n)}
    if c["call"] == "oneshot":
        rois, table = nyx.nyx_extract_batch(ctx, images, c["bins"], offsets, s["prec"], aggregate=s["agg"],
                                            symmetric=c["symmetric"])
    elif c["call"] == "noalloc":
        n = nyx.nyx_extract_batch_noalloc(ctx, images, c["bins"], offsets, s["rois"], s["table"], s["prec"],
                                          aggregate=s["agg"], symmetric=c["symmetric"])
        rois, table = s["rois"], s["table"][:n]
    elif c["call"] == "intensity":
        rois, table = nyx.nyx_intensity_features(ctx, images, c["bins"], s["prec"])
    elif c["call"] == "neighbourhood":
        rois, table = nyx.nyx_neighbourhood_features(ctx, images, c["bins"], c["alpha"], s["prec"])
    else:
        rois, bins = nyx.nyx_bin_rois(ctx, images, c["bins"], want_bins=True)
        counts = nyx.nyx_glcm_accumulate(ctx, images, rois, c["bins"], offsets, symmetric=c["symmetric"])
        table = nyx.nyx_glcm_features(ctx, counts, s["prec"])
        s["key"][:counts.nnz] = counts.keys
        s["count"][:counts.nnz] = counts.counts
        return {"table": table, "bins": bins, "key": s["key"], "count": s["count"], **_rois(rois, rois.n_rois)}
    return {"table": table, **_rois(rois, rois.n_rois)}


def work(case):
    """Each voxel's intensity and label read once, each output written once;
    two operations per voxel and offset (or neighbour) and a few hundred per
    region and matrix."""
    vox = case["images"] * case["nz"] * case["ny"] * case["nx"]
    rois = case["images"] * (case["rois"] + (1 if case["giant"] else 0))
    size = 8 if case["fp64"] else 4
    K = len(_offsets(case))
    if case["call"] in ("intensity", "neighbourhood"):
        steps, values, mats = (30, 37, 1) if case["call"] == "intensity" else ((8 if case["nz"] == 1 else 26) * 3, 37, 1)
    else:
        steps, values, mats = 2 * K + 4, 30 * nyx.table_blocks(K, 1 if case["merged"] else 0), K
    return {"bytes": 6 * vox + rois * (values * size + 44) + (2 * vox if case["call"] == "counts" else 0),
            "flops": vox * steps + rois * mats * 300}


# ------------------------------------------------------------------ 64 bits
class _Image:
    """One image with its regions numbered from 0 in label order and every
    voxel's grey level (0 outside the regions)."""

    def __init__(self, pair, bins):
        im, lab = (t if t.dim() == 3 else t[None] for t in pair)
        self.value = im.long() & 0xFFFF
        self.shape = lab.shape
        labels, inv = torch.unique(lab, return_inverse=True)
        self.zero = 1 if int(labels[0]) == 0 else 0
        self.label = labels[self.zero:].long()
        self.n = self.label.numel()
        self.roi = inv.reshape(lab.shape) - self.zero        # -1: background
        self.inside = self.roi >= 0
        self.r, self.x = self.roi[self.inside], self.value[self.inside]
        # sums and extremes per region go through `ways` partial ones each, so
        # that the voxels of a large region do not all meet in one place
        self.ways = max(1, min(4096, (1 << 24) // max(1, self.n)))
        self.part = self.r * self.ways + torch.arange(self.r.numel(), device=self.r.device) % self.ways
        ones = torch.ones_like(self.x)
        self.count = self.sum(ones)
        self.vmin, self.vmax = self.edge(self.x, "amin"), self.edge(self.x, "amax")
        D = (self.vmax - self.vmin)[self.r]
        lv = torch.where(D > 0, 1 + bins * (self.x - self.vmin[self.r]) // D.clamp(min=1), ones).clamp(max=bins)
        self.level = torch.zeros_like(self.value)
        self.level[self.inside] = lv
        z, y, x = torch.nonzero(self.inside, as_tuple=True)
        self.at = (x, y, z)
        self.box = torch.stack([self.edge(v, "amin") for v in self.at] + [self.edge(v, "amax") for v in self.at], 1)

    def sum(self, v, at=None, n=None):
        if at is not None:
            return torch.zeros(n, dtype=v.dtype, device=v.device).index_add_(0, at, v)
        return torch.zeros(self.n * self.ways, dtype=v.dtype, device=v.device).index_add_(0, self.part, v).reshape(self.n, -1).sum(1)

    def edge(self, v, how):
        start = (1 << 40) if how == "amin" else -(1 << 40)
        p = torch.full((self.n * self.ways,), start, dtype=torch.int64, device=v.device).scatter_reduce_(0, self.part, v, how)
        p = p.reshape(self.n, -1)
        return p.amin(1) if how == "amin" else p.amax(1)

    def cut(self, off):
        """Views (v, v + off) of the voxels whose neighbour is in the image."""
        a = tuple(slice(max(-d, 0), n - max(d, 0)) for d, n in zip(off, self.shape))
        b = tuple(slice(max(d, 0), n - max(-d, 0)) for d, n in zip(off, self.shape))
        return a, b

    def pairs(self, off):
        """Region and levels of every pair (v, v + off) inside one region."""
        if any(abs(d) >= n for d, n in zip(off, self.shape)):
            return (self.r[:0],) * 3
        a, b = self.cut(off)
        same = (self.roi[a] == self.roi[b]) & self.inside[a]
        return self.roi[a][same], self.level[a][same], self.level[b][same]


def _xlogx(v):
    return torch.where(v > 0, v * torch.log2(v.clamp(min=1e-300)), torch.zeros_like(v))


def _glcm_features(n, bins, r, i, j, c):
    """The 30 features of n matrices given as cells (matrix, i, j, count)."""
    c = c.double()
    acc = lambda at, v, m: torch.zeros(m, dtype=torch.float64, device=v.device).index_add_(0, at, v)  # noqa: E731
    ways = max(1, min(4096, (1 << 24) // max(1, n)))         # partial sums, as in _Image
    part = r * ways + torch.arange(r.numel(), device=c.device) % ways
    S = lambda v: acc(part, v, n * ways).reshape(n, ways).sum(1)  # noqa: E731
    T = S(c)
    p = c / T[r]
    fi, fj = i.double(), j.double()
    px = acc(r * bins + i - 1, p, n * bins).reshape(n, bins)
    py = acc(r * bins + j - 1, p, n * bins).reshape(n, bins)
    ps = acc(r * 2 * bins + i + j, p, n * 2 * bins + 1)[: n * 2 * bins].reshape(n, 2 * bins)
    top = torch.zeros((n, 1), dtype=torch.float64, device=c.device)
    both = (i + j == 2 * bins).nonzero()[:, 0]               # the sum 2 bins falls into the next row's entry 0
    ps[:, 0] = 0.0
    top[:, 0].index_add_(0, r[both], p[both])
    ps = torch.cat([ps, top], 1)
    pd = acc(r * bins + (i - j).abs(), p, n * bins).reshape(n, bins)
    lv = torch.arange(1, bins + 1, device=c.device, dtype=torch.float64)
    sv = torch.arange(0, 2 * bins + 1, device=c.device, dtype=torch.float64)
    dv = lv - 1
    mx, my = (px * lv).sum(1), (py * lv).sum(1)
    vx, vy = (px * (lv - mx[:, None]) ** 2).sum(1), (py * (lv - my[:, None]) ** 2).sum(1)
    one = ((px > 0).sum(1) == 1) | ((py > 0).sum(1) == 1)
    cov = S((fi - mx[r]) * (fj - my[r]) * p)
    HX, HY, H = -_xlogx(px).sum(1), -_xlogx(py).sum(1), -S(_xlogx(p))
    mi = S(p * torch.log2(p / (px[r, i - 1] * py[r, j - 1]))).clamp(min=0)
    dev = fi + fj - (mx + my)[r]
    da, sa = (pd * dv).sum(1), (ps * sv).sum(1)
    dif2 = (fi - fj) ** 2
    asm, acor = S(p * p), S(fi * fj * p)
    hom1, hom2 = (pd / (1 + dv)).sum(1), (pd / (1 + dv * dv)).sum(1)
    idmn, idn = (pd / (1 + dv * dv / bins ** 2)).sum(1), (pd / (1 + dv / bins)).sum(1)
    iv = (pd[:, 1:] / dv[1:] ** 2).sum(1)
    big = torch.zeros(n * ways, dtype=torch.float64, device=c.device).scatter_reduce_(0, part, p, "amax").reshape(n, ways).amax(1)
    zero = torch.zeros_like(mx)
    corr = torch.where(one, zero + 1, cov / (vx * vy).sqrt())
    imc1 = torch.where(one, zero, -mi / torch.maximum(HX, HY))
    imc2 = torch.where(one, zero, (1 - torch.exp(-2 * mi)).sqrt())
    dvar, svar = (pd * (dv - da[:, None]) ** 2).sum(1), (ps * (sv - sa[:, None]) ** 2).sum(1)
    f = torch.stack([asm, acor, S(dev ** 4 * p), S(dev ** 3 * p), S(dev ** 2 * p), S(dif2 * p), corr, da,
                     -_xlogx(pd).sum(1), dvar, da, asm, H, hom1, hom2, hom2, imc1, imc2, idmn, hom1, idn, iv, mx, H, big,
                     sa, -_xlogx(ps).sum(1), vx, svar, vx], 1)
    f[T == 0] = math.nan
    return f


def _glcm_table(im, case):
    """The feature blocks of one image and its sorted counts (matrix rows i <= j
    of symmetric counts with the diagonal halved, or all)."""
    bins, blocks, cells, pooled = case["bins"], [], [], []
    offsets = _offsets(case)
    for k, off in enumerate(offsets):
        r, i, j = im.pairs(off)
        if case["symmetric"]:
            i, j = torch.minimum(i, j), torch.maximum(i, j)
        key, c = torch.unique((r * bins + i - 1) * bins + j - 1, return_counts=True)
        if case["call"] == "counts":
            cells.append((((key // (bins * bins)) << 38) | (k << 32) | ((key // bins % bins) << 16) | (key % bins), c))
        if case["merged"]:
            pooled.append((key, c))
            if k + 1 < len(offsets):
                continue
            key, inv = torch.unique(torch.cat([q for q, _ in pooled]), return_inverse=True)
            c = torch.zeros_like(key).index_add_(0, inv, torch.cat([q for _, q in pooled]))
        r, i, j = key // (bins * bins), key // bins % bins + 1, key % bins + 1
        if case["symmetric"]:
            d = i == j
            o = ~d
            r, i, j, c = torch.cat([r, r[o]]), torch.cat([i, j[o]]), torch.cat([j, i[o]]), torch.cat([torch.where(d, 2 * c, c), c[o]])
        blocks.append(_glcm_features(im.n, bins, r, i, j, c))
    table = torch.stack(blocks, 1)
    if not case["merged"]:
        table = torch.cat([table, table.nanmean(1, keepdim=True)], 1)
    return table, cells


def _intensity_table(im, case):
    n, bins, r, x = im.count.double(), case["bins"], im.r, im.x
    xd = x.double()
    s1 = im.sum(xd)
    mean = s1 / n
    d = xd - mean[r]
    m = {k: im.sum(d ** k) / n for k in (2, 3, 4, 5, 6)}
    flat = im.vmax == im.vmin
    std = lambda k: torch.where(flat, 0 * n, m[k] / torch.where(flat, 0 * n + 1, m[2]) ** (k / 2))  # noqa: E731
    var = torch.where(n > 1, m[2] * n / (n - 1).clamp(min=1), 0 * n)
    order = torch.sort((r << 16) | x)[0] & 0xFFFF
    start = im.count.cumsum(0) - im.count

    def pct(p):
        h = (im.count - 1).double() * p / 100.0
        lo = h.floor().long()
        hi = torch.minimum(lo + 1, im.count - 1)
        a, b = order[start + lo].double(), order[start + hi].double()
        return a + (h - h.floor()) * (b - a)

    p01, p10, p25, med, p75, p90, p99 = (pct(p) for p in (1, 10, 25, 50, 75, 90, 99))
    mid = (xd >= p10[r]) & (xd <= p90[r])
    cm = im.sum(mid.double())
    mm = im.sum(torch.where(mid, xd, 0 * xd)) / cm
    rob = im.sum(torch.where(mid, (xd - mm[r]).abs(), 0 * xd)) / cm
    hist = im.sum(torch.ones_like(x), r * bins + im.level[im.inside] - 1, im.n * bins).reshape(im.n, bins)
    top = hist.max(1, keepdim=True)[0]
    mode = torch.where(hist == top, torch.arange(1, bins + 1, device=x.device), bins + 1).min(1)[0]
    ph = hist.double() / n[:, None]
    lo, hi = im.vmin.double(), im.vmax.double()
    piu = torch.where(hi + lo > 0, 100.0 * (1.0 - (hi - lo) / (hi + lo).clamp(min=1)), 0 * n + 100.0)
    wc = [im.sum(v.double() * xd) / s1 for v in im.at]
    inner = im.inside.clone()
    for axis in range(3):
        if im.shape[0] == 1 and axis == 0:
            continue
        for step in (-1, 1):
            off = [0, 0, 0]
            off[axis] = step
            a, b = im.cut(off)
            keep = torch.zeros_like(inner)
            keep[a] = im.roi[a] == im.roi[b]
            inner &= keep
    e = ~inner[im.inside]
    ne = im.sum(e.double())
    es = im.sum(torch.where(e, xd, 0 * xd))
    emean = es / ne
    esd = (im.sum(torch.where(e, (xd - emean[r]) ** 2, 0 * xd)) / (ne - 1).clamp(min=1)).sqrt()
    emin = im.edge(torch.where(e, x, x + (1 << 20)), "amin").double()
    emax = im.edge(torch.where(e, x, x - (1 << 20)), "amax").double()
    return torch.stack([mean, lo, hi, hi - lo, s1, im.sum(xd * xd), (im.sum(xd * xd) / n).sqrt(), var, var.sqrt(),
                        var.sqrt() / n.sqrt(), std(3), std(4), std(5), std(6), im.sum(d.abs()) / n, med,
                        im.sum((xd - med[r]).abs()) / n, p01, p10, p25, p75, p90, p99, p75 - p25, rob, mode.double(),
                        -_xlogx(ph).sum(1), (ph * ph).sum(1), piu, *wc, es, emin, emax, emean, esd], 1)


def _neighbourhood_table(im, case):
    bins, n, r = case["bins"], im.n, im.r
    wide = (0,) if im.shape[0] == 1 else (-1, 0, 1)
    wn, tot, dep = (torch.zeros_like(im.level) for _ in range(3))
    for off in [(z, y, x) for z in wide for y in (-1, 0, 1) for x in (-1, 0, 1) if (z, y, x) != (0, 0, 0)]:
        a, b = im.cut(off)
        same = (im.roi[a] == im.roi[b]) & im.inside[a]
        wn[a] += same
        tot[a] += torch.where(same, im.level[b], 0 * im.level[b])
        dep[a] += same & ((im.level[a] - im.level[b]).abs() <= case["alpha"])
    i, k = im.level[im.inside], dep[im.inside] + 1
    w, t = wn[im.inside], tot[im.inside]
    nk = 9 if len(wide) == 1 else 27
    N = im.count.double()
    Sm = im.sum(torch.ones_like(i), (r * bins + i - 1) * nk + k - 1, n * bins * nk).reshape(n, bins, nk).double()
    p = Sm / N[:, None, None]
    I = torch.arange(1, bins + 1, device=i.device, dtype=torch.float64)[:, None]
    K = torch.arange(1, nk + 1, device=i.device, dtype=torch.float64)[None]
    rows, cols = Sm.sum(2), Sm.sum(1)
    tot2 = lambda v: v.sum((1, 2))  # noqa: E731
    glm, dcm = tot2(I * p), tot2(K * p)
    glv, dcv = tot2((I - glm[:, None, None]) ** 2 * p), tot2((K - dcm[:, None, None]) ** 2 * p)
    cc, rr = (cols ** 2).sum(1), (rows ** 2).sum(1)
    f = {"DCENRG": tot2(p * p), "DCENT": -tot2(_xlogx(p)), "DCNU": cc / N, "DCNUN": cc / N ** 2, "DCM": dcm, "DCV": dcv,
         "GLNU": rr / N, "GLNUN": rr / N ** 2, "GLM": glm, "GLV": glv, "HDE": tot2(K * K * p),
         "HDHGLE": tot2(I * I * K * K * p), "HDLGLE": tot2(K * K / (I * I) * p), "HGLCE": tot2(I * I * p),
         "LDE": tot2(p / (K * K)), "LDHGLE": tot2(I * I / (K * K) * p), "LDLGLE": tot2(p / (I * I * K * K)),
         "LGLCE": tot2(p / (I * I))}
    has = w > 0
    cnt = im.sum(has.double(), r * bins + i - 1, n * bins).reshape(n, bins)
    s = im.sum(torch.where(has, (i - t.double() / w.clamp(min=1)).abs(), 0.0 * t.double()), r * bins + i - 1, n * bins).reshape(n, bins)
    nv = cnt.sum(1)
    q = cnt / nv.clamp(min=1)[:, None]
    on = (cnt > 0).double()
    ps, ss, ngp = (q * s).sum(1), s.sum(1), on.sum(1)
    con, den, cpx, stg = (torch.zeros(n, dtype=torch.float64, device=i.device) for _ in range(4))
    lv = I[:, 0]
    for a in range(bins):  # pairs of present levels, one level against all
        both = on[:, a:a + 1] * on
        d = (a + 1 - lv).abs()
        con += (both * q[:, a:a + 1] * q * d * d).sum(1)
        den += (both * ((a + 1) * q[:, a:a + 1] - lv * q).abs()).sum(1)
        sq = q[:, a:a + 1] + q
        cpx += (both * d * (q[:, a:a + 1] * s[:, a:a + 1] + q * s) / torch.where(sq > 0, sq, sq + 1)).sum(1)
        stg += (both * sq * d * d).sum(1)
    zero = torch.zeros_like(ps)
    t5 = torch.stack([torch.where(den > 0, ps / den, zero), torch.where(ps > 0, 1 / ps, zero + 1e6), cpx / nv,
                      torch.where(ngp > 1, con / (ngp * (ngp - 1)).clamp(min=1) * ss / nv, zero),
                      torch.where(ss > 0, stg / ss, zero)], 1)
    t5[nv == 0] = math.nan
    gl = ["LDE", "HDE", "GLNU", "DCNU", "DCNUN", "GLV", "DCV", "DCENT", "LGLCE", "HGLCE", "LDLGLE", "LDHGLE", "HDLGLE", "HDHGLE"]
    return torch.cat([torch.stack([f[v] for v in f], 1), t5, torch.stack([f[v] for v in gl], 1)], 1)


def exact(case, seed):
    tables, rois, keys, counts, bins, base = [], [], [], [], [], 0
    for at, pair in enumerate(_images(case, seed)):
        im = _Image(pair, case["bins"])
        if case["call"] == "intensity":
            tables.append(_intensity_table(im, case))
        elif case["call"] == "neighbourhood":
            tables.append(_neighbourhood_table(im, case))
        else:
            table, cells = _glcm_table(im, case)
            tables.append(table)
            for key, c in cells:
                keys.append(key + (base << 38))
                counts.append(c)
        rois.append((im.label.int(), torch.full_like(im.label, at).int(), im.count, im.vmin.short(), im.vmax.short(), im.box.int()))
        if case["call"] == "counts":
            bins.append(im.level.reshape(-1).short())
        base += im.n
    out = {"table": torch.cat(tables)}
    if case["call"] == "counts":
        key, order = torch.sort(torch.cat(keys))
        rest = torch.zeros(_cells(case) - key.numel(), dtype=torch.int64, device="cuda")
        out.update(bins=torch.cat(bins), key=torch.cat([key, rest]), count=torch.cat([torch.cat(counts)[order], rest]))
    names = ("label", "image", "n_vox", "vmin", "vmax", "bbox")
    out.update({k: torch.cat([r[m] for r in rois]) for m, k in enumerate(names)})
    return out
