"""Performance cases of the local NBNN library, through its public entry points.

The library classifies images from their 128-byte (or float, or 160-byte
location-augmented) descriptors against one resident index.  A case fixes the
index (classes x references per class), the batch (images, descriptors per
image), the neighbourhood size k, the search mode and the form of the call:

  classify  device tensors in and out (``lnbnn_classify``), or host arrays
            where ``host`` is true;
  serve     requests submitted one by one to the serving loop and polled
            (``lnbnn_submit`` / ``lnbnn_poll``), host data by nature;
  build     a new index from device tensors and the first image classified
            against it (``lnbnn_build_index``, then ``lnbnn_classify``).

Sizes are those of the synthetic workloads this repository tests and
benchmarks: 10 classes x 1,000 references; 101 x 22,500; 256 x 60,000;
the two-class end of the class sweep; images of 200, 1,500 and 500..4,000
descriptors; k in 1, 5, 10, 20.  Data follow the same recipe (prototype and
background means plus noise), drawn on the GPU from the seed.
"""
import math
import random
import time

import numpy as np
import torch

import paper_1112_0059_amd as L

MODES = {
    "i8": L.LNBNN_EXACT_I8,
    "f16": L.LNBNN_EXACT_F16,
    "bf16": L.LNBNN_EXACT_BF16,
    "nbnn": L.LNBNN_NBNN_I8,
    "fp8": L.LNBNN_FP8_RERANK,
    "fp8_2k": L.LNBNN_FP8_RERANK_2K,
}
FLOAT = ("fp8", "fp8_2k")
TUNING_CACHE = "paper_1112_0059_amd/tuning_cache.json"
PROTOS, BACKGROUNDS, P_BACKGROUND = 12, 16, 0.25
CHUNK = 1 << 20


def _case(name, mode, classes, per_class, images, desc, k, neighbours=True, dim=128, form="classify", host=False,
          tuned=False):
    lo, hi = desc if isinstance(desc, tuple) else (desc, desc)
    c = dict(mode=mode, classes=classes, per_class=per_class, images=images, desc_lo=lo, desc_hi=hi, k=k,
             neighbours=neighbours and mode != "nbnn" and form != "serve", dim=dim, form=form, host=host, tuned=tuned)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one image of the tiny parity set; launches and
        # host work count, not arithmetic
        _case("i8_tiny_one_image", "i8", 10, 1000, 1, 200, 10),
        # interactive use: one image of odd size against the 15.36M-reference
        # index, which a single image cannot fill with query blocks
        _case("i8_256c_one_image", "i8", 256, 60000, 1, 2251, 10),
        # a moderate batch on the 101-class index, k = 5
        _case("i8_101c_batch", "i8", 101, 22500, 32, 1500, 5),
        # the headline workload's index, mode and k with a quarter of its
        # images, tuned from the committed cache as the benchmark does
        _case("i8_256c_batch_tuned", "i8", 256, 60000, 128, (500, 4000), 10, neighbours=False, tuned=True),
        # the small end of the class sweep: a short sweep per descriptor
        _case("i8_2c_sweep", "i8", 2, 60000, 64, (500, 4000), 10),
        # the 16-bit exact path with longer lists
        _case("f16_101c_k20", "f16", 101, 22500, 16, (500, 4000), 20),
        # the original rule (Algorithm 1) on the 101-class index
        _case("nbnn_101c_batch", "nbnn", 101, 22500, 32, 1500, 10),
        # float descriptors: FP8 candidates and exact re-rank, few images
        # against the large index
        _case("fp8_256c_few_images", "fp8", 256, 60000, 8, (500, 4000), 10),
        # the cheaper candidate rule on one image, where the re-rank and
        # reduction are a large part
        _case("fp8_2k_101c_one_image", "fp8_2k", 101, 22500, 1, 1999, 10),
        # location-augmented rows, a few images
        _case("i8_loc_101c_batch", "i8", 101, 22500, 8, (500, 4000), 10, dim=160),
        # continuous batching: a burst of requests of mixed size
        _case("i8_101c_serve", "i8", 101, 22500, 24, (100, 4000), 10, form="serve"),
        # a new index and its first image
        _case("i8_101c_build", "i8", 101, 22500, 1, 1500, 10, form="build"),
    ]


def _sizes(case):
    """Descriptors of each image: fixed by the case alone."""
    r = random.Random(1000003 * case["images"] + 1009 * case["desc_lo"] + case["desc_hi"])
    return [r.randint(case["desc_lo"], case["desc_hi"]) for _ in range(case["images"])]


def _cost(case):
    weight = {"f16": 2.0, "bf16": 2.0, "fp8": 1.4, "fp8_2k": 1.2}.get(case["mode"], 1.0)
    return weight * case["dim"] * case["classes"] * case["per_class"] * (sum(_sizes(case)) + 600)


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    largest = max(_cost(c) for c in listed())
    while True:
        mode = rng.choice(["i8", "i8", "i8", "i8_loc", "f16", "bf16", "nbnn", "fp8", "fp8", "fp8_2k"])
        mode, dim = ("i8", 160) if mode == "i8_loc" else (mode, 128)
        lo = log_int(50, 3000)
        hi = min(4000, lo + (log_int(1, 2500) if rng.random() < 0.7 else 0))
        form = rng.choice(["classify"] * 8 + ["serve", "build"])
        c = _case(None, mode, log_int(2, 256), log_int(100, 60000), log_int(1, 128), (lo, hi),
                  rng.choice([1, 2, 5, 10, 10, 10, 15, 20, 32]), neighbours=rng.random() < 0.6, dim=dim, form=form,
                  host=form == "classify" and rng.random() < 0.15)
        if c["classes"] * c["per_class"] >= 4 * c["k"] + 1 and _cost(c) <= largest:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rows(case, g, means, backgrounds, cls):
    """Descriptors of the classes in `cls` (one row each): a prototype of the
    class or a shared background mean, plus noise."""
    n, dev = cls.shape[0], cls.device
    proto = torch.randint(PROTOS, (n,), generator=g, device=dev)
    is_bg = torch.rand(n, generator=g, device=dev) < P_BACKGROUND
    bg = torch.randint(BACKGROUNDS, (n,), generator=g, device=dev)
    x = torch.where(is_bg[:, None], backgrounds["mean"][bg], means["mean"][cls, proto])
    noise = torch.randn(n, 128, generator=g, device=dev)
    if case["mode"] in FLOAT:
        return torch.nn.functional.normalize((x + 0.08 * noise).clamp_min_(0.0) + 1e-12, dim=1)
    x = (x + 20.0 * noise).round_().clamp_(0, 255).to(torch.uint8)
    if case["dim"] == 160:
        at = means["centre"][cls, proto] + 0.08 * torch.randn(n, 2, generator=g, device=dev)
        at = torch.where(is_bg[:, None], torch.rand(n, 2, generator=g, device=dev), at).clamp_(0, 1)
        code = (204.8 * at).round_().to(torch.uint8)
        x = torch.cat([x, code[:, :1].expand(n, 16), code[:, 1:].expand(n, 16)], dim=1)
    return x


def _inputs(case, seed):
    """(references, labels, queries, offsets): device tensors, host offsets."""
    dev = "cuda"
    g = torch.Generator(device=dev).manual_seed(seed * 2 + 1)
    nc, n = case["classes"], case["classes"] * case["per_class"]
    fl = case["mode"] in FLOAT
    means, backgrounds = {}, {}
    for d, shape in ((means, (nc, PROTOS)), (backgrounds, (BACKGROUNDS,))):
        if fl:
            m = torch.randn(*shape, 128, generator=g, device=dev).clamp_min_(0.0)
            d["mean"] = torch.nn.functional.normalize(m, dim=-1)
        else:
            d["mean"] = 255.0 * torch.rand(*shape, 128, generator=g, device=dev)
    means["centre"] = 0.15 + 0.7 * torch.rand(nc, PROTOS, 2, generator=g, device=dev)
    labels = torch.arange(n, device=dev, dtype=torch.int32) // case["per_class"]
    refs = torch.empty(n, case["dim"], dtype=torch.float32 if fl else torch.uint8, device=dev)
    for at in range(0, n, CHUNK):
        refs[at:at + CHUNK] = _rows(case, g, means, backgrounds, labels[at:at + CHUNK].long())
    sizes = _sizes(case)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    cls = torch.repeat_interleave(torch.arange(case["images"]) % nc, torch.tensor(sizes)).to(dev)
    queries = torch.empty(int(offsets[-1]), case["dim"], dtype=refs.dtype, device=dev)
    for at in range(0, queries.shape[0], CHUNK):
        queries[at:at + CHUNK] = _rows(case, g, means, backgrounds, cls[at:at + CHUNK])
    return refs, labels, queries, offsets


def prepare(case, seed):
    refs, labels, queries, offsets = _inputs(case, seed)
    mode = MODES[case["mode"]]
    s = {"case": case, "mode": mode, "queries": queries, "offsets": offsets, "mask": L.LNBNN_MODE_BIT(mode)}
    if case["form"] == "build":
        s["refs"], s["labels"] = refs, labels
        return s
    s["index"] = L.lnbnn_build_index(refs, labels, case["classes"], s["mask"])
    del refs, labels
    if case["tuned"]:
        L.lnbnn_autotune(s["index"], queries, offsets, case["k"], mode, cache_path=TUNING_CACHE)
    if case["form"] == "serve":
        q = queries.cpu().numpy()
        s["requests"] = [np.ascontiguousarray(q[a:b]) for a, b in zip(offsets[:-1], offsets[1:])]
    elif case["host"]:
        s["queries"] = queries.cpu().numpy()
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _answer(out):
    names = ("class", "totals", "nbr_idx", "nbr_dist")
    return {n: v for n, v in zip(names, out) if v is not None}


def run(state):
    case, mode, k = state["case"], state["mode"], state["case"]["k"]
    if case["form"] == "build":
        ix = L.lnbnn_build_index(state["refs"], state["labels"], case["classes"], state["mask"])
        out = L.lnbnn_classify(ix, state["queries"], state["offsets"], k, mode, want_neighbours=case["neighbours"])
        ix.free()
        return _answer(out)
    ix = state["index"]
    if case["form"] == "serve":
        tickets = [L.lnbnn_submit(ix, q, k, mode) for q in state["requests"]]
        classes, totals = [], []
        for t in tickets:
            while (r := L.lnbnn_poll(ix, t)) is None:
                time.sleep(0.0002)
            classes.append(r[0])
            totals.append(r[1])
        return {"class": np.array(classes, np.int32), "totals": np.stack(totals)}
    return _answer(L.lnbnn_classify(ix, state["queries"], state["offsets"], k, mode,
                                    want_neighbours=case["neighbours"]))


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its exact result
# ---------------------------------------------------------------------------
def work(case):
    n, nq, dim, k = case["classes"] * case["per_class"], sum(_sizes(case)), case["dim"], case["k"]
    fl = case["mode"] in FLOAT
    row = 2 * dim if case["mode"] in ("f16", "bf16") else dim      # the index as its mode holds it
    nbytes = n * (row + 4) + nq * dim * (4 if fl else 1)           # operands and norms, queries
    if fl:
        nbytes += nq * 4 * k * dim * 4                             # the candidates' FP32 rows
    nbytes += case["images"] * (case["classes"] * 8 + 4)           # totals, classes
    if case["neighbours"]:
        nbytes += nq * (k + 1) * 8
    if case["form"] == "build":
        nbytes += n * (dim * (4 if fl else 1) + 4 + row)           # references and labels in, index out
    return {"bytes": nbytes, "flops": 2.0 * dim * n * nq}


def exact(case, seed):
    """Algorithm 2 (or 1) on brute-force distances in float64.  Neighbour
    indices and classes depend on ties (and, in the FP8 modes, on the
    candidate pass): no value."""
    n, nq, k = case["classes"] * case["per_class"], sum(_sizes(case)), case["k"]
    if n * nq > 4e11:
        return None
    refs, labels, queries, offsets = _inputs(case, seed)
    labels = labels.long()
    dev, nc = queries.device, case["classes"]
    image = torch.repeat_interleave(torch.arange(case["images"]), torch.from_numpy(np.diff(offsets))).to(dev)
    totals = torch.zeros(case["images"], nc, dtype=torch.float64, device=dev)
    dist = torch.empty(nq, k + 1, dtype=torch.float64, device=dev)
    qb, rb, grp = 4096, 1 << 17, 64
    for a in range(0, nq, qb):
        q = queries[a:a + qb].double()
        m = q.shape[0]
        qq = (q * q).sum(1, keepdim=True)
        best = torch.full((m, k + 1), math.inf, dtype=torch.float64, device=dev)
        lab = torch.zeros(m, k + 1, dtype=torch.long, device=dev)
        nearest = torch.full((m, nc), math.inf, dtype=torch.float64, device=dev)
        for b in range(0, n, rb):
            r = refs[b:b + rb].double()
            d = torch.addmm(qq + (r * r).sum(1)[None, :], q, r.t(), alpha=-2.0)
            if case["mode"] == "nbnn":
                for c in range(int(labels[b]), int(labels[min(n, b + rb) - 1]) + 1):   # contiguous classes
                    lo, hi = max(b, c * case["per_class"]) - b, min(b + rb, (c + 1) * case["per_class"], n) - b
                    nearest[:, c] = torch.minimum(nearest[:, c], d[:, lo:hi].amin(1))
                continue
            cols = r.shape[0]
            pad = -cols % grp
            if pad:
                d = torch.nn.functional.pad(d, (0, pad), value=math.inf)
            # the k + 1 smallest lie in the k + 1 groups with the smallest minima
            d = d.view(m, -1, grp)
            gi = torch.topk(d.amin(2), min(k + 1, d.shape[1]), dim=1, largest=False).indices
            dd = torch.gather(d, 1, gi[:, :, None].expand(-1, -1, grp)).reshape(m, -1)
            ii = (gi[:, :, None] * grp + torch.arange(grp, device=dev)).reshape(m, -1)
            dd = torch.cat([best, dd], 1)
            ll = torch.cat([lab, labels[(b + ii).clamp_max_(n - 1)]], 1)
            best, at = torch.topk(dd, k + 1, dim=1, largest=False, sorted=True)
            lab = torch.gather(ll, 1, at)
        if case["mode"] == "nbnn":
            totals.index_add_(0, image[a:a + qb], nearest)
            continue
        dist[a:a + qb] = best
        for j in range(k):
            first = torch.ones(m, dtype=torch.bool, device=dev)
            for i in range(j):
                first &= lab[:, i] != lab[:, j]
            delta = torch.where(first, best[:, j] - best[:, k], torch.zeros_like(best[:, k]))
            totals.view(-1).index_add_(0, image[a:a + qb] * nc + lab[:, j], delta)
    out = {"class": None, "totals": totals}
    if case["neighbours"]:
        out["nbr_idx"], out["nbr_dist"] = None, dist
    return out
