"""What users of this library have it do, as cases that can be timed one by one.

Three kinds of work:
  call  one product with one packed matrix, issued eagerly (gqsa_gemv);
  step  the linear layers of a few decoder layers, issued as a decoder issues them: the matrices
        that share their input in one call (q/k/v, gate/up: gqsa_gemv_multi), o and down on their
        own -- either eagerly, or captured once in a HIP graph which every token replays;
  pack  the offline step on the GPU (gqsa_pack_device) and the arrays it hands back (gqsa_export).

Shapes are the linear-layer dimensions of the benchmark (bench.py, gqsa_inputs.py) or generic
ones.  The matrices of a step are distinct, as the layers of a model are, so its weights come from
memory and not from a cache.  Weights and activations have the distributions of gqsa_inputs.py, drawn on the GPU.
"""
from __future__ import annotations

import numpy as np
import torch

import gqsa_inputs as gi
import paper_2412_17560_amd as gq

DEVICE = "cuda:0"


def _call(name, n, k, bits=4, group=16, sparsity=0.5, batch=1, panels=False, balanced=True):
    return {"name": name, "kind": "call", "n": n, "k": k, "bits": bits, "group": group, "sparsity": sparsity,
            "batch": batch, "panels": panels, "balanced": balanced}


def _step(name, hidden, kv, ffn, layers, bits=4, group=16, sparsity=0.5, batch=1, panels=False, graph=True):
    return {"name": name, "kind": "step", "hidden": hidden, "kv": kv, "ffn": ffn, "layers": layers, "bits": bits,
            "group": group, "sparsity": sparsity, "batch": batch, "panels": panels, "graph": graph}


def listed():
    return [
        # the smallest projection of a decoder layer, called by itself: launch and call overhead
        _call("call_kv", 1024, 4096),
        # one layer, every call issued eagerly: a program that does not capture graphs
        _step("layer_eager", 4096, 4096, 11008, layers=1, graph=False),
        # token generation, one sequence: the benchmark's layer set
        _step("decode_b1", 4096, 4096, 11008, layers=4),
        # the same with grouped-query attention, a wider feed-forward part and milder pruning (ragged rows of groups)
        _step("decode_gqa_s30_b1", 4096, 1024, 14336, layers=2, sparsity=0.3),
        # 8-bit codes
        _step("decode_gqa_w8_b1", 4096, 1024, 14336, layers=2, bits=8),
        # a few sequences at once, without the second image (it doubles the memory of the weights)
        _step("decode_b4", 4096, 4096, 11008, layers=2, batch=4),
        # small batches from the second image: the matrix cores
        _step("decode_b16", 4096, 4096, 11008, layers=2, batch=16, panels=True),
        _step("decode_gqa_w8_b8", 4096, 1024, 14336, layers=1, bits=8, batch=8, panels=True),
        # the vocabulary projection: the largest matrix a decoder multiplies
        _call("call_vocab", 128256, 4096),
        # rows pruned to very different lengths, some empty, some full
        _call("call_imbalanced", 28672, 8192, balanced=False),
        # larger groups and sizes that fill no tile, two rows
        _call("call_g64_ragged_b2", 5003, 4160, group=64, sparsity=0.4, batch=2),
        # offline: prune, quantise and lay out one matrix
        {"name": "pack_attention", "kind": "pack", "n": 4096, "k": 4096, "bits": 4, "group": 16, "sparsity": 0.5},
    ]


def _log_uniform(rng, low, high, multiple=1):
    v = low * (high / low) ** rng.random()
    return max(multiple, int(round(v / multiple)) * multiple)


MOST_BYTES = 3.4e8            # of a drawn case's stored groups
MOST_HOST_WEIGHTS = 2.5e8     # weights that prepare() packs on the host, for the second image


def draw(rng):
    """One more case of the same ranges: matrices from 200 rows to 130000, 256 to 16384 columns."""
    kind = rng.choice(["call", "call", "call", "step", "step", "step", "pack"])
    bits = rng.choice([4, 4, 4, 8])
    sparsity = round(rng.choice([0.0, 0.3, 0.5, 0.5, 0.5, 0.7, rng.uniform(0.0, 0.8)]), 3)
    group = rng.choice([16, 16, 16, 16, 32, 64] + ([128] if bits == 4 else [8]))
    batch = rng.choice([1, 1, 1, 2, 3, 4, 8, 16, rng.randint(1, 16)])
    panels = batch >= 5 and group >= 16
    per_weight = (group * bits // 8 + 6) / group        # bytes of a stored weight
    if kind == "pack":
        k = _log_uniform(rng, 1024, 16384, 128)
        return {"kind": "pack", "n": _log_uniform(rng, 500, 40_000_000 // k), "k": k, "bits": bits, "group": group, "sparsity": sparsity}
    unit = max(group, 16)
    if kind == "call":
        k = _log_uniform(rng, 256, 16384, unit)
        most = min(MOST_HOST_WEIGHTS if panels else 6e8, MOST_BYTES / per_weight) / k
        case = _call("", _log_uniform(rng, 200, min(130_000, int(most))), k, bits, group, sparsity, batch, panels,
                     balanced=rng.random() < 0.75)
    else:
        hidden = _log_uniform(rng, 1024, 5120, unit)
        ffn = int(hidden * rng.uniform(2.5, 3.8)) // unit * unit
        kv = hidden // rng.choice([1, 1, 4, 8])
        weights = 2 * hidden * hidden + 2 * kv * hidden + 3 * ffn * hidden
        stored = weights * (1.0 - sparsity) * per_weight
        layers = max(1, min(4, int(MOST_BYTES // stored), int((MOST_HOST_WEIGHTS if panels else 9e8) // weights)))
        if stored > MOST_BYTES or (panels and weights > MOST_HOST_WEIGHTS):     # a wide layer that is hardly pruned: half as wide
            hidden, kv, ffn = (v // 2 // unit * unit for v in (hidden, kv, ffn))
        case = _step("", hidden, kv, ffn, layers, bits, group, sparsity, batch, panels, graph=rng.random() < 0.7)
    del case["name"]
    return case


# --------------------------------------------------------------------------- inputs, made on the GPU
def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _weights(n, k, gen):
    """fp32 [n, k] ~ N(0, 0.02), 1 % of the columns times 20 (outlier channels)."""
    w = torch.randn((n, k), generator=gen, device=DEVICE)
    w.mul_(0.02)
    columns = torch.randperm(k, generator=gen, device=DEVICE)[: max(1, round(0.01 * k))]
    gain = torch.ones(k, device=DEVICE)
    gain[columns] = 20.0
    return w.mul_(gain)


def _activations(batch, k, gen):
    return torch.randn((batch, k), generator=gen, device=DEVICE).to(torch.float16)


def _keep_counts(case, seed):
    """Kept groups per row of a matrix pruned to different lengths, None if every row keeps as many."""
    if case.get("balanced", True):
        return None
    return gi.imbalanced_keep_counts(case["n"], case["k"] // case["group"], seed=seed % (1 << 32))


def _packed(case, n, k, gen, keep=None):
    w = _weights(n, k, gen)
    if not case["panels"]:
        return gq.gqsa_pack_device(w, case["group"], case["bits"], case["sparsity"], keep_per_row=keep)
    w = w.cpu().numpy()        # the second image is built on the host, ahead of the upload
    h = (gq.gqsa_pack(w, case["group"], case["bits"], case["sparsity"]) if keep is None
         else gq.gqsa_pack_rows(w, keep, case["group"], case["bits"]))
    gq.gqsa_build_panels(h)
    gq.gqsa_upload(h)
    return h


def _issue(calls):
    for handles, x, ys in calls:
        if len(handles) == 1:
            gq.gqsa_gemv(handles[0], x, ys[0])
        else:
            gq.gqsa_gemv_multi(handles, x, ys)


def prepare(case, seed):
    gen = _generator(seed)
    if case["kind"] == "pack":
        return {"w": _weights(case["n"], case["k"], gen), "case": case}
    batch = case["batch"]

    def outputs(n):
        return torch.empty((batch, n), dtype=torch.float16, device=DEVICE)

    if case["kind"] == "call":
        h = _packed(case, case["n"], case["k"], gen, _keep_counts(case, seed))
        calls = [([h], _activations(batch, case["k"], gen), [outputs(case["n"])])]
        return {"calls": calls, "outputs": calls[0][2], "graph": None, "case": case}

    hidden, kv, ffn = case["hidden"], case["kv"], case["ffn"]
    calls = []
    for _ in range(case["layers"]):
        for sizes, k in (((hidden, kv, kv), hidden), ((hidden,), hidden), ((ffn, ffn), hidden), ((hidden,), ffn)):
            calls.append(([_packed(case, n, k, gen) for n in sizes], _activations(batch, k, gen), [outputs(n) for n in sizes]))
    graph = None
    if case["graph"]:
        graph = torch.cuda.CUDAGraph()
        _issue(calls)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            _issue(calls)
    return {"calls": calls, "outputs": [y for c in calls for y in c[2]], "graph": graph, "case": case}


def run(state):
    case = state["case"]
    if case["kind"] == "pack":
        h = gq.gqsa_pack_device(state["w"], case["group"], case["bits"], case["sparsity"])
        return gq.gqsa_export(h)
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _issue(state["calls"])
    return state["outputs"]


# --------------------------------------------------------------------------- the same products in float64
def _exact_product(case, w, x, keep=None):
    """x W^T in float64 with W pruned and quantised as the format defines it, a slab of rows at a time.  The saliency
    of a group is the float64 sum of its squares in index order (the squares are exact), the quantiser's steps are
    single fp32 operations: both are reproduced to the last bit, so the same groups are kept with the same codes.
    (An fp32 quotient taken in float64 and rounded to fp32 is the fp32 quotient.)"""
    group, levels = case["group"], float(2 ** case["bits"] - 1)
    n, k = w.shape
    columns = k // group
    kept = torch.full((n,), columns - int(case["sparsity"] * columns + 0.5)) if keep is None else torch.as_tensor(np.asarray(keep))
    dropped = (columns - kept).to(w.device)
    y = torch.empty((x.shape[0], n), dtype=torch.float64, device=w.device)
    slab = max(1, (1 << 24) // k)
    for r in range(0, n, slab):
        g = w[r:r + slab].view(-1, columns, group)
        saliency = torch.zeros(g.shape[:2], dtype=torch.float64, device=w.device)
        for j in range(group):
            saliency += g[:, :, j].double().square()
        order = torch.sort(saliency, dim=1, stable=True).indices        # of equal ones the lower column goes first
        place = torch.empty_like(order).scatter_(1, order, torch.arange(columns, device=w.device).expand_as(order))
        low = g.amin(dim=2, keepdim=True)
        scale = ((g.amax(dim=2, keepdim=True) - low).double() / levels).float().half().double().clamp_(min=2.0 ** -14)
        zero = torch.round((-low.double() / scale).float()).clamp_(-2048.0, 2048.0).double()
        codes = (torch.round((g.double() / scale).float()).double() + zero).clamp_(0.0, levels)
        weights = (codes - zero) * scale * (place >= dropped[r:r + slab, None])[:, :, None]
        y[:, r:r + slab] = x.double() @ weights.view(-1, k).t()
    return y


def exact(case, seed):
    """What run() returns for these inputs, in float64 with plain torch.  Packing is compared bit for bit and has none."""
    if case["kind"] == "pack":
        return None
    gen = _generator(seed)
    if case["kind"] == "call":
        calls = [((case["n"],), case["k"])]
    else:
        hidden, kv, ffn = case["hidden"], case["kv"], case["ffn"]
        calls = [((hidden, kv, kv), hidden), ((hidden,), hidden), ((ffn, ffn), hidden), ((hidden,), ffn)] * case["layers"]
    results = []
    for sizes, k in calls:
        held = [_weights(n, k, gen) for n in sizes]      # drawn in the order in which prepare() draws them
        x = _activations(case["batch"], k, gen)
        results += [_exact_product(case, w, x, _keep_counts(case, seed)) for w in held]
    return results


# --------------------------------------------------------------------------- what a pass cannot do without
def _matrices(case):
    """(rows, columns, stored groups) of every matrix of a pass, and (columns) of every input."""
    def kept(n, k):
        columns = k // case["group"]
        return n * (columns - int(case["sparsity"] * columns + 0.5))

    if case["kind"] != "step":
        n, k = case["n"], case["k"]
        keep = _keep_counts(case, 1)
        return [(n, k, kept(n, k) if keep is None else int(np.sum(keep)))], [k]
    hidden, kv, ffn = case["hidden"], case["kv"], case["ffn"]
    shapes = [(hidden, hidden), (kv, hidden), (kv, hidden), (hidden, hidden), (ffn, hidden), (ffn, hidden), (hidden, ffn)]
    return [(n, k, kept(n, k)) for n, k in shapes] * case["layers"], [hidden, hidden, hidden, ffn] * case["layers"]


def work(case):
    """A stored group: its codes, scale, zero and index word; a row pointer per row; the input and the result
    once.  Packing: the weights once, the arrays and the image (the same bytes again) written once."""
    matrices, inputs = _matrices(case)
    code_bytes = case["group"] * case["bits"] // 8
    image = sum(groups * (code_bytes + 6) + 4 * (n + 1) for n, _, groups in matrices)
    if case["kind"] == "pack":
        n, k, groups = matrices[0]
        return {"bytes": 4 * n * k + groups * (code_bytes + 8) + 4 * (n + 1) + image, "flops": 0}
    batch = case["batch"]
    return {"bytes": image + 2 * batch * (sum(inputs) + sum(n for n, _, _ in matrices)),
            "flops": 2 * batch * case["group"] * sum(groups for _, _, groups in matrices)}


def tolerance(case):
    """Packing fixes every tie, so its arrays are exact.  A product is summed in fp32 and rounded once to fp16: against
    float64 its 2-norm is off by 2.1e-4 and no value by more than 4.9e-4, which is the rounding of the result."""
    return "exact" if case["kind"] == "pack" else {"rel": 8e-4, "max": 2e-3}
