"""The work this library is timed on: contractions, gradients, chains,
permutes and batches through the public entry points of
paper_2102_06827_amd, over the sizes its users bring.

listed()        the named cases
draw(rng)       one more case of the same kinds and ranges
prepare(case)   the inputs on the GPU and the plan or batch a program keeps
run(state)      one pass, returning its whole outputs
work(case)      the bytes and operations a pass cannot do without
exact(case)     the same outputs in 64 bits, from plain torch

Labels a-h are virtual orbitals and i-p occupied ones, as in coupled-cluster
theory; the counts of either come from the molecule and the basis set, so odd
and ragged extents are as common as round ones.
"""
import math

import torch

import paper_2102_06827_amd as comet

_DTYPE = {"f64": torch.float64, "f32": torch.float32}
_SIZE = {"f64": 8, "f32": 4}

# two-virtual two-occupied contractions: block-interleaved, the CCSD-like one,
# a plain matrix product, a transposed output, summation labels at both ends
# of an operand, and an operand whose unit-stride label is free
PATTERNS = ["abij=acik*cbkj", "abij=acik*bkcj", "abij=abcd*cdij", "abij=ijcd*cdab", "abij=ciak*bkjc",
            "ajbi=kcia*cjkb"]
CHAINS = ["ia=cdmn*inad*mc", "ia=cdmn*id*na*mc", "abij=mnef*am*fn*ebij"]
PERMUTES = ["aick=acik", "ijab=abij", "abcijk=aijbck", "ji=ij", "baji=abij"]
BATCHED = ["bij=bik*bkj", "ibj=kbi*jbk"]
SPLITS = ["split_int8", "split_bf16", "split_bf16x3", "split_fp16x2"]


def _operands(spec):
    out, rhs = spec.split("=")
    return out, rhs.split("*")


def _extents(case):
    """label -> extent"""
    if "extents" in case:
        return {kv.split("=")[0]: int(kv.split("=")[1]) for kv in case["extents"].split(",")}
    return {ch: case["virtual"] if ch in "abcdefgh" else case["occupied"]
            for ch in case["spec"] if ch.isalpha()}


def _shape(labels, ext):
    return tuple(ext[ch] for ch in labels)


def _count(labels, ext):
    return math.prod(ext[ch] for ch in labels)


def _problems(case):
    """The (spec, extents) of a batch, from the case alone."""
    import random
    rng = random.Random(case["problems_seed"])
    step = case["step"]
    out = []
    for _ in range(case["problems"]):
        spec = rng.choice(PATTERNS)
        labels = sorted(set(spec) - {"=", "*"})
        out.append((spec, {ch: step * rng.randint(-(-8 // step), case["largest"] // step) for ch in labels}))
    return out


def _grad_specs(spec):
    c, (a, b) = _operands(spec)
    return "%s=%s*%s" % (a, c, b), "%s=%s*%s" % (b, a, c)


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def listed():
    return [
        # one small binary contraction from a program's inner loop (a small
        # molecule's step), called by spec: latency and launches
        {"name": "small_f64", "kind": "contract", "spec": "abij=acik*cbkj", "law": "uniform", "dtype": "f64",
         "compute": "default", "extents": "a=16,b=16,c=16,i=16,j=16,k=16"},
        # the particle-hole term of a CCSD iteration, planned once and run on
        # every iteration's amplitudes
        {"name": "ccsd_f64", "kind": "plan", "spec": "abij=acik*bkcj", "law": "decay", "dtype": "f64",
         "compute": "default", "virtual": 96, "occupied": 32},
        # the same for a molecule whose orbital counts are odd
        {"name": "ccsd_odd_f64", "kind": "plan", "spec": "abij=acik*bkcj", "law": "decay", "dtype": "f64",
         "compute": "default", "virtual": 75, "occupied": 23},
        # single-precision amplitudes of an ordinary size
        {"name": "ccsd_f32", "kind": "contract", "spec": "abij=ciak*bkjc", "law": "decay", "dtype": "f32",
         "compute": "default", "virtual": 80, "occupied": 28},
        # the same term in split precision at FP64-class error
        {"name": "ccsd_int8", "kind": "plan", "spec": "abij=acik*bkcj", "law": "decay", "dtype": "f64",
         "compute": "split_int8", "virtual": 96, "occupied": 32},
        # single precision on the 16-bit matrix cores, extents that are not
        # multiples of a vector
        {"name": "ccsd_bf16x3", "kind": "contract", "spec": "abij=acik*bkcj", "law": "decay", "dtype": "f32",
         "compute": "split_bf16x3", "virtual": 66, "occupied": 22},
        # fitting amplitudes: the update C0 + A * B, forward and backward
        {"name": "grad_f64", "kind": "grad", "spec": "abij=acik*cbkj", "law": "decay", "dtype": "f64",
         "compute": "default", "virtual": 60, "occupied": 20},
        # a triples-like term: a short summation into a six-index output
        {"name": "triples_f64", "kind": "plan", "spec": "abcijk=daij*bcdk", "law": "uniform", "dtype": "f64",
         "compute": "default", "virtual": 32, "occupied": 16},
        # a four-operand term by its cheapest grouping
        {"name": "chain_f64", "kind": "chain", "spec": "abij=mnef*am*fn*ebij", "law": "uniform", "dtype": "f64",
         "compute": "default", "virtual": 96, "occupied": 32},
        # amplitudes brought into another index order, odd extents
        {"name": "permute_f64", "kind": "permute", "spec": "ijab=abij", "law": "uniform", "dtype": "f64",
         "virtual": 99, "occupied": 33},
        # many uneven contractions in one launch, with both their gradients
        {"name": "batch_f32", "kind": "batch", "dtype": "f32", "compute": "default", "problems": 96,
         "problems_seed": 5001, "step": 8, "largest": 64},
        # a label in all three tensors: many small products (one per point
        # group block or k point)
        {"name": "blocks_f64", "kind": "contract", "spec": "bij=bik*bkj", "law": "uniform", "dtype": "f64",
         "compute": "default", "extents": "b=4096,i=64,j=64,k=64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["small", "ccsd", "ccsd", "ccsd", "split", "grad", "triples", "chain", "permute", "batch",
                       "blocks"])
    # three of four in double precision, as in the listed cases
    dtype = rng.choice(["f64", "f64", "f64", "f32"])
    v, o = rng.randint(24, 96), rng.randint(8, 32)
    if kind == "small":
        spec = rng.choice(PATTERNS)
        ext = ",".join("%s=%d" % (ch, _log_int(rng, 4, 24)) for ch in "abcdijk" if ch in spec)
        return {"kind": "contract", "spec": spec, "law": "uniform", "dtype": dtype, "compute": "default",
                "extents": ext}
    if kind == "ccsd":
        return {"kind": rng.choice(["plan", "contract"]), "spec": rng.choice(PATTERNS), "law": "decay",
                "dtype": dtype, "compute": "default", "virtual": v, "occupied": o}
    if kind == "split":
        dtype = rng.choice(["f64", "f32"])
        compute = rng.choice(SPLITS) if dtype == "f64" else "split_bf16x3"
        return {"kind": rng.choice(["plan", "contract"]), "spec": rng.choice(PATTERNS), "law": "decay",
                "dtype": dtype, "compute": compute, "virtual": v, "occupied": o}
    if kind == "grad":
        return {"kind": "grad", "spec": rng.choice(PATTERNS), "law": "decay", "dtype": dtype, "compute": "default",
                "virtual": rng.randint(20, 72), "occupied": rng.randint(6, 24)}
    if kind == "triples":
        return {"kind": "plan", "spec": "abcijk=daij*bcdk", "law": "uniform", "dtype": dtype, "compute": "default",
                "virtual": rng.randint(12, 32), "occupied": rng.randint(6, 16)}
    if kind == "chain":
        return {"kind": "chain", "spec": rng.choice(CHAINS), "law": "uniform", "dtype": dtype, "compute": "default",
                "virtual": v, "occupied": o}
    if kind == "permute":
        spec = rng.choice(PERMUTES)
        case = {"kind": "permute", "spec": spec, "law": "uniform", "dtype": dtype}
        if spec == "ji=ij":
            case["extents"] = "i=%d,j=%d" % (_log_int(rng, 128, 8192), _log_int(rng, 128, 8192))
        elif len(spec) > 9:
            case["virtual"], case["occupied"] = rng.randint(10, 32), rng.randint(6, 16)
        else:
            case["virtual"], case["occupied"] = rng.randint(24, 128), rng.randint(8, 40)
        return case
    if kind == "batch":
        dtype = rng.choice(["f32", "f32", "f64"])
        return {"kind": "batch", "dtype": dtype,
                "compute": rng.choice(["default", "split_bf16x3"]) if dtype == "f32" else "default",
                "problems": _log_int(rng, 8, 48), "problems_seed": rng.randrange(1 << 30),
                "step": rng.choice([8, 8, 1]), "largest": rng.randint(24, 56)}
    n = _log_int(rng, 16, 512)
    rest = max(8, min(4096, int(2 ** 24 / n ** 2)))
    near = [max(8, n + rng.randint(-n // 4, n // 4)) for _ in range(2)]
    return {"kind": "contract", "spec": rng.choice(BATCHED), "law": "uniform", "dtype": dtype, "compute": "default",
            "extents": "b=%d,i=%d,j=%d,k=%d" % (_log_int(rng, 8, rest) if rest > 8 else 8, n, near[0], near[1])}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _values(labels, ext, law, dtype, g):
    """uniform[-1, 1], or normal amplitudes that decay with the gap between
    the two virtual and the two occupied indices."""
    shape = _shape(labels, ext)
    if law == "uniform":
        return torch.rand(shape, dtype=dtype, device="cuda", generator=g).mul_(2.0).sub_(1.0)
    x = torch.randn(shape, dtype=dtype, device="cuda", generator=g)
    for group in ("abcdefgh", "ijklmnop"):
        pos = [p for p, ch in enumerate(labels) if ch in group]
        if len(pos) >= 2:
            line = [torch.arange(shape[p], dtype=dtype, device="cuda").reshape(
                [-1 if q == p else 1 for q in range(len(shape))]) for p in pos[:2]]
            x.mul_(torch.exp(-(line[0] - line[1]).abs() / 8.0))
    return x


def _inputs(case, seed):
    """The input tensors of a case, a list (of lists, for a batch)."""
    g = _generator(seed)
    dtype = _DTYPE[case["dtype"]]
    if case["kind"] == "batch":
        out = []
        for spec, ext in _problems(case):
            c, (a, b) = _operands(spec)
            out.append([_values(t, ext, "uniform", dtype, g) for t in (a, b, c)])
        return out
    ext = _extents(case)
    if case["kind"] == "permute":
        return [_values(case["spec"].split("=")[1], ext, case["law"], dtype, g)]
    c, ops = _operands(case["spec"])
    out = [_values(t, ext, case["law"], dtype, g) for t in ops]
    if case["kind"] == "grad":
        # the previous amplitudes and the upstream gradient
        out += [_values(c, ext, case["law"], dtype, g), _values(c, ext, "uniform", dtype, g)]
    return out


def _arena(like):
    """One zeroed buffer and a view of it shaped like each tensor, each
    starting at a multiple of 64 elements."""
    starts, total = [], 0
    for t in like:
        starts.append(total)
        total += -(-t.numel() // 64) * 64
    flat = torch.zeros(total, dtype=like[0].dtype, device=like[0].device)
    return flat, [flat[s:s + t.numel()].view(t.shape) for s, t in zip(starts, like)]


def prepare(case, seed):
    tensors = _inputs(case, seed)
    state = {"case": case, "tensors": tensors}
    kind = case["kind"]
    if kind == "plan":
        state["plan"] = comet.Plan(case["spec"], tensors[0], tensors[1], compute=case["compute"])
    elif kind == "grad":
        for t in tensors[:3]:
            t.requires_grad_(True)
    elif kind == "batch":
        # the outputs of all problems live in three arenas: C, dA and dB
        arenas = [_arena([ts[i] for ts in tensors]) for i in (2, 0, 1)]
        problems = []
        for p, ((spec, _), (A, B, W)) in enumerate(zip(_problems(case), tensors)):
            sa, sb = _grad_specs(spec)
            C, dA, dB = [views[p] for _, views in arenas]
            problems += [dict(spec=spec, A=A, B=B, C=C), dict(spec=sa, A=W, B=B, C=dA), dict(spec=sb, A=A, B=W, C=dB)]
        state["batch"] = comet.Batch(problems, dtype=_DTYPE[case["dtype"]], compute=case["compute"])
        state["outs"] = [flat for flat, _ in arenas]
    return state


def run(state):
    case, t = state["case"], state["tensors"]
    kind = case["kind"]
    if kind == "plan":
        return state["plan"](t[0], t[1])
    if kind == "contract":
        return comet.contract(case["spec"], t[0], t[1], compute=case["compute"])
    if kind == "grad":
        C = comet.contract_ad(case["spec"], t[0], t[1], t[2], beta=1.0, compute=case["compute"])
        dA, dB, dC0 = torch.autograd.grad(C, t[:3], t[3])
        return C.detach(), dA, dB, dC0
    if kind == "chain":
        return comet.contract_chain(case["spec"], t, compute=case["compute"])
    if kind == "permute":
        return comet.permute(case["spec"], t[0])
    state["batch"]()
    return state["outs"]


# --------------------------------------------------------------------------
# what a pass needs, and its outputs in 64 bits
# --------------------------------------------------------------------------

def _product_work(spec, ext, size):
    c, ops = _operands(spec)
    return {"bytes": size * sum(_count(t, ext) for t in [c] + ops),
            "flops": 2 * _count(set("".join(ops)), ext)}


def work(case):
    size = _SIZE[case["dtype"]]
    kind = case["kind"]
    if kind == "permute":
        return {"bytes": 2 * size * _count(case["spec"].split("=")[1], _extents(case)), "flops": 0}
    if kind == "batch":
        total = {"bytes": 0, "flops": 0}
        for spec, ext in _problems(case):
            w = _product_work(spec, ext, size)
            # forward and two gradients; C written, its gradient read, A and B
            # read and their gradients written
            total["bytes"] += 2 * w["bytes"]
            total["flops"] += 3 * w["flops"]
        return total
    ext = _extents(case)
    w = _product_work(case["spec"], ext, size)
    if kind == "grad":
        # as above, with C0 read and its gradient written
        c = case["spec"].split("=")[0]
        return {"bytes": 2 * w["bytes"] + 2 * size * _count(c, ext), "flops": 3 * w["flops"]}
    if kind == "chain":
        labels = comet.chain_labels(case["spec"])
        w["flops"] = int(comet.chain_plan(case["spec"], [ext[ch] for ch in labels])["flops"])
    return w


def _product64(spec, tensors):
    """A contraction of FP64 tensors as matrix products of reordered operands."""
    c, (a, b) = _operands(spec)
    A, B = tensors
    batch = [ch for ch in c if ch in a and ch in b]
    m = [ch for ch in c if ch in a and ch not in b]
    n = [ch for ch in c if ch in b and ch not in a]
    k = [ch for ch in a if ch in b and ch not in c]
    ext = dict(zip(a + b, tuple(A.shape) + tuple(B.shape)))
    dims = [math.prod(ext[ch] for ch in group) for group in (batch, m, n, k)]
    A = A.permute([a.index(ch) for ch in batch + m + k]).reshape(dims[0], dims[1], dims[3]).contiguous()
    B = B.permute([b.index(ch) for ch in batch + k + n]).reshape(dims[0], dims[3], dims[2]).contiguous()
    C = torch.bmm(A, B).reshape([ext[ch] for ch in batch + m + n])
    order = batch + m + n
    return C.permute([order.index(ch) for ch in c]).contiguous()


def _chain64(spec, tensors):
    c, ops = _operands(spec)
    terms = list(zip(ops, tensors))
    # the library's own grouping is not needed for the value; the one with
    # the fewest operations keeps this quick
    ext = {ch: n for t, x in terms for ch, n in zip(t, x.shape)}
    plan = comet.chain_plan(spec, [ext[ch] for ch in comet.chain_labels(spec)])
    for step in plan["steps"]:
        left, right = terms[step["left"]], terms[step["right"]]
        out = step["spec"].split("=")[0]
        pair = "%s=%s*%s" % (out, left[0], right[0])
        terms.append((out, _product64(pair, (left[1], right[1]))))
    labels, value = terms[-1]
    return value.permute([labels.index(ch) for ch in c]).contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind == "permute":
        out, inp = case["spec"].split("=")
        x = _inputs(case, seed)[0]
        return x.to(torch.float64).permute([inp.index(ch) for ch in out]).contiguous()
    if kind == "batch":
        tensors = [[x.to(torch.float64) for x in ts] for ts in _inputs(case, seed)]
        arenas = [_arena([ts[i] for ts in tensors]) for i in (2, 0, 1)]
        for p, ((spec, _), (A, B, W)) in enumerate(zip(_problems(case), tensors)):
            sa, sb = _grad_specs(spec)
            for (_, views), value in zip(arenas, (_product64(spec, (A, B)), _product64(sa, (W, B)),
                                                  _product64(sb, (A, W)))):
                views[p].copy_(value)
        return [flat for flat, _ in arenas]
    t = [x.to(torch.float64) for x in _inputs(case, seed)]
    if kind == "chain":
        return _chain64(case["spec"], t)
    if kind == "grad":
        A, B, C0, W = t
        sa, sb = _grad_specs(case["spec"])
        return C0 + _product64(case["spec"], (A, B)), _product64(sa, (W, B)), _product64(sb, (A, W)), W.clone()
    return _product64(case["spec"], t)
