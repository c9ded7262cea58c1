"""What the performance of this library is measured on: the work that a prover (and the verifier of its paths)
has it do, through the public entry points of the package.

    quantise     fp16 activations of a forward pass -> int16, per-tensor scales on the device
    commit       one tensor -> one commitment
    commit_batch several tensors (the weight matrices of a layer) -> one commitment each, in one call
    entries_tree Terkle tree whose leaves are the entries of one tensor
    build        the activations of a forward pass: quantised, one commitment per tensor, the tree over them
    open         openings of such a tree down to tensor entries
    verify       paths of such a tree checked against its root
    prove_entry  openings of an entries tree and their verification, as served for one layer
    interpolate  the coefficient route: values on the grid -> monomial coefficients

Values are what the path meets in earnest: activations N(0, 1) in fp16, quantised to int16 by their largest
magnitude; weights int8 uniform in [-127, 127].  The public parameters come from the fixed test trapdoor; everything
else comes from the seed.  All results are exact: field elements, group elements and quantised integers.
"""
import random

import numpy as np
import torch

import paper_2602_12630_amd as T
import tc_inputs

R_MODULUS = 0x73EDA753299D7D483339D80809A1D80553BDA402FFFE5BFEFFFFFFFF00000001
NODE = tc_inputs.NODE_SHAPE
# A group addition in affine form with a shared inversion: five products and a square of Fp, 300 limb multiply-adds each
# at 32-bit limbs; an Fr product has 136 of them.  One multiply-add counts as two operations.
OPS_PER_ADDITION = 2 * 6 * 300
OPS_PER_FR_PRODUCT = 2 * 136
POINT_BYTES = 96
FR_BYTES = 32


def listed():
    return [
        # the smallest call: the commitment of a 1024-entry int8 tensor of order 3; launches and depth are all of it
        {"name": "commit_tiny_i8", "kind": "commit", "shape": "4x16x16", "dtype": "i8"},
        # one residual-stream activation, 512 tokens x 4096
        {"name": "commit_activation_i16", "kind": "commit", "shape": "512x4096", "dtype": "i16"},
        # an MLP intermediate of a prompt whose length is no round number
        {"name": "commit_mlp_ragged_i16", "kind": "commit", "shape": "487x11008", "dtype": "i16"},
        # the attention weights of a layer, Wq Wk Wv Wo, committed once when a model is registered
        {"name": "commit_weights_i8", "kind": "commit_batch", "shape": "4096x4096", "dtype": "i8", "count": 4},
        # scales and values of the 96 activations of a LLaMA2-7B-shaped forward
        {"name": "quantise_forward", "kind": "quantise", "layers": 32, "tokens": 512, "hidden": 4096, "mlp": 11008},
        # entries tree over one activation: 139 813 nodes in six levels
        {"name": "entries_tree_activation", "kind": "entries_tree", "shape": "512x4096", "dtype": "i16"},
        # the headline: a LLaMA2-7B-shaped forward of 512 tokens quantised, committed and put under its tree
        {"name": "build_forward", "kind": "build", "layers": 32, "tokens": 512, "hidden": 4096, "mlp": 11008},
        # the same model on a short prompt: 96 small tensors of ragged length
        {"name": "build_forward_19_tokens", "kind": "build", "layers": 32, "tokens": 19, "hidden": 4096, "mlp": 11008},
        # 64 random openings of the headline's tree, down to tensor entries
        {"name": "open_forward_64", "kind": "open", "layers": 32, "tokens": 512, "hidden": 4096, "mlp": 11008, "paths": 64},
        # 64 paths of a forward's tree verified in one batch
        {"name": "verify_forward_64", "kind": "verify", "layers": 32, "tokens": 64, "hidden": 4096, "mlp": 11008, "paths": 64},
        # eight entries of one activation opened and verified
        {"name": "prove_entry_8", "kind": "prove_entry", "shape": "512x4096", "dtype": "i16", "paths": 8},
        # the coefficient array of one activation
        {"name": "interpolate_activation", "kind": "interpolate", "shape": "512x4096", "dtype": "i16"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["commit", "commit", "commit_batch", "quantise", "entries_tree", "build", "build", "open", "verify",
                       "prove_entry", "interpolate"])
    case = {"kind": kind}
    if kind == "commit":
        total = _log_int(rng, 1024, 487 * 11008)
        rows = _log_int(rng, 1, min(1024, total // 2))
        case["shape"] = "%dx%d" % (rows, max(2, total // rows))
        case["dtype"] = rng.choice(["i8", "i16"])
    elif kind == "commit_batch":
        case["count"] = rng.randint(2, 8)
        rows = _log_int(rng, 16, 4096)
        case["shape"] = "%dx%d" % (rows, min(_log_int(rng, 64, 11008), 4 * 4096 * 4096 // (case["count"] * rows)))
        case["dtype"] = rng.choice(["i8", "i8", "i16"])
    elif kind in ("quantise", "build", "open", "verify"):
        case["layers"] = rng.randint(1, 32)
        case["tokens"] = _log_int(rng, 2, 512 if kind in ("quantise", "build") else 256)
        case["hidden"] = rng.choice([1024, 2048, 4096, _log_int(rng, 256, 4096)])
        case["mlp"] = case["hidden"] * 43 // 16
        if kind in ("open", "verify"):
            case["paths"] = _log_int(rng, 1, 64)
    else:
        total = _log_int(rng, 1024, 512 * 4096)
        rows = _log_int(rng, 8, 512)
        case["shape"] = "%dx%d" % (rows, max(8, min(4096, total // rows)))
        case["dtype"] = rng.choice(["i8", "i16", "i16"])
        if kind == "prove_entry":
            case["paths"] = _log_int(rng, 1, 32)
    return case


# ---- what the cases are made of ----------------------------------------------------------------------------------
def _shape(case):
    return tuple(int(d) for d in case["shape"].split("x"))


def _forward_shapes(case):
    """per layer: residual output, attention output, MLP intermediate"""
    t, h, f = case["tokens"], case["hidden"], case["mlp"]
    return [(t, h), (t, h), (t, f)]


def _size(shape):
    n = 1
    for d in shape:
        n *= d
    return n


class State:
    """What a program holds between calls: a context, public parameters, buffers, trees; given back with the object."""

    def __init__(self, case):
        self.case = case
        self.held = []
        self.ctx = T.Context(torch.cuda.current_device(), torch.cuda.current_stream().cuda_stream)
        self.tau = tc_inputs.trapdoor_bytes()

    def srs(self, shape, flags=0):
        s = self.ctx.setup_from_trapdoor(self.tau, shape, flags)
        self.held.append(s)
        return s

    def node_srs(self):
        return self.srs(NODE, T.TC_SRS_SUFFIX | T.TC_SRS_FIXED_BASE)

    def close(self):
        for h in reversed(self.held):
            h.close()
        self.held = []
        if self.ctx is not None:
            self.ctx.close()
            self.ctx = None

    def __del__(self):
        self.close()


def _activation(n, gen):
    return torch.randn(n, generator=gen, device="cuda", dtype=torch.float32).to(torch.float16)


def _scalars(st, n, dtype, gen):
    if dtype == "i8":
        return torch.randint(-127, 128, (n,), generator=gen, device="cuda", dtype=torch.int8)
    x, q = _activation(n, gen), torch.empty(n, dtype=torch.int16, device="cuda")
    scale = torch.zeros(1, dtype=torch.float32, device="cuda")
    st.ctx.quant_scale(x, n, scale)
    st.ctx.encode_tensor_scaled(x, T.TC_F16, n, scale, q)
    st.ctx.sync()
    return q


def _dtype(case):
    return T.TC_I8 if case["dtype"] == "i8" else T.TC_I16


def _forward_inputs(st, case, gen):
    st.shapes = _forward_shapes(case) * case["layers"]
    st.xs = [_activation(_size(s), gen) for s in st.shapes]
    st.ns = [x.numel() for x in st.xs]
    # the quantised tensors side by side in one buffer, each on a boundary of 256 bytes
    first = [0]
    for n in st.ns:
        first.append(first[-1] + (n + 127) // 128 * 128)
    st.values = torch.zeros(first[-1], dtype=torch.int16, device="cuda")
    st.qs = [st.values[i:i + n] for i, n in zip(first, st.ns)]
    st.scales = torch.zeros(len(st.xs), dtype=torch.float32, device="cuda")
    st.grid = (case["layers"], 3)


def _forward_parameters(st, case):
    st.nodes = st.node_srs()
    by_shape = {s: st.srs(s, T.TC_SRS_SUFFIX | T.TC_SRS_OPEN_TABLE) for s in set(_forward_shapes(case))}
    st.leaf_srs = [by_shape[s] for s in st.shapes]
    st.dtypes = [T.TC_I16] * len(st.shapes)


def _forward_tree(st):
    st.ctx.encode_batch_scaled(st.xs, st.ns, st.scales, st.qs)
    return st.ctx.terkle_build_tensors(st.nodes, st.leaf_srs, st.qs, st.dtypes, st.grid, NODE)


def _forward_positions(st, case, seed):
    rng = random.Random(seed)
    st.leaves = [(rng.randrange(case["layers"]), rng.randrange(3)) for _ in range(case["paths"])]
    st.inners = [tuple(rng.randrange(d) for d in st.shapes[3 * l[0] + l[1]]) for l in st.leaves]


def _field_bytes(values):
    return [(int(v) % R_MODULUS).to_bytes(32, "little") for v in values]


def prepare(case, seed):
    kind = case["kind"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    st = State(case)
    if kind in ("commit", "commit_batch"):
        shape = _shape(case)
        st.p = st.srs(shape)
        st.ts = [_scalars(st, _size(shape), case["dtype"], gen) for _ in range(case.get("count", 1))]
    elif kind == "quantise":
        _forward_inputs(st, case, gen)
    elif kind == "entries_tree":
        st.nodes = st.node_srs()
        st.t = _scalars(st, _size(_shape(case)), case["dtype"], gen)
    elif kind in ("build", "open", "verify"):
        _forward_inputs(st, case, gen)
        _forward_parameters(st, case)
        if kind != "build":
            st.tree = _forward_tree(st)
            st.held.append(st.tree)
            _forward_positions(st, case, seed)
        if kind == "verify":
            st.vk = st.ctx.vk_from_trapdoor(st.tau)
            st.proofs = st.tree.open_batch(st.leaves, st.inners)
            st.paths = [st.tree.path(l, i) for l, i in zip(st.leaves, st.inners)]
            st.roots = [st.tree.root] * len(st.paths)
            flat = [st.qs[3 * l[0] + l[1]][i[0] * st.shapes[3 * l[0] + l[1]][1] + i[1]] for l, i in zip(st.leaves, st.inners)]
            values = torch.stack(flat).cpu().tolist()
            rng = random.Random(seed + 1)          # now and then a verifier meets a value that was not committed
            st.opened = _field_bytes([v + (rng.random() < 0.1) for v in values])
    elif kind == "prove_entry":
        shape = _shape(case)
        st.nodes = st.node_srs()
        st.t = _scalars(st, _size(shape), case["dtype"], gen)
        st.tree = st.ctx.terkle_build_entries(st.nodes, st.t, _dtype(case), shape, NODE)
        st.held.append(st.tree)
        st.vk = st.ctx.vk_from_trapdoor(st.tau)
        rng = random.Random(seed)
        st.leaves = [tuple(rng.randrange(d) for d in shape) for _ in range(case["paths"])]
        st.paths = [st.tree.path(l) for l in st.leaves]
        st.roots = [st.tree.root] * len(st.paths)
        st.opened = _field_bytes(st.t[torch.tensor([l[0] * shape[1] + l[1] for l in st.leaves], device="cuda")].cpu().tolist())
    elif kind == "interpolate":
        n = _size(_shape(case))
        st.t = _scalars(st, n, case["dtype"], gen)
        st.out = torch.empty((n, 8), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    return st


def _bytes(parts):
    return np.frombuffer(b"".join(parts), dtype=np.uint8)


def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "commit":
        return _bytes([st.ctx.commit(st.p, st.ts[0], _dtype(case))])
    if kind == "commit_batch":
        k = case["count"]
        return _bytes(st.ctx.commit_batch([st.p] * k, st.ts, [_dtype(case)] * k))
    if kind == "quantise":
        st.ctx.encode_batch_scaled(st.xs, st.ns, st.scales, st.qs)
        return {"scales": st.scales, "values": st.values}
    if kind == "entries_tree":
        # the root binds every node: any other node changes phi of it, and with it the commitments above
        tree = st.ctx.terkle_build_entries(st.nodes, st.t, _dtype(case), _shape(case), NODE)
        root = tree.root
        tree.close()
        return _bytes([root])
    if kind == "build":
        tree = _forward_tree(st)
        root = tree.root
        tree.close()
        return {"root": _bytes([root]), "scales": st.scales, "values": st.values}
    if kind == "open":
        return _bytes(st.tree.open_batch(st.leaves, st.inners))
    if kind == "verify":
        return np.array(st.ctx.verify_paths_batch(st.vk, st.paths, st.roots, st.opened, st.proofs), dtype=np.uint8)
    if kind == "prove_entry":
        proofs = st.tree.open_batch(st.leaves)
        ok = st.ctx.verify_paths_batch(st.vk, st.paths, st.roots, st.opened, proofs)
        return {"proofs": _bytes(proofs), "ok": np.array(ok, dtype=np.uint8)}
    if kind == "interpolate":
        st.ctx.interpolate(_shape(case), st.t, _dtype(case), st.out)
        return st.out
    raise ValueError(kind)


def _tree_nodes(grid):
    nodes, grid = [], tuple(grid)
    while True:
        grid = tuple((g + b - 1) // b for g, b in zip(grid, NODE))
        nodes.append(_size(grid))
        if nodes[-1] == 1:
            return nodes


def work(case):
    kind = case["kind"]
    if kind in ("commit", "commit_batch"):
        # every scalar and every point of the SRS once, an addition per entry
        n, k = _size(_shape(case)), case.get("count", 1)
        esz = 1 if case["dtype"] == "i8" else 2
        return {"bytes": n * (POINT_BYTES + k * esz), "flops": n * k * OPS_PER_ADDITION}
    if kind == "interpolate":
        # Newton form: d (d - 1) / 2 products for the differences of a line and as many for the expansion
        shape = _shape(case)
        n = _size(shape)
        return {"bytes": n * (FR_BYTES + (1 if case["dtype"] == "i8" else 2)),
                "flops": sum(n * (d - 1) for d in shape) * OPS_PER_FR_PRODUCT}
    if kind == "entries_tree":
        # an addition per entry at the bottom; above, sixteen 16-bit windows of every child's image in Fr
        shape = _shape(case)
        n, nodes = _size(shape), _tree_nodes(shape)
        upper = 16 * sum(nodes[:-1])
        return {"bytes": n * (1 if case["dtype"] == "i8" else 2) + sum(nodes) * (POINT_BYTES + FR_BYTES),
                "flops": (n + upper) * OPS_PER_ADDITION}
    if kind == "prove_entry":
        # per path and level: 20 quotient values of sixteen windows each to open; two half-length chains of doublings
        # (seven products each) per proof element to verify
        steps = case["paths"] * len(_tree_nodes(_shape(case)))
        return {"bytes": steps * 4 * POINT_BYTES, "flops": steps * (20 * 16 * OPS_PER_ADDITION + 4 * 127 * 7 * 600)}
    # the kinds over a forward pass
    sizes = [_size(s) for s in _forward_shapes(case)] * case["layers"]
    n = sum(sizes)
    srs_points = sum(_size(s) for s in set(_forward_shapes(case)))
    if kind == "quantise":
        return {"bytes": 4 * n, "flops": 2 * n}
    if kind == "build":
        return {"bytes": 4 * n + srs_points * POINT_BYTES, "flops": n * OPS_PER_ADDITION}
    if kind == "open":
        # first quotient of every path: the rows of its tensor, two 8-bit digits per entry (a tensor may serve several
        # paths; at most one of each there is)
        tensors = min(case["paths"], len(sizes))
        entries = tensors * n // len(sizes)
        return {"bytes": 2 * entries + srs_points * POINT_BYTES, "flops": 2 * entries * OPS_PER_ADDITION}
    steps = case["paths"] * (1 + len(_tree_nodes((case["layers"], 3))))
    return {"bytes": steps * 4 * POINT_BYTES, "flops": steps * 4 * 127 * 7 * 600}


def tolerance(case):
    return "exact"
