"""Performance cases of the particle compressor, at its public entry points.

The ranges they stand for: particle sets of 10^3 (the smallest sets of a
batch) to 2^27 particles (the largest set that one call is benchmarked on),
2-D and 3-D, FP32 and FP64, interleaved and one array per axis, relative
bounds 1e-4 and 1e-3, leaf sizes 8 to 128 (the autotuner's candidates), with
and without the source index of every output slot, references stored as codes
or as coordinates; compression, decompression, batches of many sets, the bit
box reduction on moderate sets, and the entropy stage (sequence layout, Huffman
encoding and decoding).  Inputs are drawn on the GPU: a uniform cube, a
cosmology-shaped set (background and Gaussian halos), a fluid-shaped set (a
jittered lattice in a vortex) and a fusion-shaped 2-D section, all in shuffled
storage order.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2404_02826_amd as bbx

DTYPES = {"float32": torch.float32, "float64": torch.float64}
DEFAULTS = {"dims": 3, "dtype": "float32", "eb": 1e-4, "leaf": 32, "layout": "aos", "perm": False,
            "ref_mode": 0, "reduce": 0}


def listed():
    return [
        # a set of the smallest size, there and back: latency of the two calls
        _case("roundtrip-1000", kind="roundtrip", shape="uniform", n=1000, eb=1e-3),
        # the plain single-set workload, one call at a time
        _case("compress-uniform-65536", kind="compress", shape="uniform", n=65536, eb=1e-3),
        # a served request of middle size, archived as the paper stores it (the
        # references' coordinates) with the source index of every slot, for
        # data that travels with the positions
        _case("compress-cosmology-1000003-exactref", kind="compress", shape="cosmology", n=1000003,
              perm=True, ref_mode=1),
        # an N-body snapshot
        _case("compress-cosmology-2^24", kind="compress", shape="cosmology", n=1 << 24),
        # a fluid time step: the benchmark set
        _case("compress-fluid-2^27", kind="compress", shape="fluid", n=1 << 27),
        # the same kind of step kept in double precision, one array per axis,
        # with a ragged count
        _case("compress-fluid-33554467-f64", kind="compress", shape="fluid", n=33554467,
              dtype="float64", layout="soa"),
        # a 2-D Poincare section, at the size of the paper's data set
        _case("compress-poincare-13077313", kind="compress", shape="poincare", dims=2, n=13077313),
        # the algorithm with the bit box reduction, on a set of moderate size
        _case("compress-reduced-65536", kind="compress", shape="uniform", n=65536, eb=1e-3, reduce=1),
        # reading the fluid time step back
        _case("decompress-fluid-2^27", kind="decompress", shape="fluid", n=1 << 27),
        # many independent sets in one job
        _case("batch-256", kind="batch", shape="mixed", sets=256, n=1000000, mix=5),
        # archiving a snapshot: sequence layout with its reorderings, Huffman coded
        _case("encode-cosmology-2^24", kind="encode", shape="cosmology", n=1 << 24, ref_mode=1),
        # reading the archive's bytes back
        _case("decode-cosmology-2^24", kind="decode", shape="cosmology", n=1 << 24, ref_mode=1),
    ]


def draw(rng):
    kind = rng.choice(["compress"] * 6 + ["decompress"] * 3 + ["roundtrip", "batch", "encode", "decode"])
    shape = rng.choice(["uniform", "cosmology", "fluid", "poincare"])
    c = dict(kind=kind, shape=shape, dims=2 if shape == "poincare" else 3,
             dtype=rng.choice(["float32", "float32", "float64"]), eb=rng.choice([1e-4, 1e-3]),
             leaf=rng.choice([8, 16, 32, 32, 32, 64, 128]))
    if kind == "batch":
        return _case(None, **dict(c, shape="mixed", dims=3, sets=rng.randint(8, 256),
                                  n=int(10 ** rng.uniform(4, 6)), mix=rng.randint(0, 1 << 30)))
    if kind in ("encode", "decode"):
        return _case(None, **dict(c, n=_size(rng, 1e4, 1 << 24), ref_mode=1))
    c["layout"] = rng.choice(["aos", "aos", "soa"])
    c["perm"] = rng.random() < 0.25
    c["reduce"] = 1 if rng.random() < 0.15 else 0
    if not c["reduce"]:
        c["ref_mode"] = 1 if rng.random() < 0.25 else 0
    most = 1 << 27 if c["dtype"] == "float32" else 1 << 26
    if c["reduce"]:  # its loop takes as long as the set has leaves
        most = min(65536, 2048 * c["leaf"])
    return _case(None, **dict(c, n=_size(rng, 1e3, 65536 if kind == "roundtrip" else most)))


def _case(name, **kw):
    c = dict(DEFAULTS, **kw)
    if name:
        c["name"] = name
    return c


def _size(rng, lo, hi):
    """Log-uniform; three in four odd, the others a multiple of 1,024 or the largest power of two below."""
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    how = rng.random()
    if how < 0.75:
        return min(n | 1, int(hi) - 1)
    return max(1024, n // 1024 * 1024) if how < 0.9 else 1 << (n.bit_length() - 1)


# ---------------------------------------------------------------- inputs

def _positions(shape, n, dims, dtype, gen):
    """Positions (n, dims) on the GPU in shuffled order."""
    dev = gen.device
    two_pi = 2.0 * math.pi

    def rand(*size):
        return torch.rand(*size, generator=gen, device=dev, dtype=torch.float64)

    if shape == "uniform":
        return torch.rand(n, dims, generator=gen, device=dev, dtype=dtype)
    if shape == "cosmology":
        box, halos = 256.0, 2000
        centres = rand(halos, dims) * box
        radii = torch.exp(math.log(0.5) + 0.7 * torch.randn(halos, generator=gen, device=dev, dtype=torch.float64))
        member = torch.randint(0, halos, (n,), generator=gen, device=dev)
        p = torch.randn(n, dims, generator=gen, device=dev, dtype=torch.float64)
        p = p * radii[member][:, None] + centres[member]
        p = torch.where(rand(n, 1) < 0.3, rand(n, dims) * box, torch.remainder(p, box)).to(dtype)
        top = torch.nextafter(torch.tensor(box, dtype=dtype), torch.tensor(0.0, dtype=dtype))
        return p.clamp_(max=float(top))
    if shape == "fluid":  # a random n of the cells of a cube-like lattice
        if n & (n - 1) == 0:
            k = n.bit_length() - 1
            nx, ny, nz = (1 << (k // 3 + (i < k % 3)) for i in range(3))
        else:
            nx = ny = nz = math.ceil(n ** (1.0 / 3.0))
            while nx ** 3 < n:
                nx, ny, nz = nx + 1, ny + 1, nz + 1
        cell = torch.randperm(nx * ny * nz, generator=gen, device=dev)[:n]
        p = torch.empty(n, 3, device=dev, dtype=torch.float64)
        p[:, 0] = cell % nx
        p[:, 1] = (cell // nx) % ny
        p[:, 2] = cell // (nx * ny)
        del cell
        p += rand(n, 3) * 0.6 + 0.2
        move = torch.stack([torch.sin(two_pi * p[:, 1] / ny), torch.sin(two_pi * p[:, 2] / nz),
                            torch.sin(two_pi * p[:, 0] / nx)], dim=1)
        return p.add_(move, alpha=2.0).to(dtype)
    if shape == "poincare":  # flux surfaces, three island chains, an edge band
        a = 0.6
        u = rand(n)
        surf = (0.95 * a * torch.sqrt(rand(600)))[torch.randint(0, 600, (n,), generator=gen, device=dev)]
        chain = torch.tensor([[0.55 * a, 3, 0.030 * a], [0.75 * a, 4, 0.025 * a], [0.90 * a, 5, 0.020 * a]],
                             device=dev, dtype=torch.float64)
        c = chain[torch.randint(0, 3, (n,), generator=gen, device=dev)]
        t, size = rand(n) * two_pi, rand(n) * 0.8 + 0.2
        rho_i = c[:, 0] + c[:, 2] * size * torch.sin(t)
        th_i = two_pi * (torch.floor(rand(n) * c[:, 1]) + 0.25) / c[:, 1] + c[:, 2] / c[:, 0] * 2.0 * size * torch.cos(t)
        rho = torch.where(u < 0.7, surf, torch.where(u < 0.9, rho_i, a * (rand(n) * 0.08 + 0.96)))
        th = torch.where((u >= 0.7) & (u < 0.9), th_i, rand(n) * two_pi)
        p = torch.stack([1.7 + rho * torch.cos(th + 0.35 * torch.sin(th)) + 0.1 * rho * torch.sin(th) ** 2,
                         1.7 * rho * torch.sin(th)], dim=1)
        return (p + 1e-4 * torch.randn(n, 2, generator=gen, device=dev, dtype=torch.float64)).to(dtype)
    raise ValueError(shape)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _input(case, seed):
    p = _positions(case["shape"], case["n"], case["dims"], DTYPES[case["dtype"]], _gen(seed))
    return p.t().contiguous() if case["layout"] == "soa" else p.contiguous()


def _batch_sizes(case):
    """(size, shape, bound) of each set: sizes log-uniform from 10^3 to the case's n."""
    rng = random.Random(case["mix"])
    return [(int(round(10.0 ** rng.uniform(3.0, math.log10(case["n"])))), rng.choice(["uniform", "cosmology"]),
             rng.choice([1e-3, 1e-4])) for _ in range(case["sets"])]


def _compressor(case):
    return bbx.Compressor(case["n"], case["dims"], DTYPES[case["dtype"]], leaf_size=case["leaf"],
                          layout=case["layout"], want_perm=case["perm"], ref_mode=case["ref_mode"],
                          reduce=case["reduce"])


# ---------------------------------------------------------------- the calls

def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        gen = _gen(seed)
        dtype = DTYPES[case["dtype"]]
        batch = bbx.BatchCompressor(
            [{"pos": _positions(shape, n, 3, dtype, gen), "eb": eb, "leaf_size": case["leaf"]}
             for n, shape, eb in _batch_sizes(case)])
        batch.out.zero_()
        return {"kind": kind, "batch": batch}
    pos = _input(case, seed)
    st = {"kind": kind, "eb": case["eb"], "comp": _compressor(case)}
    st["comp"].out.zero_()  # the bytes behind the stream stay as they are
    if kind == "compress":
        return dict(st, pos=pos)
    stream = st["comp"](pos, case["eb"]).clone()
    header = stream[:128].cpu().numpy().tobytes()
    if kind == "roundtrip":
        return dict(st, pos=pos, dec=bbx.Decompressor(header, case["layout"]))
    del st["comp"]
    if kind == "decompress":
        return dict(st, stream=stream, dec=bbx.Decompressor(header, case["layout"]))
    # the archive's buffer: no archive is larger than the positions
    archive = torch.zeros(pos.numel() * pos.element_size(), dtype=torch.uint8, device="cuda")
    if kind == "encode":
        return dict(st, stream=stream, archive=archive)
    return dict(st, packed=bbx.huffman_encode(bbx.export_sequences_reordered(stream)[0]), archive=archive)


def run(state):
    kind = state["kind"]
    if kind in ("compress", "roundtrip"):
        comp = state["comp"]
        stream = comp(state["pos"], state["eb"])
        out = [comp.out, stream.numel()]  # the whole buffer, which has the same size for any input
        if kind == "roundtrip":
            out.append(state["dec"](stream))
        if comp.perm is not None:
            out.append(comp.perm)
        return out
    if kind == "decompress":
        return [state["dec"](state["stream"])]
    if kind == "batch":
        batch = state["batch"]
        batch()
        return [batch.out, batch.d_size, batch.d_status]
    archive = state["archive"]
    if kind == "encode":
        layout, order = bbx.export_sequences_reordered(state["stream"])
        data = bbx.huffman_encode(layout)
        archive[:data.numel()].copy_(data)
        return [archive, data.numel(), order]
    data = bbx.huffman_decode(state["packed"])
    archive[:data.numel()].copy_(data)
    return [archive, data.numel()]


def _stream_bytes(n, dims, dtype, eb, leaf, ref_mode, seq_bits=0):
    """About the stream's size: leaves of `leaf` particles that share the box evenly."""
    leaves = max(1, 2 ** math.ceil(math.log2(max(1.0, n / leaf))))
    span = 0.5 / eb
    width = max(1.0, math.log2(span / leaves ** (1.0 / dims)) + 1.0)
    code = 8 * DTYPES[dtype].itemsize if ref_mode else math.log2(span)
    return 128 + (dims * ((n - leaves) * width + leaves * (5 + code)) + seq_bits * leaves) / 8


def work(case):
    """Inputs read once and outputs written once; operations: the FP64
    arithmetic of (de)quantization, five a coordinate."""
    n, dims = case["n"], case["dims"]
    item = DTYPES[case["dtype"]].itemsize
    if case["kind"] == "batch":
        sets = _batch_sizes(case)
        total = sum(n for n, _, _ in sets)
        return {"bytes": sum(n * 3 * item + _stream_bytes(n, 3, case["dtype"], eb, case["leaf"], 0)
                             for n, _, eb in sets), "flops": 15.0 * total}
    stream = _stream_bytes(n, dims, case["dtype"], case["eb"], case["leaf"], case["ref_mode"])
    layout = _stream_bytes(n, dims, case["dtype"], case["eb"], case["leaf"], 1, 32)
    if case["kind"] == "encode":
        return {"bytes": stream + 2 * layout, "flops": 0.0}
    if case["kind"] == "decode":
        return {"bytes": 2 * layout, "flops": 0.0}
    moved = n * dims * item + stream
    if case["perm"] and case["kind"] != "decompress":
        moved += 4 * n
    twice = 2 if case["kind"] == "roundtrip" else 1
    return {"bytes": twice * moved, "flops": 5.0 * twice * n * dims}


# ---------------------------------------------------------------- expected values

def exact(case, seed):
    """Decompressed positions in 64 bits (streams, indices and bytes have no such value)."""
    kind = case["kind"]
    if kind not in ("decompress", "roundtrip") or case["reduce"] or case["n"] > 1 << 20:
        return None
    pos = _input(case, seed)
    x = (pos.t() if case["layout"] == "soa" else pos).cpu().numpy()
    want = _reconstruct(x, case["eb"], case["leaf"], case["ref_mode"])
    want = np.ascontiguousarray(want.T) if case["layout"] == "soa" else want
    if kind == "decompress":
        return [want]
    return [None, None, want] + ([None] if case["perm"] else [])


def _reconstruct(x, eb, leaf, ref_mode):
    """Quantize, split at the medians along the axes in turn until at most
    `leaf` particles, and give each particle its bin's centre: leaves depth
    first, the member nearest the box centre first, then by input index."""
    n, dims = x.shape
    v = x.astype(np.float64)
    lo, hi = v.min(axis=0), v.max(axis=0)
    bound = eb * float((hi - lo).max())
    most = float(np.abs(v).max()) + bound
    guard = math.ldexp(most, -48)
    if x.dtype == np.float32:
        guard += max(math.ldexp(1.0, math.frexp(most)[1] - 25), math.ldexp(1.0, -150))
    width = 2.0 * (bound - guard)
    q = np.floor((v - lo) * (1.0 / width) + 0.5).astype(np.int64)
    order, node = np.arange(n), np.zeros(n, np.int64)  # members by node, then by index
    starts, sizes, depth = np.array([0]), np.array([n]), 0
    while sizes.max() > leaf:
        by = np.lexsort((order, q[order, depth % dims], node))
        rank = np.empty(n, np.int64)
        rank[by] = np.arange(n) - starts[node[by]]
        split = sizes > leaf
        right = split[node] & (rank >= (sizes // 2)[node])
        order = order[np.lexsort((order, right, node))]
        left = np.where(split, sizes // 2, sizes)
        sizes = np.stack([left, sizes - left], axis=1).ravel()
        sizes = sizes[sizes > 0]
        starts = np.concatenate([[0], np.cumsum(sizes)[:-1]])
        node = np.repeat(np.arange(len(sizes)), sizes)
        depth += 1
    c = q[order]
    box = np.minimum.reduceat(c, starts) + np.maximum.reduceat(c, starts)
    far = ((2 * c - box[node]) ** 2).sum(axis=1)
    ref = np.lexsort((order, far, node))[starts]
    first = np.zeros(n, bool)
    first[ref] = True
    order = order[np.lexsort((order, ~first, node))]
    out = lo + q[order] * width
    if ref_mode:
        out[starts] = v[order[starts]]
    return out
