"""Performance cases of libmdt: what a user's program has it do, through the Python binding's public calls.

Every case moves seeded random bytes that are resident in device memory; irregular layouts come with the case.  A pass
of most kinds is one exchange: pack from a source array into packed buffers, then unpack those into a destination array
of the same layout.
Kinds (each draws its sizes from the range in ``draw``):

vector   strided blocks of a basic type, one pack and one unpack enqueued (the latency-bound end)
faces    halo faces of an n^3 float64 array: one launch per face ("plain"), one batch per direction as created
         ("batch"), or one autotuned batch per direction ("tuned")
records  particle records struct {int32, float64[k], char[5]}
blocks   hindexed layout of short byte blocks in permuted order
ranges   a records or blocks transfer cut in byte ranges of a budget, one enqueue per range (pipelined sends)
rows     interior of a 2-D float64 matrix (long runs, bandwidth-bound)
darray   one rank's block-cyclic share of an n^3 float64 array
mix      a batch of pack requests of uneven sizes over vectors, halo faces and an hindexed layout
copy     typed copies with no packed buffer: periodic halo self-exchange, or padded records to tight ones
flatten  a type's iovec segments written to device memory
serving  a burst of requests through the server: packs, then unpacks of what they packed
"""
import math

import numpy as np
import torch

from paper_2402_12274_amd import inputs, mdt

MiB = 1 << 20
DTYPES = {"DOUBLE": 8, "FLOAT": 4, "INT16": 2, "BYTE": 1}


def listed():
    return [
        # one small strided vector: launch and host latency
        {"name": "vector_small", "kind": "vector", "n": 1024, "bl": 1, "stride": 2, "dtype": "DOUBLE"},
        # a small subdomain's exchange, a launch per face
        {"name": "faces_130_plain", "kind": "faces", "n": 130, "w1": 2, "w2": 0, "how": "plain"},
        # the halo step of a large domain, tuned once and run for many steps
        {"name": "faces_512_tuned", "kind": "faces", "n": 512, "w1": 1, "w2": 4, "how": "tuned"},
        # all particles of a large rank
        {"name": "records_4m", "kind": "records", "count": 4_000_000, "k": 3},
        # unstructured mesh or sparse exchange: short blocks anywhere in 2 GiB
        {"name": "blocks_1m", "kind": "blocks", "n": 1_000_000, "mean": 24, "span": 1 << 31, "layout_seed": 1},
        # a message sent in 1 MiB pieces
        {"name": "ranges_1mib", "kind": "ranges", "layout": "records", "count": 1_000_000, "k": 3, "budget": MiB},
        # a matrix without its border
        {"name": "rows_8192", "kind": "rows", "rows": 8192, "cols": 8192, "border": 64},
        # redistribution of a block-cyclic array
        {"name": "darray_512", "kind": "darray", "n": 512, "block": 16, "procs": 2, "rank": 5},
        # many requests of mixed types and sizes in one launch, the batch as created
        {"name": "mix_4096", "kind": "mix", "requests": 4096, "hi": 16 * MiB, "layout_seed": 3},
        # ghost layers of a periodic domain on one GPU
        {"name": "copy_halo_512", "kind": "copy", "layout": "halo", "n": 512},
        # segment list of an irregular type for a kernel or a NIC to read
        {"name": "flatten_1m", "kind": "flatten", "layout": "blocks", "n": 1_000_000, "mean": 24, "span": 1 << 31,
         "layout_seed": 2},
        # requests of resident types as a serving loop gets them
        {"name": "serving_64", "kind": "serving", "requests": 64, "ntypes": 32, "layout_seed": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["vector", "faces", "records", "blocks", "ranges", "rows", "darray", "mix", "copy", "flatten",
                       "serving"])
    if kind == "vector":
        n, bl = _log(rng, 64, 4_000_000), rng.randint(1, 16)
        return {"kind": kind, "n": n, "bl": bl, "stride": bl + rng.randint(1, 48), "dtype": rng.choice(sorted(DTYPES))}
    if kind == "faces":
        return {"kind": kind, "n": _log(rng, 40, 512), "w1": rng.randint(1, 4), "w2": rng.choice([0, 5, 6]),
                "how": rng.choice(["plain", "batch", "tuned"])}
    if kind == "records":
        return {"kind": kind, "count": _log(rng, 1000, 4_000_000), "k": rng.randint(1, 6)}
    if kind == "blocks":
        return _draw_blocks(rng, {"kind": kind})
    if kind == "ranges":
        if rng.random() < 0.5:
            case = {"kind": kind, "layout": "records", "count": _log(rng, 20_000, 4_000_000), "k": rng.randint(1, 6)}
            total = case["count"] * (9 + 8 * case["k"])
        else:
            case = _draw_blocks(rng, {"kind": kind, "layout": "blocks"})
            total = case["n"] * case["mean"]
        case["budget"] = max(_log(rng, 64 << 10, 4 * MiB), total // 100) + rng.randint(0, 15)
        return case
    if kind == "rows":
        return {"kind": kind, "rows": _log(rng, 100, 8192), "cols": _log(rng, 200, 8192), "border": rng.randint(1, 48)}
    if kind == "darray":
        # the corner ranks: their shares are ragged in every dimension or in none
        return {"kind": kind, "n": _log(rng, 64, 512), "block": rng.randint(1, 32), "procs": 2,
                "rank": rng.choice([0, 7])}
    if kind == "mix":
        return {"kind": kind, "requests": _log(rng, 16, 2048), "hi": _log(rng, 64 << 10, 16 * MiB),
                "layout_seed": rng.randrange(1 << 30)}
    if kind == "copy":
        if rng.random() < 0.5:
            return {"kind": kind, "layout": "halo", "n": _log(rng, 40, 512)}
        return {"kind": kind, "layout": "records", "count": _log(rng, 1000, 4_000_000), "k": rng.randint(1, 6)}
    if kind == "flatten":
        if rng.random() < 0.5:
            return _draw_blocks(rng, {"kind": kind, "layout": "blocks"})
        return {"kind": kind, "layout": "face", "n": _log(rng, 40, 512), "w": rng.randint(1, 4)}
    return {"kind": kind, "requests": _log(rng, 8, 128), "ntypes": 4 * rng.randint(2, 10),
            "layout_seed": rng.randrange(1 << 30)}


def _draw_blocks(rng, case):
    case["n"], case["mean"] = _log(rng, 4096, 1_000_000), rng.randint(6, 64)
    case["span"] = case["n"] * rng.randint(300, 2100)
    case["layout_seed"] = rng.randrange(1 << 30)
    return case


# ---------------------------------------------------------------------------
# layouts: specs, and (for exact) the byte offsets of a typemap in map order


def _random(nbytes, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=g)


def _faces(case):
    widths = [w for w in (case["w1"], case["w2"]) if w]
    return [(w, dim, side) for w in widths for dim in (0, 1, 2) for side in ("lo", "hi")]


def _blocks(case):
    return inputs.hindexed_blocks(nblocks=case["n"], span=case["span"], mean=float(case["mean"]),
                                  seed=case["layout_seed"])


def _record(k):
    return ("struct", [1, k, 5], [0, 8, 8 + 8 * k], [("basic", "INT32"), inputs.DOUBLE, ("basic", "CHAR")])


def _tight_record(k):
    return ("struct", [4, 8 * k, 5], [0, 4, 4 + 8 * k], [inputs.BYTE] * 3)


def _ghost(n, w, dim, side):
    sub, start = [n - 2 * w] * 3, [w] * 3
    sub[dim], start[dim] = w, (n - w if side == "lo" else 0)
    return ("subarray", [n, n, n], sub, start, "C", inputs.DOUBLE)


def _parts(case):
    """(spec, count) of each request, and the bytes of the array they lie in."""
    kind = case["kind"]
    layout = case.get("layout", kind)
    if kind == "vector":
        e = DTYPES[case["dtype"]]
        spec = ("vector", case["n"], case["bl"], case["stride"], ("basic", case["dtype"]))
        return [(spec, 1)], ((case["n"] - 1) * case["stride"] + case["bl"]) * e
    if kind == "faces":
        return [(inputs.halo_face(case["n"], *f), 1) for f in _faces(case)], case["n"] ** 3 * 8
    if kind == "flatten" and layout == "face":
        return [(inputs.halo_face(case["n"], case["w"], 2, "lo"), 1)], case["n"] ** 3 * 8
    if layout == "records":
        return [(_record(case["k"]), case["count"])], case["count"] * (16 + 8 * case["k"])
    if layout == "blocks":
        return [(inputs.hindexed_type(*_blocks(case)), 1)], case["span"]
    if kind == "rows":
        r, c, b = case["rows"], case["cols"], case["border"]
        return [(("subarray", [r, c], [r - 2 * b, c - 2 * b], [b, b], "C", inputs.DOUBLE), 1)], r * c * 8
    if kind == "darray":
        n, p = case["n"], case["procs"]
        return [(("darray", p ** 3, case["rank"], [n] * 3, ["cyclic"] * 3, [case["block"]] * 3, [p] * 3, "C",
                  inputs.DOUBLE), 1)], n ** 3 * 8
    raise ValueError(kind)


def _box(dims, start=0):
    """Byte offsets start + sum of one term of each dimension, the last one fastest."""
    idx = torch.full((1,), start, dtype=torch.int64, device="cuda")
    for d in dims:
        d = torch.as_tensor(d, dtype=torch.int64, device="cuda")
        idx = (idx[:, None] + d[None, :]).reshape(-1)
    return idx


def _steps(n, stride):
    return torch.arange(n, dtype=torch.int64, device="cuda") * stride


def _face_box(n, sub, start):
    return _box([_steps(sub[0], n * n * 8), _steps(sub[1], n * 8), _steps(sub[2] * 8, 1)],
                (start[0] * n * n + start[1] * n + start[2]) * 8)


def _offsets(case):
    """Typemap byte offsets of each request, by the definitions of the constructors."""
    kind = case["kind"]
    layout = case.get("layout", kind)
    if kind == "vector":
        e = DTYPES[case["dtype"]]
        return [_box([_steps(case["n"], case["stride"] * e), _steps(case["bl"] * e, 1)])]
    if kind == "faces":
        return [_face_box(case["n"], *inputs.halo_face(case["n"], *f)[2:4]) for f in _faces(case)]
    if layout == "records":
        k = case["k"]
        return [_box([_steps(case["count"], 16 + 8 * k),
                      list(range(4)) + list(range(8, 8 + 8 * k)) + list(range(8 + 8 * k, 13 + 8 * k))])]
    if layout == "blocks":
        lens, disps = (torch.from_numpy(a).cuda() for a in _blocks(case))
        first = torch.cumsum(lens, 0) - lens
        return [torch.repeat_interleave(disps - first, lens) + _steps(int(lens.sum()), 1)]
    if kind == "rows":
        r, c, b = case["rows"], case["cols"], case["border"]
        return [_box([_steps(r - 2 * b, c * 8), _steps((c - 2 * b) * 8, 1)], (b * c + b) * 8)]
    if kind == "darray":
        n, p, r = case["n"], case["procs"], case["rank"]
        own = []
        for d in range(3):
            i = torch.arange(n, device="cuda")
            own.append(i[(i // case["block"]) % p == (r // p ** (2 - d)) % p])
        return [_box([own[0] * (n * n * 8), own[1] * (n * 8), own[2] * 8, _steps(8, 1)])]
    return None


# ---------------------------------------------------------------------------
# what a program has before the call


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "stream": mdt.Stream(torch.cuda.current_stream().cuda_stream)}
    if kind == "mix":
        _prepare_mix(st, case, seed)
    elif kind == "serving":
        _prepare_serving(st, case, seed)
    elif kind == "copy":
        _prepare_copy(st, case, seed)
    elif kind == "flatten":
        (spec, _), = _parts(case)[0]
        st["type"] = mdt.build_type(spec)
        st["segments"] = st["type"].iov_len(-1)[0]
        st["base"] = int(seed) << 12  # the address of the buffer that the segments are for
        st["iov"] = torch.zeros(st["segments"], 2, dtype=torch.int64, device="cuda")
    else:
        parts, nbytes = _parts(case)
        st["reqs"] = [(mdt.build_type(spec), count) for spec, count in parts]
        st["src"] = _random(nbytes, seed)
        st["dst"] = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        st["packed"] = [torch.zeros(t.size() * c, dtype=torch.uint8, device="cuda") for t, c in st["reqs"]]
        if case.get("how") in ("batch", "tuned"):
            st["pack"], st["unpack"] = mdt.Batch(), mdt.Batch()
            for (t, c), out in zip(st["reqs"], st["packed"]):
                st["pack"].add_pack(st["src"].data_ptr(), c, t, 0, out.data_ptr(), -1)
                st["unpack"].add_unpack(out.data_ptr(), out.numel(), st["dst"].data_ptr(), c, t, 0)
            if case["how"] == "tuned":
                st["pack"].autotune(st["stream"])
                st["unpack"].autotune(st["stream"])
    return st


def _prepare_mix(st, case, seed):
    reqs = inputs.batch_mix(nreq=case["requests"], seed=case["layout_seed"], hi=case["hi"])
    lens, disps = inputs.hindexed_blocks(seed=case["layout_seed"])
    st["arenas"] = {"vector": _random(((1 << 21) - 1) * 64 * 8 + 8, seed), "face": _random(512 ** 3 * 8, seed + 1),
                    "hindexed": _random(1 << 31, seed + 2)}
    types = {}
    plan = []
    for r in reqs:
        if r["spec_key"] not in types:
            types[r["spec_key"]] = mdt.build_type(r["spec"] or inputs.hindexed_type(lens, disps))
        t = types[r["spec_key"]]
        plan.append((t, st["arenas"][r["kind"]], min(r["target"], t.size())))
    offs = np.concatenate([[0], np.cumsum([(n + 255) // 256 * 256 for _, _, n in plan])])
    st["out"] = torch.zeros(int(offs[-1]), dtype=torch.uint8, device="cuda")
    st["batch"] = mdt.Batch()
    for (t, src, n), o in zip(plan, offs):
        st["batch"].add_pack(src.data_ptr(), 1, t, 0, st["out"].data_ptr() + int(o), n)


def _prepare_copy(st, case, seed):
    if case["layout"] == "halo":
        n = case["n"]
        st["src"] = st["dst"] = _random(n ** 3 * 8, seed)
        faces = [(w, dim, side) for w in (1, 4) for dim in (0, 1, 2) for side in ("lo", "hi")]
        st["pairs"] = [(mdt.build_type(inputs.halo_face(n, *f)), mdt.build_type(_ghost(n, *f)), 1) for f in faces]
    else:
        k, count = case["k"], case["count"]
        st["src"] = _random(count * (16 + 8 * k), seed)
        st["dst"] = torch.zeros(count * (9 + 8 * k), dtype=torch.uint8, device="cuda")
        st["pairs"] = [(mdt.build_type(_record(k)), mdt.build_type(_tight_record(k)), count)]


def _prepare_serving(st, case, seed):
    st["src"] = _random(1 << 30, seed)
    st["dst"] = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
    types = [mdt.build_type(spec) for _, spec in inputs.serving_types(seed=case["layout_seed"], ntypes=case["ntypes"])]
    trace = inputs.serving_trace(20000.0, 0.05, case["ntypes"], seed=case["layout_seed"])
    st["plan"] = []
    for i in range(case["requests"]):
        t, target = types[int(trace["type_index"][i])], min(int(trace["target"][i]), 4 * MiB)
        count = max(1, min(target // t.size(), (1 << 30) // t.extent()[1]))
        st["plan"].append((t, count, min(target, t.size() * count)))
    st["server"] = mdt.Server(arena_bytes=1 << 30)


# ---------------------------------------------------------------------------
# one pass


def run(st):
    case, ms = st["case"], st["stream"]
    kind = case["kind"]
    if kind == "mix":
        st["batch"].launch(ms)
        return st["out"]
    if kind == "copy":
        for a, b, count in st["pairs"]:
            mdt.mdt_typed_copy_enqueue(st["src"].data_ptr(), count, a, st["dst"].data_ptr(), count, b, 0, -1, ms)
        return st["dst"]
    if kind == "flatten":
        mdt.mdt_type_iov_enqueue(st["type"], 0, st["iov"].data_ptr(), st["segments"], st["base"], ms)
        return st["iov"]
    if kind == "serving":
        return _run_serving(st)
    src, dst = st["src"].data_ptr(), st["dst"].data_ptr()
    if "pack" in st:
        st["pack"].launch(ms)
        st["unpack"].launch(ms)
    elif kind == "ranges":
        (t, count), = st["reqs"]
        total, step, buf = st["packed"][0].numel(), case["budget"], st["packed"][0].data_ptr()
        for at in range(0, total, step):
            mdt.mdt_pack_enqueue(src, count, t, at, buf + at, step, ms)
        for at in range(0, total, step):
            mdt.mdt_unpack_enqueue(buf + at, min(step, total - at), dst, count, t, at, ms)
    else:
        for (t, count), out in zip(st["reqs"], st["packed"]):
            mdt.mdt_pack_enqueue(src, count, t, 0, out.data_ptr(), -1, ms)
        for (t, count), out in zip(st["reqs"], st["packed"]):
            mdt.mdt_unpack_enqueue(out.data_ptr(), out.numel(), dst, count, t, 0, ms)
    return {"packed": st["packed"], "unpacked": st["dst"]}


def _run_serving(st):
    """Pack every request, unpack each from where the server packed it, then give its memory back."""
    srv, src, dst = st["server"], st["src"].data_ptr(), st["dst"].data_ptr()
    packs = [srv.submit_pack(src, count, t, 0, n) for t, count, n in st["plan"]]
    unpacks = []
    for (t, count, n), r in zip(st["plan"], packs):
        srv.wait(r)
        unpacks.append(srv.submit_unpack(srv.result(r)[1], n, dst, count, t, 0))
    for p, u in zip(packs, unpacks):
        srv.wait(u)
        srv.release(u)
        srv.release(p)
    return st["dst"]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what it has to give


def work(case):
    """Each packed byte is read once and written once per direction; a typed copy has one direction, a batch mix only
    packs, and flattening writes 16 bytes per segment (and reads as many for a listed layout)."""
    kind = case["kind"]
    if kind == "vector":
        b = 4 * case["n"] * case["bl"] * DTYPES[case["dtype"]]
    elif kind == "faces":
        b = 4 * sum(8 * w * (case["n"] - 2 * w) ** 2 for w, _, _ in _faces(case))
    elif kind == "rows":
        b = 32 * (case["rows"] - 2 * case["border"]) * (case["cols"] - 2 * case["border"])
    elif kind == "darray":
        b = 32 * (case["n"] / case["procs"]) ** 3
    elif kind == "mix":
        reqs = inputs.batch_mix(nreq=case["requests"], seed=case["layout_seed"], hi=case["hi"])
        b = 2 * sum(min(r["target"], 8 * math.prod(r["spec"][2])) if r["kind"] == "face" else r["target"] for r in reqs)
    elif kind == "copy" and case["layout"] == "halo":
        b = 2 * 6 * 8 * ((case["n"] - 2) ** 2 + 4 * (case["n"] - 8) ** 2)
    elif kind == "flatten":
        b = 32 * case["n"] if case["layout"] == "blocks" else 16 * (case["n"] - 2 * case["w"]) ** 2
    elif kind == "serving":
        b = 4 * 130_000 * case["requests"]  # the trace's mean request (Zipf sizes, rejected above 4 MiB)
    elif case.get("layout", kind) == "records":
        b = (2 if kind == "copy" else 4) * case["count"] * (9 + 8 * case["k"])
    else:
        b = 4 * case["n"] * case["mean"]
    return {"bytes": b, "flops": 0}


def exact(case, seed):
    """The same bytes moved by plain indexing."""
    kind = case["kind"]
    if kind in ("mix", "serving"):
        return None
    if kind == "flatten":
        if case["layout"] == "face":
            n, w = case["n"], case["w"]
            base = _box([_steps(n - 2 * w, n * n * 8), _steps(n - 2 * w, n * 8)], (w * n * n + w * n + w) * 8)
            return torch.stack([base + (int(seed) << 12), torch.full_like(base, 8 * w)], 1)
        lens, disps = (torch.from_numpy(a).cuda() for a in _blocks(case))
        new = torch.cat([torch.ones(1, dtype=torch.bool, device="cuda"), disps[1:] != (disps + lens)[:-1]])
        ends = torch.cumsum(lens, 0)
        first = (ends - lens)[new]
        return torch.stack([disps[new] + (int(seed) << 12), torch.diff(first, append=ends[-1:])], 1)
    if kind == "copy":
        if case["layout"] == "records":
            src = _random(case["count"] * (16 + 8 * case["k"]), seed)
            return src[_offsets(case)[0]]
        n = case["n"]
        dst = _random(n ** 3 * 8, seed)
        for w in (1, 4):
            for dim in (0, 1, 2):
                for side in ("lo", "hi"):
                    a, b = inputs.halo_face(n, w, dim, side), _ghost(n, w, dim, side)
                    dst[_face_box(n, *b[2:4])] = dst[_face_box(n, *a[2:4])]
        return dst
    nbytes = _parts(case)[1]
    src, dst = _random(nbytes, seed), torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    packed = []
    for idx in _offsets(case):
        packed.append(src[idx])
        dst[idx] = packed[-1]
    return {"packed": packed, "unpacked": dst}
