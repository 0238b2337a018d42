"""Performance cases of the data-sharing runtime, through its public entry points.

Each case is a dict of plain values.  `kind` names the form of use:

  affine   one small region (four shared int32 scalars): launch, wait, read the sum
  chain    one fma-chain region (shared scalars, optionally a shared array, published
           as a frame or as a list of references): launch, wait, read the sum
  static   the same chain through the launch that allocates nothing: its result
           record stays on the device, nothing waits
  sweep    regions of 1, 2, 4, ... 64 shared scalars launched back to back on one
           stream, then each region's sum read
  gather   shared arrays gathered into int32 outputs, flat or through two or three
           nested parallel levels
  program  one region whose master runs several parallel loops over two frames
  batched  many regions in one persistent launch: launch, wait, read some sums
  served   a server session: start, submit a burst of requests, collect them, stop

Sizes are those of the repository's workloads (dsr_workloads/configs.py, bench.py) and of
its tests; `draw` spreads cases over the same ranges.  Values are those of the workloads
too: int32 scalars uniform on [-2^20, 2^20], fp64 scalars on the 2^-52 grid of [-1, 1), x on the
2^-23 grid of [-1, 1), array elements on [0, 2^16).
"""
import math

import numpy as np
import torch

from dsr_workloads import configs as W
from paper_1711_10413_amd import dsr as D

SWEEP_KS = (1, 2, 4, 8, 16, 32, 64)
READ_SUMS = 64                 # sums a batched program reads back


def listed():
    return [
        # the plain region of the paper's first figure: launch latency, nothing else
        {"name": "affine_4x256_1k", "kind": "affine", "n": 1024, "teams": 4, "wg": 256},
        # an ordinary small region, ragged: 64 teams, odd length, fixed costs dominate
        {"name": "chain_k8_65537", "kind": "chain", "n": 65537, "teams": 64, "wg": 256, "ni": 4, "nf": 4,
         "alen": 0, "joins": 0, "slab": 4096, "form": "frame", "tail": 0},
        # the same work for a caller that cannot allocate (a tight loop, results on the device)
        {"name": "static_k8_64k", "kind": "static", "n": 65536, "teams": 64, "wg": 256, "ni": 4, "nf": 4,
         "alen": 0, "joins": 1, "slab": 4096},
        # the scalar-sharing sweep: seven large regions streaming back to back
        {"name": "sweep_16m", "kind": "sweep", "n": 1 << 24, "teams": 512, "wg": 256, "joins": 1, "slab": 4096},
        # a large region published through a reference list that overflows the on-chip list
        {"name": "list_k38_16m", "kind": "chain", "n": 1 << 24, "teams": 512, "wg": 256, "ni": 19, "nf": 19,
         "alen": 0, "joins": 0, "slab": 4096, "form": "list", "tail": 0},
        # the largest request of the batched and served mixes run alone: 48 scalars and a 32 KiB frame
        {"name": "chain_frame32k_1m", "kind": "chain", "n": 1 << 20, "teams": 16, "wg": 256, "ni": 32, "nf": 16,
         "alen": 8128, "joins": 0, "slab": 65536, "form": "frame", "tail": 0},
        # shared arrays on the on-chip stack, two nested levels
        {"name": "nested2_2x4096_64m", "kind": "gather", "n": 1 << 26, "teams": 2048, "wg": 256, "arrays": 2,
         "length": 4096, "depth": 2, "joins": 1, "slab": 32768},
        # arrays larger than a CU's on-chip memory: every team's frame goes to its HBM stack
        {"name": "nested2_3x16384_64m", "kind": "gather", "n": 1 << 26, "teams": 2048, "wg": 256, "arrays": 3,
         "length": 16384, "depth": 2, "joins": 1, "slab": 0},
        # three nested levels, odd array length and loop length
        {"name": "nested3_3x257_10m", "kind": "gather", "n": 10000019, "teams": 512, "wg": 256, "arrays": 3,
         "length": 257, "depth": 3, "joins": 1, "slab": 4096},
        # several parallel loops of different bodies in one region
        {"name": "program_1m", "kind": "program", "n": 1 << 20, "teams": 128, "wg": 256, "ni": 3, "nf": 2,
         "arrays": 1, "length": 1024, "joins": 0, "slab": 16384},
        # the batched workload: 10,000 regions in one launch, replayed from a graph
        {"name": "batched_10000", "kind": "batched", "count": 10000, "table": 3, "longest": 1 << 20, "chunk": 65536,
         "wg": 128, "joins": 1, "slab": 33792, "graph": 1},
        # a burst of served requests from 64 templates, a whole session
        {"name": "served_256", "kind": "served", "count": 256, "pool": 64, "table": 4, "longest": 1 << 20,
         "chunk": 65536, "wg": 256, "joins": 0, "slab": 65536},
    ]


def _log(rng, lo, hi):
    return min(hi, int(lo * (hi / lo) ** rng.random()))


def _counts(rng):
    """int32 and fp64 scalar counts: the sweep's, or any pair up to 64 in all."""
    if rng.random() < 0.4:
        k = rng.choice(SWEEP_KS)
        return (k + 1) // 2, k // 2
    return rng.randint(1, 32), rng.randint(0, 32)


def draw(rng):
    kind = rng.choice(["affine", "chain", "chain", "chain", "static", "sweep", "gather", "gather", "program", "batched",
                       "served"])
    wg = rng.choice([64, 128, 256, 256, 256, 512, 1024])
    joins = rng.randint(0, 1)
    if kind == "affine":
        n = _log(rng, 64, 1 << 18)
        return {"kind": kind, "n": n, "teams": rng.randint(1, max(1, min(64, n // 64))), "wg": wg}
    if kind in ("chain", "static"):
        n = _log(rng, 256, 1 << 24 if kind == "chain" else 1 << 20)
        ni, nf = _counts(rng)
        alen = rng.choice([0, 0, _log(rng, 3, 8128)])
        c = {"kind": kind, "n": n, "teams": min(1024 if kind == "chain" else 256, max(1, n // _log(rng, 1024, 65536))),
             "wg": wg, "ni": ni, "nf": nf, "alen": alen, "joins": joins, "slab": rng.choice([0, 4096, 36864])}
        if kind == "chain":
            c["form"] = rng.choice(["frame", "frame", "list"])
            c["tail"] = rng.choice([0, 0, 0, 1])
        return c
    if kind == "sweep":
        return {"kind": kind, "n": _log(rng, 1 << 16, 1 << 24), "teams": rng.choice([128, 256, 512, 1024]), "wg": 256,
                "joins": joins, "slab": rng.choice([0, 4096])}
    if kind == "gather":
        arrays, length = rng.randint(1, 4), _log(rng, 16, 16384)
        if rng.random() < 0.5:
            length = max(16, length & ~3)
        frame = (4 * arrays * length + 15) // 16 * 16
        return {"kind": kind, "n": _log(rng, 4096, 1 << 26), "teams": rng.choice([64, 256, 512, 1024, 2048]), "wg": wg,
                "arrays": arrays, "length": length, "depth": rng.choice([1, 2, 3]), "joins": joins,
                "slab": rng.choice([0, frame if frame <= 131072 else 0])}
    if kind == "program":
        ni, nf = _counts(rng)
        return {"kind": kind, "n": _log(rng, 1024, 1 << 22), "teams": rng.choice([4, 32, 128, 256]), "wg": wg,
                "ni": ni, "nf": nf, "arrays": rng.randint(1, 4), "length": _log(rng, 16, 2048), "joins": joins,
                "slab": rng.choice([0, 65536])}
    if kind == "served":
        return {"kind": kind, "count": rng.randint(32, 512), "pool": rng.randint(8, 64), "table": rng.randint(5, 1 << 20),
                "longest": 1 << 20, "chunk": 65536, "wg": rng.choice([128, 256]), "joins": joins, "slab": 65536}
    count = _log(rng, 200, 4000)
    return {"kind": "batched", "count": count, "table": rng.randint(5, 1 << 20), "longest": 1 << 20, "chunk": 65536,
            "wg": rng.choice([64, 128, 256]), "joins": 1, "slab": 33792, "graph": rng.randint(0, 1)}


# ---- inputs -----------------------------------------------------------------------
def _gpu(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _x(n, g):
    """fp32 on the 2^-23 grid of [-1, 1)."""
    return torch.randint(-(1 << 23), 1 << 23, (n,), dtype=torch.int32, device="cuda", generator=g).float() * 2.0 ** -23


def _scalars(rs, ni, nf):
    s_i = rs.randint(W.I32_LO, W.I32_HI + 1, ni).astype(np.int32)
    s_f = rs.randint(0, 1 << 53, nf).astype(np.float64) * 2.0 ** -52 - 1.0
    return s_i, s_f


def _array(rs, n):
    return rs.randint(0, 1 << 16, n).astype(np.int32)


class _Held:
    """What a program holds between calls: the context, its regions, batch, buffers."""

    def __init__(self, case, **cfg):
        self.case = case
        self.ctx = D.dsr_init(**cfg)
        self.regions = []
        self.batch = None

    def __del__(self):
        try:
            if self.batch is not None:
                D.dsr_batch_free(self.batch)
            for r in self.regions:
                D.dsr_region_free(r)
            D.dsr_destroy(self.ctx)
        except Exception:
            pass


def _affine(case, seed):
    rs = np.random.RandomState(seed % (1 << 32))
    return [int(v) for v in rs.randint(-1000, 1001, 4)]


def _chain_values(case, seed):
    rs = np.random.RandomState(seed % (1 << 32))
    s_i, s_f = _scalars(rs, case["ni"], case["nf"])
    arr = _array(rs, case["alen"]) if case.get("alen") else None
    return s_i, s_f, arr, _x(case["n"], _gpu(seed))


def _arrays(case, seed):
    rs = np.random.RandomState(seed % (1 << 32))
    return [_array(rs, case["length"]) for _ in range(case["arrays"])]


def _sweep_scalars(seed):
    rs = np.random.RandomState(seed % (1 << 32))
    return [_scalars(rs, (k + 1) // 2, k // 2) for k in SWEEP_KS]


def _sweep_x(case, seed):
    g = _gpu(seed)
    return [_x(case["n"], g) for _ in SWEEP_KS]


def _table(case, count):
    """Loop lengths and frame sizes of the mixed workload (log-uniform), and where each
    region's elements lie in the shared buffers."""
    ls, fs = W.cfg4_descriptors(count, seed=case["table"])
    ls = np.minimum(ls, case["longest"])
    offs = np.zeros(count + 1, np.int64)
    offs[1:] = np.cumsum((ls + 63) // 64 * 64)
    return ls, fs, offs


def _mixed(case, count, seed):
    """(ni, nf, alen, scalars, array) of each region of the mixed workload."""
    rs = np.random.RandomState(seed % (1 << 32))
    ls, fs, offs = _table(case, count)
    comp = [W.frame_composition(int(f)) for f in fs]
    s_i = rs.randint(W.I32_LO, W.I32_HI + 1, (count, 32)).astype(np.int32)
    s_f = rs.randint(0, 1 << 53, (count, 16)).astype(np.float64) * 2.0 ** -52 - 1.0
    flat = _array(rs, sum(c[2] for c in comp))
    out, at = [], 0
    for q, (ni, nf, alen) in enumerate(comp):
        out.append((s_i[q, :ni], s_f[q, :nf], flat[at:at + alen]))
        at += alen
    return ls, offs, out


def _up16(v):
    return (v + 15) // 16 * 16


def _chain_region(ctx, case, s_i, s_f, arr, x, y):
    """One region sharing the scalars (and the array) in a frame, or through a list of
    references to the same variables."""
    img, size = D.fma_chain_frame(s_i, s_f, arr)
    ni, nf, alen = len(s_i), len(s_f), 0 if arr is None else len(arr)
    r = D.dsr_region_begin(ctx, case["teams"])
    f = D.dsr_push(r, size, img)
    sched = D.DSR_SCHED_DYNAMIC_TAIL if case.get("tail") else D.DSR_SCHED_STATIC
    args = {"inp": x.data_ptr(), "out": y.data_ptr(), "ni": ni, "nf": nf, "alen": alen, "schedule": sched}
    if case.get("form") == "list":
        refs = [(f, 0)] + [(f, 24 + 8 * nf + 4 * k) for k in range(ni)] + [(f, 24 + 8 * k) for k in range(nf)]
        if alen:
            refs.append((f, _up16(24 + 8 * nf + 4 * ni)))
        D.dsr_publish_list(r, refs, D.DSR_BODY_FMA_CHAIN_REFS, case["n"], **args)
    else:
        D.dsr_publish(r, f, D.DSR_BODY_FMA_CHAIN, case["n"], **args)
    D.dsr_pop(r, f)
    return r


# ---- preparation ----------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    if kind == "affine":
        s = _Held(case, wg_size=case["wg"], lds_slab_bytes=4096, hbm_slab_bytes=4096, max_teams=case["teams"])
        s.out = torch.zeros(case["n"], dtype=torch.int32, device="cuda")
        r = D.dsr_region_begin(s.ctx, case["teams"])
        f = D.dsr_push(r, 24, D.affine_xor_frame(*_affine(case, seed)))
        D.dsr_publish(r, f, D.DSR_BODY_AFFINE_XOR, case["n"], out=s.out.data_ptr())
        D.dsr_pop(r, f)
        s.regions.append(r)
        return s
    if kind in ("chain", "static"):
        s_i, s_f, arr, s_x = _chain_values(case, seed)
        slot = _up16(24 + 8 * case["nf"] + 4 * case["ni"]) + _up16(4 * case["alen"]) + 1024
        s = _Held(case, wg_size=case["wg"], lds_slab_bytes=case["slab"], hbm_slab_bytes=slot,
                  max_teams=case["teams"], master_joins=case["joins"])
        s.x, s.y = s_x, torch.zeros(case["n"], dtype=torch.float64, device="cuda")
        s.regions.append(_chain_region(s.ctx, case, s_i, s_f, arr, s.x, s.y))
        if kind == "static":
            s.rec = torch.zeros(D.C.sizeof(D.dsr_result_rec), dtype=torch.uint8, device="cuda")
        return s
    if kind == "sweep":
        s = _Held(case, wg_size=case["wg"], lds_slab_bytes=case["slab"], hbm_slab_bytes=4096,
                  max_teams=case["teams"], master_joins=case["joins"])
        s.xs = _sweep_x(case, seed)
        s.ys = [torch.zeros(case["n"], dtype=torch.float64, device="cuda") for _ in SWEEP_KS]
        s.regions = [_chain_region(s.ctx, case, s_i, s_f, None, x, y)
                     for (s_i, s_f), x, y in zip(_sweep_scalars(seed), s.xs, s.ys)]
        return s
    if kind == "gather":
        arrs = _arrays(case, seed)
        frame = 4 * case["arrays"] * case["length"]
        s = _Held(case, wg_size=case["wg"], lds_slab_bytes=case["slab"], hbm_slab_bytes=_up16(frame),
                  max_teams=case["teams"], master_joins=case["joins"])
        s.out = torch.zeros(case["n"], dtype=torch.int32, device="cuda")
        r = D.dsr_region_begin(s.ctx, case["teams"])
        f = D.dsr_push(r, frame, D.gather_frame(arrs))
        more = {"depth": case["depth"]} if case["depth"] > 1 else {}
        D.dsr_publish(r, f, D.DSR_BODY_GATHER_NESTED if case["depth"] > 1 else D.DSR_BODY_GATHER, case["n"],
                      out=s.out.data_ptr(), arrays=case["arrays"], length=case["length"], **more)
        D.dsr_pop(r, f)
        s.regions.append(r)
        return s
    if kind == "program":
        s_i, s_f, _, x = _chain_values(case, seed)
        arrs = _arrays(case, seed)
        frame = 4 * case["arrays"] * case["length"]
        s = _Held(case, wg_size=case["wg"], lds_slab_bytes=case["slab"], hbm_slab_bytes=_up16(frame) + 2048,
                  max_teams=case["teams"], master_joins=case["joins"])
        n = case["n"]
        s.x, s.y = x, torch.zeros(n, dtype=torch.float64, device="cuda")
        s.out = torch.zeros(n, dtype=torch.int32, device="cuda")
        s.arr = torch.zeros(n, dtype=torch.int32, device="cuda")
        r = D.dsr_region_begin(s.ctx, case["teams"])
        img, size = D.fma_chain_frame(s_i, s_f)
        f0 = D.dsr_push(r, size, img)
        D.dsr_publish(r, f0, D.DSR_BODY_FMA_CHAIN, n, inp=s.x.data_ptr(), out=s.y.data_ptr(), ni=len(s_i), nf=len(s_f))
        f1 = D.dsr_push(r, 24, D.affine_xor_frame(*_affine(case, seed)))
        D.dsr_publish(r, f1, D.DSR_BODY_AFFINE_XOR, n, out=s.out.data_ptr())
        D.dsr_pop(r, f1)
        f2 = D.dsr_push(r, frame, D.gather_frame(arrs))
        D.dsr_publish(r, f2, D.DSR_BODY_GATHER, n, out=s.arr.data_ptr(), arrays=case["arrays"], length=case["length"])
        D.dsr_pop(r, f2)
        D.dsr_pop(r, f0)
        s.regions.append(r)
        return s
    count = case["count"] if kind == "batched" else case["pool"]
    ls, offs, mixed = _mixed(case, count, seed)
    s = _Held(case, wg_size=case["wg"], lds_slab_bytes=case["slab"], hbm_slab_bytes=65536, max_teams=4096,
              master_joins=case["joins"])
    s.x = _x(int(offs[-1]), _gpu(seed))
    if kind == "batched":
        s.y = torch.zeros(int(offs[-1]), dtype=torch.float64, device="cuda")
        out_at = offs
    else:
        # every request writes to its own part of the output buffer
        which = np.random.RandomState(case["table"]).randint(0, count, case["count"])
        out_at = np.zeros(case["count"] + 1, np.int64)
        out_at[1:] = np.cumsum((ls[which] + 63) // 64 * 64)
        s.y = torch.zeros(int(out_at[-1]), dtype=torch.float64, device="cuda")
        s.requests = [(int(w), s.y.data_ptr() + 8 * int(o)) for w, o in zip(which, out_at)]
    regs = [D.fma_chain_region(s.ctx, max(1, -(-int(ls[q]) // case["chunk"])), s_i, s_f, arr, int(ls[q]),
                               s.x.data_ptr() + 4 * int(offs[q]), s.y.data_ptr() + 8 * int(out_at[q]))
            for q, (s_i, s_f, arr) in enumerate(mixed)]
    if kind == "batched":
        s.batch = D.dsr_batch_create(s.ctx, regs)
        for r in regs:
            D.dsr_region_free(r)
        D.dsr_batch_tune(s.batch, wg_size=case["wg"], lds_slab_bytes=case["slab"], master_joins=case["joins"],
                         use_graph=case["graph"])
        s.read = np.linspace(0, count - 1, min(count, READ_SUMS)).astype(int).tolist()
    else:
        for r in regs:
            D.dsr_region_freeze(r)
        s.regions = regs
    return s


# ---- one pass ---------------------------------------------------------------------------
def run(s):
    kind = s.case["kind"]
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "static":
        D.dsr_launch_static(s.regions[0], s.rec.data_ptr(), stream)
        return {"y": s.y, "record": s.rec}
    if kind == "batched":
        D.dsr_batch_launch(s.batch, stream)
        status = D.dsr_batch_sync(s.batch)
        return {"y": s.y, "sums": np.array([D.dsr_batch_result(s.batch, q)[1] for q in s.read]), "status": status}
    if kind == "served":
        return _session(s)
    for r in s.regions:
        D.dsr_launch(r, stream)
    status = [D.dsr_region_sync(r) for r in s.regions]
    if kind == "affine":
        return {"out": s.out, "sum": D.dsr_region_reduction(s.regions[0], 0)[0], "status": status}
    if kind == "gather":
        return {"out": s.out, "status": status}
    if kind == "program":
        return {"y": s.y, "out": s.out, "arr": s.arr, "sum": D.dsr_region_reduction(s.regions[0], 0)[1],
                "total": D.dsr_region_reduction(s.regions[0], 1)[0], "status": status}
    return {"y": s.ys if kind == "sweep" else s.y,
            "sums": np.array([D.dsr_region_reduction(r, 0)[1] for r in s.regions]), "status": status}


def _session(s):
    c = s.case
    # work the requests read or overwrite has to be finished when they are submitted
    torch.cuda.current_stream().synchronize()
    srv = D.dsr_serve_start(s.ctx, wg_size=c["wg"], lds_slab_bytes=c["slab"], master_joins=c["joins"], slots=256,
                            slot_bytes=40960, max_teams=64, ring_items=1 << 15, idle_ms=3000)
    which, done, q = {}, [], 0
    try:
        while len(done) < len(s.requests):
            while q < len(s.requests):
                t, out = s.requests[q]
                try:
                    which[D.dsr_serve_submit(srv, s.regions[t], [out])] = q
                except D.DsrError as e:
                    if e.code != D.DSR_E_BUSY:
                        raise
                    break
                q += 1
            done += D.dsr_serve_poll(srv)
    finally:
        D.dsr_serve_stop(srv)
    sums, status = np.zeros(len(done)), np.zeros(len(done), np.int64)
    for d in done:
        at = which[d["ticket"]]
        sums[at], status[at] = d["f64"][0], d["status"]
    return {"y": s.y, "sums": sums, "status": status}


# ---- bytes and operations a pass cannot do without ----------------------------------------
def work(case):
    kind, n = case["kind"], case.get("n", 0)
    if kind == "affine":
        return {"bytes": 4 * n + 24, "flops": 0}
    if kind in ("chain", "static"):
        k = case["ni"] + case["nf"]
        return {"bytes": 12 * n + 24 + 8 * case["nf"] + 4 * case["ni"] + 4 * case["alen"], "flops": (2 * k + 1) * n}
    if kind == "sweep":
        # seven regions, each with its own input and output
        return {"bytes": 12 * n * len(SWEEP_KS), "flops": n * sum(2 * k + 1 for k in SWEEP_KS)}
    if kind == "gather":
        return {"bytes": 4 * n + 4 * case["arrays"] * case["length"], "flops": 0}
    if kind == "program":
        return {"bytes": (12 + 4 + 4) * n + 4 * case["arrays"] * case["length"],
                "flops": (2 * (case["ni"] + case["nf"]) + 1) * n}
    count = case["count"] if kind == "batched" else case["pool"]
    ls, fs, _ = _table(case, count)
    if kind == "served":
        which = np.random.RandomState(case["table"]).randint(0, count, case["count"])
        ls, fs = ls[which], fs[which]
    ks = [ni + nf for ni, nf, _ in (W.frame_composition(int(f)) for f in fs)]
    return {"bytes": int(12 * ls.sum() + fs.sum()), "flops": int(sum((2 * k + 1) * int(L) for k, L in zip(ks, ls)))}


# ---- the same values in 64 bits --------------------------------------------------------------
def _chain_exact(s_i, s_f, arr, x):
    """arr[i mod len] + x[i] * (the scalars' sum), in fp64."""
    y = x.double() * (math.fsum([float(v) for v in s_i]) + math.fsum([float(v) for v in s_f]))
    if arr is not None and len(arr):
        a = torch.from_numpy(np.ascontiguousarray(arr)).cuda().double()
        y += a.repeat(-(-len(x) // len(arr)))[:len(x)]
    return y


def exact(case, seed):
    kind = case["kind"]
    if kind in ("affine", "gather"):
        return None                      # whole numbers
    if kind in ("chain", "static", "program"):
        s_i, s_f, arr, x = _chain_values(case, seed)
        y = _chain_exact(s_i, s_f, arr, x)
        total = float(y.sum())
        if kind == "chain":
            return {"y": y, "sums": np.array([total]), "status": None}
        if kind == "static":
            return {"y": y, "record": None}
        return {"y": y, "out": None, "arr": None, "sum": total, "total": None, "status": None}
    if kind == "sweep":
        ys = [_chain_exact(s_i, s_f, None, x) for (s_i, s_f), x in zip(_sweep_scalars(seed), _sweep_x(case, seed))]
        return {"y": ys, "sums": np.array([float(y.sum()) for y in ys]), "status": None}
    count = case["count"] if kind == "batched" else case["pool"]
    ls, offs, mixed = _mixed(case, count, seed)
    x = _x(int(offs[-1]), _gpu(seed))
    if kind == "batched":
        which, at = np.arange(count), offs
    else:
        which = np.random.RandomState(case["table"]).randint(0, count, case["count"])
        at = np.zeros(case["count"] + 1, np.int64)
        at[1:] = np.cumsum((ls[which] + 63) // 64 * 64)
    y = torch.zeros(int(at[-1]), dtype=torch.float64, device="cuda")
    for k, q in enumerate(which):
        s_i, s_f, arr = mixed[q]
        y[int(at[k]):int(at[k]) + int(ls[q])] = _chain_exact(s_i, s_f, arr, x[int(offs[q]):int(offs[q]) + int(ls[q])])
    read = np.linspace(0, count - 1, min(count, READ_SUMS)).astype(int).tolist() if kind == "batched" else range(len(which))
    sums = np.array([float(y[int(at[k]):int(at[k]) + int(ls[which[k]])].sum()) for k in read])
    return {"y": y, "sums": sums, "status": None}
