"""Performance cases of the halo-exchange buffer engine.

Five kinds of work, each through the package's public entry points with the
library's default schedules (tuning is optional, and a solver that exchanges
a few hundred times on a changing mesh does not pay for it):

* ``rank``   one rank's persistent request, as a distributed program holds it:
             Start (pack), Wait (redistribution, unpack), backward of the pack
* ``world``  every rank of a decomposition on one GPU with the simulated
             transfer: Start, Wait, and the backward where the case asks for it
* ``batch``  many independent uneven requests driven as one batch
* ``train``  the differentiable exchange inside a training step
* ``setup``  plan, message lists, batch and first exchange of a new matrix

Sizes are those of the stencil, random-matrix and batched workloads of the
benchmark, and generic ones around them.
"""
import numpy as np
import torch

import paper_2309_07337_amd as P
from paper_2309_07337_amd.autograd import HaloExchange, halo_gather

VARIANTS = {"plain": P.HX_PLAIN, "2step": P.HX_LOCALITY_2STEP, "3step": P.HX_LOCALITY_3STEP}
DTYPES = {"f32": torch.float32, "f64": torch.float64}
FAR = 0.3  # random matrices: share of a row's entries drawn from all columns


def listed():
    f = dict
    return [
        # the smallest call: one rank of a 2D solver (128 x 128 rows, four neighbours),
        # one exchange per iteration, all latency
        f(name="rank_5pt_f64", kind="rank", matrix="5pt", px=4, py=4, bx=128, by=128, variant="plain", ppn=4,
          node_map="block", ncols=1, dtype="f64", backward=False),
        # one rank of the random matrix with its redistribution and backward: thousands
        # of halo rows over every other rank
        f(name="rank_random_f64", kind="rank", matrix="random", n=1 << 18, ranks=256, nnz=32, variant="2step", ppn=16,
          node_map="block", ncols=1, dtype="f64", backward=True),
        # one smoothing step of a 3D 27-point problem on all 512 ranks: a few MB, launch-bound
        f(name="world_27pt_f64", kind="world", matrix="27pt", px=8, py=8, pz=8, bx=16, by=16, bz=16, variant="2step",
          ppn=64, node_map="block", ncols=1, dtype="f64", backward=False),
        # the largest: 4096 ranks of the 2^22-row random matrix, one value per row, node-aware
        f(name="world_random_f64", kind="world", matrix="random", n=1 << 22, ranks=4096, nnz=32, variant="2step",
          ppn=128, node_map="block", ncols=1, dtype="f64", backward=False),
        # single precision with the backward through the plan's stages
        f(name="world_random_f32_bwd", kind="world", matrix="random", n=1 << 20, ranks=1024, nnz=32, variant="2step",
          ppn=64, node_map="cyclic", ncols=1, dtype="f32", backward=True),
        # aggregated messages, three values per row (displacements, velocities), uneven ranks
        f(name="world_3step_f64x3", kind="world", matrix="random", n=700_001, ranks=509, nnz=24, variant="3step",
          ppn=32, node_map="block", ncols=3, dtype="f64", backward=False),
        # the benchmark's batched exchange with its backward: uneven plans, 16 values per row
        f(name="batch_f64x16", kind="batch", plans=60, hmin=1000, hmax=1_000_000, ncols=16, dtype="f64"),
        # five conserved variables per cell: rows of 40 bytes
        f(name="batch_f64x5", kind="batch", plans=40, hmin=500, hmax=400_000, ncols=5, dtype="f64"),
        # training step over the 27-point mesh, 64 features per node
        f(name="train_27pt_f32x64", kind="train", matrix="27pt", px=8, py=8, pz=8, bx=16, by=16, bz=16,
          variant="plain", ppn=64, node_map="block", ncols=64, dtype="f32"),
        # training step over an irregular graph with a feature width that is no power of two
        f(name="train_random_f32x100", kind="train", matrix="random", n=150_000, ranks=120, nnz=16, variant="plain",
          ppn=8, node_map="block", ncols=100, dtype="f32"),
        # a new 27-point matrix: halo discovery, lists, batch, first exchange
        f(name="setup_27pt", kind="setup", matrix="27pt", px=8, py=8, pz=8, bx=16, by=16, bz=16, variant="2step",
          ppn=64, node_map="block", ncols=1, dtype="f64", source="csr"),
        # a new irregular matrix on a thousand ranks
        f(name="setup_random", kind="setup", matrix="random", n=1 << 20, ranks=1024, nnz=32, variant="2step", ppn=32,
          node_map="block", ncols=1, dtype="f64", source="csr"),
    ]


def _log_int(rng, lo, hi):
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def _draw_matrix(rng, big):
    """A matrix of at most about `big` rows."""
    kind = rng.choice(["5pt", "27pt", "random", "random"])
    if kind == "5pt":
        px, py = rng.randint(1, 12), rng.randint(2, 12)
        side = max(2, int((_log_int(rng, 400, big) / (px * py)) ** 0.5))
        return dict(matrix="5pt", px=px, py=py, bx=side + rng.randint(0, 3), by=side, ranks=px * py)
    if kind == "27pt":
        px, py, pz = (rng.randint(1, 8) for _ in range(3))
        pz = max(pz, 2)
        side = max(2, int((_log_int(rng, 2000, big) / (px * py * pz)) ** (1 / 3)))
        side = min(side, 40)
        return dict(matrix="27pt", px=px, py=py, pz=pz, bx=side, by=side, bz=max(1, side - rng.randint(0, 2)),
                    ranks=px * py * pz)
    n = _log_int(rng, 5000, big)
    return dict(matrix="random", n=n, ranks=max(2, min(_log_int(rng, 4, 1024), n // 256)), nnz=rng.randint(5, 32))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["rank", "world", "world", "batch", "batch", "train", "setup"])
    dtype = rng.choice(["f64", "f64", "f32"])
    if kind == "batch":
        ncols = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 16, 20, 24, 32])
        hmax = int(min(1_000_000, _log_int(rng, 4000, 1_000_000) * 16 // ncols))
        return dict(kind="batch", plans=rng.randint(1, 60), hmin=rng.randint(1, 1000), hmax=max(hmax, 2000),
                    ncols=ncols, dtype=dtype)
    if kind == "train":
        c = _draw_matrix(rng, 200_000)
        c.update(kind="train", ncols=_log_int(rng, 4, 128), dtype=rng.choice(["f32", "f32", "f64"]))
    elif kind == "rank":
        c = _draw_matrix(rng, 300_000)
        c.update(kind="rank", ncols=rng.choice([1, 1, 2, 3, 5, 16]), dtype=dtype, backward=rng.random() < 0.5)
    elif kind == "world":
        c = _draw_matrix(rng, 1_500_000)
        c.update(kind="world", ncols=rng.choice([1, 1, 1, 2, 3, 4, 5, 7]), dtype=dtype, backward=rng.random() < 0.5)
    else:
        c = _draw_matrix(rng, 1_000_000)
        c.update(kind="setup", ncols=1, dtype=dtype, source=rng.choice(["csr", "csr", "halos"]))
    c["variant"] = "plain" if kind == "train" else rng.choice(["plain", "2step", "2step", "3step"])
    c["ppn"] = rng.randint(1, max(1, c["ranks"] // 2))
    c["node_map"] = "block" if c["variant"] == "3step" else rng.choice(["block", "block", "cyclic"])
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _rank_count(case):
    if case["matrix"] == "random":
        return case["ranks"]
    return case["px"] * case["py"] * case.get("pz", 1)


def _row_count(case):
    if case["matrix"] == "random":
        return case["n"]
    return _rank_count(case) * case["bx"] * case["by"] * case.get("bz", 1)


def _row_starts(case):
    R, n = _rank_count(case), _row_count(case)
    return np.arange(R + 1, dtype=np.int64) * n // R


def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * int(seed) + stream)


def _values(shape, dtype, seed, stream):
    return torch.rand(shape, dtype=dtype, device="cuda", generator=_gen(seed, stream)) * 2 - 1


def _stencil(case):
    """CSR of a 5- or 27-point stencil; ranks own blocks, rows numbered block by block."""
    px, py, pz = case["px"], case["py"], case.get("pz", 1)
    bx, by, bz = case["bx"], case["by"], case.get("bz", 1)
    n = _row_count(case)
    row = torch.arange(n, device="cuda")
    blk, loc = row // (bx * by * bz), row % (bx * by * bz)
    x = (blk % px) * bx + loc % bx
    y = (blk // px % py) * by + loc // bx % by
    z = (blk // (px * py)) * bz + loc // (bx * by)
    if case["matrix"] == "5pt":
        steps = [(0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0)]
    else:
        steps = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
    cols = torch.empty((n, len(steps)), dtype=torch.int32, device="cuda")
    for k, (dx, dy, dz) in enumerate(steps):
        X, Y, Z = x + dx, y + dy, z + dz
        ok = (X >= 0) & (X < px * bx) & (Y >= 0) & (Y < py * by) & (Z >= 0) & (Z < pz * bz)
        c = (X // bx + px * (Y // by + py * (Z // bz))) * (bx * by * bz) + X % bx + bx * (Y % by + by * (Z % bz))
        cols[:, k] = torch.where(ok, c, -1)
    ok = cols >= 0
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(ok.sum(1), 0, out=row_ptr[1:])
    return row_ptr, cols[ok]


def _relabel(case, seed):
    """A permutation of the rows that keeps every row on its rank: each seed's
    random matrix has other columns, and lists of the same sizes."""
    rs = torch.from_numpy(_row_starts(case)).cuda()
    n = _row_count(case)
    rank = torch.searchsorted(rs, torch.arange(n, device="cuda"), right=True) - 1
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=_gen(seed, 5))
    return torch.argsort(2 * rank + u)


def _random_matrix(case, seed):
    """CSR of random rows: an entry is anywhere with probability FAR, else in its rank's rows."""
    n, k = case["n"], case["nnz"]
    rs = torch.from_numpy(_row_starts(case)).cuda()
    rank = torch.searchsorted(rs, torch.arange(n, device="cuda"), right=True) - 1
    g = _gen(0, 1)
    u = torch.rand((n, k), device="cuda", generator=g)
    far = torch.rand((n, k), device="cuda", generator=g) < FAR
    lo, size = rs[rank][:, None], (rs[rank + 1] - rs[rank])[:, None]
    near_col = lo + torch.minimum((u * size).long(), size - 1)
    far_col = torch.randint(0, n, (n, k), device="cuda", generator=g)
    cols = _relabel(case, seed)[torch.where(far, far_col, near_col).reshape(-1)].to(torch.int32)
    return torch.arange(n + 1, dtype=torch.int64, device="cuda") * k, cols


def _matrix(case, seed):
    return _random_matrix(case, seed) if case["matrix"] == "random" else _stencil(case)


def _halos(case, row_ptr, cols):
    """(per-rank offsets, columns): the distinct off-rank columns of every rank, ascending."""
    n, R = _row_count(case), _rank_count(case)
    rs = torch.from_numpy(_row_starts(case)).cuda()
    keys = []
    step = 1 << 22  # rows at a time
    for r0 in range(0, n, step):
        r1 = min(n, r0 + step)
        e0, e1 = int(row_ptr[r0]), int(row_ptr[r1])
        row = torch.repeat_interleave(torch.arange(r0, r1, device="cuda"), row_ptr[r0 + 1:r1 + 1] - row_ptr[r0:r1])
        rank = torch.searchsorted(rs, row, right=True) - 1
        c = cols[e0:e1].long()
        off = (c < rs[rank]) | (c >= rs[rank + 1])
        keys.append(torch.unique(rank[off] * n + c[off]))
    key = torch.unique(torch.cat(keys))
    ptr = torch.searchsorted(key, torch.arange(R + 1, device="cuda") * n)
    return ptr, (key % n).to(torch.int32)


def _send_arena(req, ncols, dtype):
    """The request's send arena; the view keeps the request that owns the memory."""
    view = P.req_arena_view(req, P.HX_ARENA_SEND, ncols, dtype)
    view.req = req
    return view


def _build_plan(case, row_ptr, cols):
    return P.hx_plan_from_csr(_rank_count(case), _row_starts(case), case["ppn"], VARIANTS[case["variant"]], row_ptr,
                              cols, node_map=case["node_map"])


def _batch_sizes(case):
    """Rows of each plan: spread evenly over the logarithm of the range, in no particular order."""
    r = np.random.default_rng(7)
    u = (r.permutation(case["plans"]) + r.random(case["plans"])) / case["plans"]
    return [int(h) for h in np.exp(np.log(case["hmin"]) + u * np.log(case["hmax"] / case["hmin"])).clip(min=1)]


def _batch_lists(seed, b, h):
    """Plan b of h rows: its neighbours, message sizes (h in all), and per message ascending local rows."""
    r = np.random.default_rng(b)
    k = int(min(h, max(1, 4096.0 ** r.random())))
    procs = np.sort(r.choice(4095, k, replace=False) + 1).astype(np.int32)
    counts = 1 + np.bincount(r.integers(0, k, h - k), minlength=k)
    msg = torch.repeat_interleave(torch.arange(k, device="cuda"), torch.from_numpy(counts).cuda())
    key = torch.sort(msg * h + torch.randint(0, h, (h,), device="cuda", generator=_gen(seed, 100 + b))).values
    return procs, counts.astype(np.int32), (key % h).to(torch.int32)


def _pool(case):
    """First row of every plan in the pooled halos and gradients (each at a multiple of 32 rows), and the end."""
    return np.concatenate([[0], np.cumsum([(h + 31) // 32 * 32 for h in _batch_sizes(case)])])


# ---------------------------------------------------------------------------
# The five kinds
# ---------------------------------------------------------------------------
def prepare(case, seed):
    st = dict(case=case)
    kind, C, dt = case["kind"], case["ncols"], DTYPES[case["dtype"]]
    if kind == "batch":
        at = _pool(case)
        st.update(halo=torch.zeros((int(at[-1]), C), dtype=dt, device="cuda"), reqs=[], sends=[])
        st["g_x"] = torch.zeros_like(st["halo"])
        for b, h in enumerate(_batch_sizes(case)):
            procs, counts, idx = _batch_lists(seed, b, h)
            x, g_send = _values((h, C), dt, seed, 1000 + b), _values((h, C), dt, seed, 3000 + b)
            halo, g_x = (st[k][int(at[b]):int(at[b]) + h] for k in ("halo", "g_x"))
            topo = P.hx_topo_create(0, 4096, procs, procs)
            req = P.hx_neighbor_alltoallv_init(x, counts, None, idx.cpu().numpy(), halo, counts, None, topo)
            P.req_arena_view(req, P.HX_ARENA_RECV, C, dt).copy_(_values((h, C), dt, seed, 2000 + b))
            P.hx_req_bind_grad(req, g_send, g_x)
            st["reqs"].append(req)
            st["sends"].append(_send_arena(req, C, dt))
        st["batch"] = P.hx_batch_init(st["reqs"])
        return st
    row_ptr, cols = _matrix(case, seed)
    n = _row_count(case)
    if kind == "setup":
        hptr, hcols = _halos(case, row_ptr, cols)
        st.update(row_ptr=row_ptr, cols=cols, halo_ptr=hptr.cpu().numpy(), halo_cols=hcols,
                  x=_values((n, C), dt, seed, 2), halo=torch.zeros((int(hptr[-1]), C), dtype=dt, device="cuda"))
        return st
    plan = _build_plan(case, row_ptr, cols)
    hptr, _ = _halos(case, row_ptr, cols)
    H = int(hptr[-1])
    del row_ptr, cols
    if kind == "rank":
        rank, first, last = _the_rank(case)
        x_all, halo_all = _values((n, C), dt, seed, 2), torch.zeros((H, C), dtype=dt, device="cuda")
        x, halo = x_all[first:last].clone(), torch.zeros((int(hptr[rank + 1] - hptr[rank]), C), dtype=dt, device="cuda")
        req = P.hx_req_from_plan(plan, rank, x, halo)
        recv = P.req_arena_view(req, P.HX_ARENA_RECV, C, dt)
        # the receive arena holds what the rank's peers send
        world = P.hx_batch_from_plan(plan, x_all, halo_all, flags=P.HX_WORLD_SIM_TRANSFER)
        P.hx_batch_start(world)
        P.hx_batch_wait(world)
        arena, at = P.batch_arena_view(world, P.HX_ARENA_RECV, C, dt), 0
        for part in (P.HX_ARENA_RECV, P.HX_ARENA_RECV | 2):
            a0, a1 = (P.hx_batch_arena_offset(world, part, r) for r in (rank, rank + 1))
            recv[at:at + a1 - a0] = arena[a0:a1]
            at += a1 - a0
        torch.cuda.synchronize()
        st.update(req=req, x=x, halo=halo, send=_send_arena(req, C, dt))
        if case["backward"]:
            e1 = int(P.hx_plan_field(plan, rank, "s1_idx").size)
            st.update(g_send=_values((e1, C), dt, seed, 4), g_x=torch.zeros_like(x))
        return st
    if kind == "train":
        st["ex"] = HaloExchange(plan, n, H, C, dtype=dt)
        st["x"] = _values((n, C), dt, seed, 2).requires_grad_(True)
        st["g"] = _values((H, C), dt, seed, 3)
        return st
    x, halo = _values((n, C), dt, seed, 2), torch.zeros((H, C), dtype=dt, device="cuda")
    flags = P.HX_WORLD_SIM_TRANSFER | (P.HX_WORLD_STAGED_BACKWARD if case["backward"] else 0)
    st.update(x=x, halo=halo, batch=P.hx_batch_from_plan(plan, x, halo, flags=flags))
    if case["backward"]:
        st.update(g_halo=_values((H, C), dt, seed, 3), g_x=torch.zeros_like(x))
        P.hx_batch_bind_grad(st["batch"], st["g_halo"], st["g_x"])
    return st


def _the_rank(case):
    """The rank of a one-rank case, in the middle of the decomposition, and the rows its request reads."""
    R, rs = _rank_count(case), _row_starts(case)
    if case["matrix"] == "random":
        rank = R // 2
    else:
        px, py, pz = case["px"], case["py"], case.get("pz", 1)
        rank = px // 2 + px * (py // 2 + py * (pz // 2))
    first, last = rank, rank + 1
    if case["variant"] == "3step":  # the rows of its whole node
        first = rank // case["ppn"] * case["ppn"]
        last = min(R, first + case["ppn"])
    return rank, int(rs[first]), int(rs[last])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "rank":
        P.hx_start(state["req"])
        P.hx_wait(state["req"])
        if not case["backward"]:
            return state["send"], state["halo"]
        P.hx_backward_noalloc(state["req"], state["g_send"], state["g_x"])
        return state["send"], state["halo"], state["g_x"]
    if kind == "world":
        P.hx_batch_start(state["batch"])
        P.hx_batch_wait(state["batch"])
        if not case["backward"]:
            return state["halo"]
        P.hx_batch_backward(state["batch"])
        return state["halo"], state["g_x"]
    if kind == "batch":
        P.hx_batch_start(state["batch"])
        P.hx_batch_wait(state["batch"])
        P.hx_batch_backward(state["batch"])
        return state["sends"], state["halo"], state["g_x"]
    if kind == "train":
        y = halo_gather(state["x"], state["ex"])
        gx, = torch.autograd.grad(y, state["x"], state["g"])
        return y.detach(), gx
    # setup: the lists a transport posts its messages from, and the first exchange
    R, rs, variant = _rank_count(case), _row_starts(case), VARIANTS[case["variant"]]
    if case["source"] == "csr":
        plan = _build_plan(case, state["row_ptr"], state["cols"])
    else:
        plan = P.hx_plan_from_halos(R, rs, case["ppn"], variant, state["halo_ptr"], state["halo_cols"],
                                    node_map=case["node_map"])
    lists = [P.hx_plan_field_all(plan, f) for f in ("s1_procs", "s1_counts", "r1_procs", "r1_counts", "s2_procs",
                                                    "s2_counts", "r2_procs", "r2_counts")]
    batch = P.hx_batch_from_plan(plan, state["x"], state["halo"], flags=P.HX_WORLD_SIM_TRANSFER)
    P.hx_batch_start(batch)
    P.hx_batch_wait(batch)
    return state["halo"], lists


# ---------------------------------------------------------------------------
# Work and exact results
# ---------------------------------------------------------------------------
def _halo_rows(case):
    """Expected halo rows of all ranks."""
    n, R = _row_count(case), _rank_count(case)
    if case["matrix"] == "random":
        m, other = n / R * case["nnz"] * FAR * (1 - 1 / R), n * (1 - 1 / R)  # draws of one rank, columns they hit
        return R * other * (1 - float(np.exp(-m / other)))
    p = [case["px"], case["py"], case.get("pz", 1)]
    b = [case["bx"], case["by"], case.get("bz", 1)]
    if case["matrix"] == "27pt":
        ext = [pi * bi + 2 * (pi - 1) for pi, bi in zip(p, b)]
        return float(ext[0] * ext[1] * ext[2] - n)
    return float(2 * (p[0] - 1) * p[1] * b[1] + 2 * (p[1] - 1) * p[0] * b[0])


def work(case):
    """Bytes one pass cannot do without: vectors and gradients read once, send
    slots, receive slots, halo and gradients written once (a member's or rank's
    receive slots are read instead), one 4-byte index per gathered row; for a
    setup the matrix or halo lists, read once, with the lists written once.
    Additions of the backward as flops."""
    C, rb = case["ncols"], case["ncols"] * (8 if case["dtype"] == "f64" else 4)
    if case["kind"] == "batch":
        h = float(sum(_batch_sizes(case)))
        # x read, send written; recv read, halo written; g_send read, g_x written; pack and sum indices
        return dict(bytes=6 * h * rb + 8 * h, flops=h * C)
    n, H = _row_count(case), _halo_rows(case)
    if case["kind"] == "rank":
        R = _rank_count(case)
        n, H = n / R, H / R
        bwd = (H + n) * rb + 4 * H if case["backward"] else 0
        return dict(bytes=min(n, H) * rb + 3 * H * rb + 4 * H + bwd, flops=H * C if case["backward"] else 0)
    fwd = n * rb + 3 * H * rb + 4 * H
    if case["kind"] == "setup":
        if case["source"] == "csr":
            nnz = n * (case["nnz"] if case["matrix"] == "random" else (5 if case["matrix"] == "5pt" else 27))
            return dict(bytes=8 * n + 4 * nnz + 12 * H + fwd, flops=0)
        return dict(bytes=4 * H + 12 * H + fwd, flops=0)
    if case["kind"] == "train" or case["backward"]:
        return dict(bytes=fwd + (H + n) * rb + 4 * H, flops=H * C)
    return dict(bytes=fwd, flops=0)


def _row_sums(rows, index, values):
    """Sum of the values of each index, in 64 bits."""
    out = torch.zeros((rows, values.shape[1]), dtype=torch.float64, device="cuda")
    return out.index_add_(0, index.long(), values.double())


def exact(case, seed):
    kind, C, dt = case["kind"], case["ncols"], DTYPES[case["dtype"]]
    if kind == "batch":
        at, sends = _pool(case), []
        halo = torch.zeros((int(at[-1]), C), dtype=torch.float64, device="cuda")
        g_x = torch.zeros_like(halo)
        for b, h in enumerate(_batch_sizes(case)):
            idx, own = _batch_lists(seed, b, h)[2], slice(int(at[b]), int(at[b]) + h)
            sends.append(_values((h, C), dt, seed, 1000 + b)[idx.long()].double())
            halo[own] = _values((h, C), dt, seed, 2000 + b).double()
            g_x[own] = _row_sums(h, idx, _values((h, C), dt, seed, 3000 + b))
        return sends, halo, g_x
    n = _row_count(case)
    x = _values((n, C), dt, seed, 2)
    hptr, hcols = _halos(case, *_matrix(case, seed))
    if kind == "rank":
        rank, first, last = _the_rank(case)
        halo = x[hcols[int(hptr[rank]):int(hptr[rank + 1])].long()].double()
        if case["variant"] != "plain":  # the slots' order is the plan's own
            return (None, halo, None) if case["backward"] else (None, halo)
        # the plain plan's slots: by destination rank, then by row
        sent = hcols[(hcols >= first) & (hcols < last)].long()
        if not case["backward"]:
            return x[sent].double(), halo
        g_send = _values((int(sent.numel()), C), dt, seed, 4)
        return x[sent].double(), halo, _row_sums(last - first, sent - first, g_send)
    halo = x[hcols.long()].double()
    if kind == "setup":
        return halo, None
    if kind == "train" or case["backward"]:
        g = _values((int(hcols.numel()), C), dt, seed, 3)
        return halo, _row_sums(n, hcols, g)
    return halo
