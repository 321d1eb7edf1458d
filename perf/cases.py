"""What is timed: the work a user has this library do, over the real range.

Each case is one pass through the public entry points of
``paper_1603_06958_amd`` (the ctypes binding and the serving loop):

* ``noalloc``: one family, device sequences in and every pair's LCS out on the
  device, with no allocation (a caller inside a tight loop or a capture);
* ``tiles``: a plan that the program keeps, its tiles delivered to host memory
  (LCS, indel distances or float32 similarities);
* ``condensed``: a plan whose device tiles the program gathers into one
  condensed matrix on the device;
* ``tree``: a family's guide tree, device tiles into the GPU single-linkage
  consumer (the plan kept, or made for the family in the same pass);
* ``profile``: one level of the progressive stage, single sequences aligned to
  profiles;
* ``gapped``: the gapped representation of a profile's sequences, made, given
  gap runs twice and decoded;
* ``serve``: a mix of families through the continuous-batching server.

Sizes follow the seeded workloads in ``inputs.py`` (families of 50 to 100,000
sequences, root lengths 30 to 2,000, profile levels of widths 50 to 500) cut
to what one pass of at most a second or so allows.  Families are made here by
a vectorised form of the same recipe (a random binary tree; per edge 10%
substitutions and 2% indel events of Geometric(1/2) length), because the
workloads' own generator takes minutes at these sizes.
"""
import ctypes
import math
import zlib

import numpy as np
import torch

from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs, serve

GAP = 0xFF


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest family of a batch, inside a loop that may not allocate: launches and latency
        dict(name="noalloc_small", kind="noalloc", k=48, lo=50, hi=300, root=0, sigma=20),
        # the entry point's largest family, tree-evolved, root length 300
        dict(name="noalloc_large", kind="noalloc", k=8192, lo=0, hi=0, root=300, sigma=20),
        # 100 i.i.d. ragged sequences, empty ones among them, all 32 codes, float32 similarities on the host
        dict(name="tiles_small", kind="tiles", nfam=1, k_lo=100, k_hi=100, lo=0, hi=300, root_lo=0, root_hi=0, sigma=32,
             values="sim"),
        # many families of very different sizes and lengths (up to 2,000 residues) batched in one plan
        dict(name="tiles_batch", kind="tiles", nfam=24, k_lo=50, k_hi=1500, lo=0, hi=0, root_lo=30, root_hi=2000,
             sigma=20, values="lcs"),
        # one large family of log-normal lengths, row tile by row tile, gathered on the device
        dict(name="condensed_large", kind="condensed", k=20000, root=250, spread=0.3),
        # a small family seen once: plan, tiles and guide tree in one go
        dict(name="tree_once", kind="tree", k=300, root=250, spread=0.0, once=1, tile_rows=1024),
        # a family of short domains: many pairs, little work a pair
        dict(name="tree_short", kind="tree", k=12000, root=60, spread=0.0, once=0, tile_rows=1024),
        # a large family of log-normal lengths to its guide tree
        dict(name="tree_large", kind="tree", k=30000, root=250, spread=0.3, once=0, tile_rows=1024),
        # a full level of the progressive stage
        dict(name="profile_level", kind="profile", nprob=1200, n_lo=50, n_hi=500, K_lo=1, K_hi=200, sigma=20),
        # the top of a tree: a few wide problems, whose inputs are too large for LDS
        dict(name="profile_wide", kind="profile", nprob=6, n_lo=900, n_hi=1500, K_lo=100, K_hi=400, sigma=20),
        # the sequences of a large profile in the gapped representation
        dict(name="gapped_profile", kind="gapped", k=20000, root=250, spread=0.3, nruns=64),
        # small and middling jobs that arrive together at a server
        dict(name="serve_mix", kind="serve", njobs=16, k_lo=100, k_hi=1500, root_lo=50, root_hi=800),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "noalloc", "tiles", "tiles", "condensed", "tree", "tree", "tree", "profile", "profile",
                       "gapped", "serve"])
    if kind == "noalloc":
        k = _log_int(rng, 2, 8192)
        if rng.random() < 0.5:
            sigma = rng.choice([4, 20, 25, 32])
            hi = rng.randint(30, 896 if sigma <= 20 else 512)
            return dict(kind=kind, k=k, lo=rng.randint(0, hi), hi=hi, root=0, sigma=sigma)
        return dict(kind=kind, k=k, lo=0, hi=0, root=_log_int(rng, 30, 600), sigma=20)
    if kind == "tiles":
        values = rng.choice(["lcs", "indel", "sim"])
        if rng.random() < 0.5:
            k = _log_int(rng, 20, 1500)
            return dict(kind=kind, nfam=1, k_lo=k, k_hi=k, lo=rng.randint(0, 60), hi=rng.randint(61, 1200), root_lo=0,
                        root_hi=0, sigma=rng.choice([20, 23, 32]), values=values)
        return dict(kind=kind, nfam=rng.randint(2, 32), k_lo=rng.randint(20, 60), k_hi=rng.randint(200, 1500), lo=0, hi=0,
                    root_lo=rng.randint(30, 100), root_hi=rng.randint(300, 2000), sigma=20, values=values)
    if kind == "condensed":
        return dict(kind=kind, k=_log_int(rng, 1000, 20000), root=_log_int(rng, 60, 250), spread=rng.choice([0.0, 0.3]))
    if kind == "tree":
        once = rng.randint(0, 1)
        k = _log_int(rng, 20, 2000) if once else _log_int(rng, 200, 30000)
        return dict(kind=kind, k=k, root=_log_int(rng, 30, 250), spread=rng.choice([0.0, 0.3]), once=once,
                    tile_rows=rng.choice([257, 1024]))
    if kind == "profile":
        if rng.random() < 0.5:
            return dict(kind=kind, nprob=_log_int(rng, 20, 1200), n_lo=rng.randint(20, 60), n_hi=rng.randint(100, 500),
                        K_lo=1, K_hi=rng.randint(10, 200), sigma=rng.choice([20, 32]))
        return dict(kind=kind, nprob=rng.randint(1, 24), n_lo=rng.randint(50, 400), n_hi=rng.randint(401, 1500), K_lo=1,
                    K_hi=rng.randint(20, 400), sigma=20)
    if kind == "gapped":
        return dict(kind=kind, k=_log_int(rng, 100, 20000), root=_log_int(rng, 30, 600), spread=rng.choice([0.05, 0.3]),
                    nruns=rng.randint(1, 100))
    return dict(kind=kind, njobs=rng.randint(2, 24), k_lo=rng.randint(50, 150), k_hi=rng.randint(300, 1500),
                root_lo=rng.randint(30, 60), root_hi=rng.randint(200, 900))


# ------------------------------------------------------------------ inputs

def _sizes(case):
    """Generator of a case's sizes: every seed's inputs have the same ones."""
    return np.random.default_rng(zlib.crc32(repr(sorted((k, v) for k, v in case.items() if k != "name")).encode()))


def _gather(starts, lens):
    """Flat index of ragged pieces (start, length), back to back."""
    off = np.zeros(lens.size + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    return np.repeat(starts - off[:-1], lens) + np.arange(off[-1]), off


def _mutate(codes, off, changed, rng):
    """One tree edge for every sequence marked in `changed`."""
    n = codes.size
    lens = np.diff(off)
    on = np.repeat(changed, lens)
    u = rng.random(n, dtype=np.float32)
    codes = codes.copy()
    hit = np.flatnonzero((u < 0.10) & on)
    codes[hit] = (codes[hit] + rng.integers(1, 20, hit.size, dtype=np.uint8)) % 20
    counts = np.ones(n, np.int64)
    dele = np.flatnonzero((u > 0.99) & on)
    end = np.minimum(dele + rng.geometric(0.5, dele.size), np.repeat(off[1:], lens)[dele])
    for s, e in ((dele, end),):
        mark = np.zeros(n + 1, np.int64)
        np.add.at(mark, s, 1)
        np.add.at(mark, e, -1)
        counts[np.cumsum(mark[:-1]) > 0] = 0
    ins = np.flatnonzero((u > 0.98) & (u <= 0.99) & on)
    extra = np.zeros(n, np.int64)
    extra[ins] = rng.geometric(0.5, ins.size)
    total = counts + extra
    cs = np.zeros(n + 1, np.int64)
    np.cumsum(total, out=cs[1:])
    out = np.repeat(codes, total)
    new, _ = _gather(cs[ins] + counts[ins], extra[ins])
    out[new] = rng.integers(0, 20, new.size, dtype=np.uint8)
    return out, cs[off]


def _targets(k, root, spread, rng):
    """Log-normal lengths around a root's."""
    return np.clip(np.round(root * np.exp(spread * rng.standard_normal(k))), min(40, root), 1500).astype(np.int64)


def _family(k, root, rng, want=None):
    """k leaves of a random binary tree, trimmed or padded to lengths `want` if given: (codes uint8, offsets int64)."""
    codes = rng.integers(0, 20, root, dtype=np.uint8)
    off = np.array([0, root], np.int64)
    while off.size - 1 < k:
        n = off.size - 1
        m = min(k - n, max(1, int(0.6 * n)))
        reps = np.ones(n, np.int64)
        reps[rng.permutation(n)[:m]] = 2
        lens = np.repeat(np.diff(off), reps)
        idx, off2 = _gather(np.repeat(off[:-1], reps), lens)
        codes, off = _mutate(codes[idx], off2, np.repeat(reps == 2, reps), rng)
    if want is not None:
        lens = np.diff(off)
        keep = np.minimum(lens, want)
        src, _ = _gather(off[:-1], keep)
        new = np.zeros(k + 1, np.int64)
        np.cumsum(want, out=new[1:])
        dst, _ = _gather(new[:-1], keep)
        out = rng.integers(0, 20, new[-1], dtype=np.uint8)
        out[dst] = codes[src]
        codes, off = out, new
    return codes, off


def _random(k, lo, hi, sigma, rng):
    off = np.zeros(k + 1, np.int64)
    np.cumsum(rng.integers(lo, hi + 1, k), out=off[1:])
    return rng.integers(0, sigma, int(off[-1]), dtype=np.uint8), off


def _log_ints(rng, lo, hi, n):
    return np.round(np.exp(rng.uniform(math.log(lo), math.log(hi), n))).astype(int)


def _profile(m, n, K, sigma, rng):
    """A profile of K noisy, gapped copies of a random consensus, and a sequence near it."""
    cons = rng.integers(0, sigma, n, dtype=np.uint8)
    noise = rng.integers(0, sigma, (K, n), dtype=np.uint8)
    u = rng.random((K, n), dtype=np.float32)
    rows = np.where(u < 0.7, cons, noise)
    col = np.arange(n)
    start = rng.random((K, n), dtype=np.float32) < 0.05
    end = np.where(start, col + rng.geometric(1 / 3, (K, n)), 0)
    gap = np.maximum.accumulate(end, axis=1) > col
    lead = np.where(rng.random(K) < 0.3, rng.integers(0, n // 4 + 1, K), 0)
    trail = np.where(rng.random(K) < 0.3, rng.integers(0, n // 4 + 1, K), 0)
    gap |= (col < lead[:, None]) | (col >= n - trail[:, None])
    rows[gap] = GAP
    seq = cons[np.minimum(np.arange(m) * n // m, n - 1)].copy()
    hit = rng.random(m) < 0.1
    seq[hit] = rng.integers(0, sigma, int(hit.sum()), dtype=np.uint8)
    return seq, rows


def _batch(case, rng):
    """The families of a `tiles` case back to back: codes, sequence offsets, family offsets."""
    sizes = _sizes(case)
    ks = _log_ints(sizes, case["k_lo"], case["k_hi"], case["nfam"])
    if case["root_lo"]:
        roots = _log_ints(sizes, case["root_lo"], case["root_hi"], case["nfam"])
        fams = [_family(int(k), int(r), rng) for k, r in zip(ks, roots)]
    else:
        fams = [_random(int(k), case["lo"], case["hi"], case["sigma"], rng) for k in ks]
    codes = np.concatenate([c for c, _ in fams])
    lens = np.concatenate([np.diff(o) for _, o in fams])
    off = np.zeros(lens.size + 1, np.uint64)
    np.cumsum(lens, out=off[1:])
    fam = np.zeros(ks.size + 1, np.uint32)
    np.cumsum(ks, out=fam[1:])
    return codes, off, fam


def prepare(case, seed):
    rng, sizes = np.random.default_rng(seed), _sizes(case)
    kind = case["kind"]
    if kind in ("condensed", "tree", "gapped"):
        want = _targets(case["k"], case["root"], case["spread"], sizes) if case["spread"] else None
    if kind == "noalloc":
        if case["root"]:
            codes, off = _family(case["k"], case["root"], rng)
            lim = B.NOALLOC_MAX_LEN
            if int(np.diff(off).max()) > lim:  # keep within the entry point's length limit
                keep = np.minimum(np.diff(off), lim)
                idx, off2 = _gather(off[:-1], keep)
                codes, off = codes[idx], off2
        else:
            codes, off = _random(case["k"], case["lo"], case["hi"], case["sigma"], rng)
        k = case["k"]
        return dict(kind=kind, k=k, sigma=case["sigma"], codes=torch.from_numpy(np.append(codes, np.uint8(0))).cuda(),
                    off=torch.from_numpy(off.astype(np.int64)).cuda(),
                    out=torch.empty(k * (k - 1) // 2, dtype=torch.int32, device="cuda"),
                    status=torch.empty(1, dtype=torch.int32, device="cuda"))
    if kind == "tiles":
        codes, off, fam = _batch(case, rng)
        flags = {"lcs": 0, "indel": B.OUT_INDEL, "sim": B.OUT_SIM}[case["values"]]
        plan = B.Plan(codes, off, fam, alphabet_size=case["sigma"], flags=flags)
        return dict(kind=kind, plan=plan)
    if kind == "condensed":
        codes, off = _family(case["k"], case["root"], rng, want)
        plan = B.Plan(codes, off, flags=B.DEVICE_TILES)
        k = case["k"]
        return dict(kind=kind, plan=plan, out=torch.empty(k * (k - 1) // 2, dtype=torch.int32, device="cuda"))
    if kind == "tree":
        codes, off = _family(case["k"], case["root"], rng, want)
        st = dict(kind=kind, codes=codes, off=off.astype(np.uint64), lens=np.diff(off).astype(np.uint32),
                  tile_rows=case["tile_rows"], plan=None)
        if not case["once"]:
            st["plan"] = B.Plan(codes, st["off"], flags=B.DEVICE_TILES, tile_rows=case["tile_rows"])
        return st
    if kind == "profile":
        ns = _log_ints(sizes, case["n_lo"], case["n_hi"], case["nprob"])
        Ks = _log_ints(sizes, case["K_lo"], case["K_hi"], case["nprob"])
        ms = np.maximum(1, np.round(ns * sizes.uniform(0.85, 1.15, case["nprob"]))).astype(int)
        problems = [_profile(int(m), int(n), int(K), case["sigma"], rng) for m, n, K in zip(ms, ns, Ks)]
        return dict(kind=kind, problems=problems, room=int((ms + ns).sum()), subst=inputs.synthetic_subst(case["sigma"], 7),
                    costs=B.gap_costs_scaled(1000, (2.0, 1.0, 12.0, 1.0)))
    if kind == "gapped":
        codes, off = _family(case["k"], case["root"], rng, want)
        lens = np.diff(off)
        runs = []
        width = int(lens.min())
        for _ in range(2):  # columns of the narrowest sequence before each round
            col = np.sort(rng.integers(1, width + 2, case["nruns"])).astype(np.uint32)
            ln = sizes.geometric(1 / 3, case["nruns"]).astype(np.uint32)
            runs.append((col, ln))
            width += int(ln.sum())
        return dict(kind=kind, codes=codes, off=off.astype(np.uint64), runs=runs)
    ks = _log_ints(sizes, case["k_lo"], case["k_hi"], case["njobs"])
    roots = _log_ints(sizes, case["root_lo"], case["root_hi"], case["njobs"])
    jobs = []
    for k, r in zip(ks, roots):
        codes, off = _family(int(k), int(r), rng)
        jobs.append((codes, off.astype(np.uint64)))
    return dict(kind=kind, jobs=jobs, server=serve.Server(tile_rows=256, step_values=1 << 24, step_cells=1 << 41))


# ------------------------------------------------------------------ one pass

class _DeviceArray:
    """int32 device memory at an address, for torch."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = dict(shape=(n,), typestr="<i4", data=(ptr, False), version=3, strides=None)


def run(state):
    kind = state["kind"]
    if kind == "noalloc":
        B.family_noalloc(state["codes"].data_ptr(), state["off"].data_ptr(), state["k"], state["out"].data_ptr(),
                         state["status"].data_ptr(), alphabet_size=state["sigma"],
                         stream=torch.cuda.current_stream().cuda_stream)
        return state["out"], state["status"]
    if kind == "tiles":
        tiles = state["plan"].collect()
        return list(tiles.values())
    if kind == "condensed":
        out, at = state["out"], [0]
        cur = torch.cuda.current_stream()

        def gather(t):
            n = int(t.count)
            if n:
                s = torch.cuda.ExternalStream(t.stream)
                s.wait_stream(cur)
                with torch.cuda.stream(s):
                    src = torch.as_tensor(_DeviceArray(ctypes.cast(t.lcs, ctypes.c_void_p).value, n), device="cuda")
                    out[at[0]:at[0] + n].copy_(src)
                cur.wait_stream(s)
            at[0] += n
            return 0

        state["plan"].run(gather)
        return out
    if kind == "tree":
        plan = state["plan"] or B.Plan(state["codes"], state["off"], flags=B.DEVICE_TILES, tile_rows=state["tile_rows"])
        mst = B.Mst(state["lens"])
        plan.run_native(B.Mst.consume_fn(), mst.handle)
        tree = mst.guide_tree()
        mst.close()
        if state["plan"] is None:
            plan.close()
        return tree
    if kind == "profile":
        score, ops = B.profile_align(state["problems"], state["subst"], state["costs"])
        path = np.full(state["room"], GAP, np.uint8)  # every problem's alignment, back to back
        cat = np.concatenate(ops)
        path[:cat.size] = cat
        return score, path, np.array([o.size for o in ops])
    if kind == "gapped":
        g = B.Gapped(state["codes"], state["off"])
        for col, ln in state["runs"]:
            g.insert(col, ln)
        width, rows = g.width(), g.decode()
        g.close()
        return width, rows
    srv, got = state["server"], {}

    def take(t):
        got.setdefault(int(t.family), []).append(B.tile_array(t).copy())
        return 0

    ids = [srv.submit(c, o) for c, o in state["jobs"]]
    while srv.step(take):
        pass
    return [np.concatenate(got[i]) for i in ids]


# ------------------------------------------------------------------ its cost

def work(case):
    """Bytes and operations of a pass that nothing can do without, at the case's nominal sizes: 3 operations per 32 cells
    of a pair's LCS matrix, 20 per cell of a profile DP; inputs read and outputs written once."""
    kind = case["kind"]

    def mean_log(lo, hi, p=1):  # E[x^p] of a log-uniform size
        return float(lo) ** p if hi <= lo else (hi ** p - lo ** p) / (p * math.log(hi / lo))

    def lcs(k, L1, L2):  # pairs and operations of a family of mean length L1 (mean square of a pair L2)
        pairs = k * (k - 1) / 2
        return pairs, pairs * L2 * 3 / 32, k * (L1 + 8)

    if kind == "noalloc":
        L = case["root"] or (case["lo"] + case["hi"]) / 2
        pairs, ops, inb = lcs(case["k"], L, L * L)
        return {"bytes": inb + 4 * pairs, "flops": ops}
    if kind == "tiles":
        k1, k2 = mean_log(case["k_lo"], case["k_hi"]), mean_log(case["k_lo"], case["k_hi"], 2)
        if case["root_lo"]:
            L1, L2 = mean_log(case["root_lo"], case["root_hi"]), mean_log(case["root_lo"], case["root_hi"], 2)
        else:
            L1 = (case["lo"] + case["hi"]) / 2
            L2 = L1 * L1
        pairs = case["nfam"] * (k2 - k1) / 2
        return {"bytes": case["nfam"] * k1 * (L1 + 8) + 4 * pairs, "flops": pairs * L2 * 3 / 32}
    if kind == "condensed":
        pairs, ops, inb = lcs(case["k"], case["root"], case["root"] ** 2)
        return {"bytes": inb + 4 * pairs, "flops": ops}
    if kind == "tree":
        pairs, ops, inb = lcs(case["k"], case["root"], case["root"] ** 2)
        return {"bytes": inb + 24 * case["k"], "flops": ops + pairs}
    if kind == "profile":
        n1, n2 = mean_log(case["n_lo"], case["n_hi"]), mean_log(case["n_lo"], case["n_hi"], 2)
        K = mean_log(case["K_lo"], case["K_hi"])
        return {"bytes": case["nprob"] * (n1 * (K + 3) + 16), "flops": case["nprob"] * 20 * n2}
    if kind == "gapped":
        k, n = case["k"], case["root"]
        return {"bytes": k * (n + 8) + k * (n + 6 * case["nruns"]), "flops": k * (n + 2 * case["nruns"])}
    k1, k2 = mean_log(case["k_lo"], case["k_hi"]), mean_log(case["k_lo"], case["k_hi"], 2)
    L1, L2 = mean_log(case["root_lo"], case["root_hi"]), mean_log(case["root_lo"], case["root_hi"], 2)
    pairs = case["njobs"] * (k2 - k1) / 2
    return {"bytes": case["njobs"] * k1 * (L1 + 8) + 4 * pairs, "flops": pairs * L2 * 3 / 32}


# ------------------------------------------------------------------ the values in 64 bits

def _lcs(a, mask, b):
    """LCS length of a (as bit masks per code) and b by a big-integer bit vector."""
    full = (1 << a) - 1
    V = full
    for c in b:
        U = V & mask[c]
        V = ((V + U) | (V - U)) & full
    return a - V.bit_count() if hasattr(V, "bit_count") else a - bin(V).count("1")


def exact(case, seed):
    """Float64 similarities LCS / indel^2 of the small families that return them; every other output is whole numbers."""
    if case["kind"] != "tiles" or case["values"] != "sim" or case["nfam"] * case["k_hi"] ** 2 > 120 ** 2:
        return None
    rng = np.random.default_rng(seed)
    codes, off, fam = _batch(case, rng)
    out = []
    for f in range(fam.size - 1):
        seqs = [codes[int(off[i]):int(off[i + 1])].tolist() for i in range(int(fam[f]), int(fam[f + 1]))]
        vals = []
        for i, a in enumerate(seqs):
            mask = [0] * 32
            for p, c in enumerate(a):
                mask[c] |= 1 << p
            for b in seqs[i + 1:]:
                lcs = _lcs(len(a), mask, b)
                d = len(a) + len(b) - 2 * lcs
                vals.append(lcs / float(d * d) if d else math.inf)
        out.append(np.array(vals, np.float64))  # k_hi <= 120: one tile a family
    return out
