"""Timed cases of the FCIQMC projector: what a user's program runs on one GPU.

A case is one call pattern of the package (a solver, replicas, excited-state
runs, a batch, a server, a checkpoint and resume) at one size.  `prepare`
builds the solver and grows the walker population to its target, so that a
pass starts from a populated vector with the shift in control; `run` advances
it and returns the statistics rows (and, where the vector is small, the vector
itself in address order).  The seed of a case is the seed of the counter-based
generator: another seed is another trajectory from the first step on.

Systems are those of the Bose-Hubbard examples, tests and benchmark of this
repository: the ring in real space, momentum space, and the periodic square
lattice with Gutzwiller importance sampling.
"""
import math

import numpy as np

import paper_2601_19505_amd as fq

RING, MOM, LATTICE = "ring", "momentum", "lattice"
MODELS = {RING: fq.REAL1D, MOM: fq.MOM1D, LATTICE: fq.REAL2D}

# the hash and tile shapes of the benchmark's large runs; 0 is the library's choice
TUNED = dict(lds_slots=2048, block=512, spawn_block=256)
DEFAULT = dict(lds_slots=0, block=0, spawn_block=0)

# a populated vector of small systems is returned with the rows
STATE_UP_TO = 20_000
YREF = 10.0


def _case(name, kind, model, M, target, steps, **more):
    case = dict(kind=kind, model=model, M=M, N=M, lx=0, t=1.0, u=6.0, g=0.0, dtau=1e-3, target=float(target),
                words=1, grow=400, steps=steps, instances=1, buckets=0, table=0, spawn=0, early=False,
                initiator=-1.0)
    case.update(DEFAULT if target <= 20_000 else TUNED)
    case.update(more)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # a first experiment on a laptop-sized system: the 6/6 ring at 1e3 walkers, hundreds of short steps
        _case("ring6", "solver", RING, 6, 1e3, 500, table=1024, spawn=8192),
        # the variational energy from two replicas of a small momentum-space system
        _case("replicas_mom8", "replicas", MOM, 8, 1e3, 300, u=4.0, instances=2),
        # the published accuracy run: the 12/12 ring at 1e5 walkers
        _case("ring12", "solver", RING, 12, 1e5, 100),
        # the same ring under early compression, as in a study of compression efficiency
        _case("ring12_early", "solver", RING, 12, 1e4, 100, early=True, grow=200),
        # a system with a sign problem under the initiator rule
        _case("mom16_initiator", "solver", MOM, 16, 1e6, 50, u=4.0, dtau=5e-4, initiator=3.0, grow=600,
              table=1_000_000, spawn=4_000_000),
        # ground and first excited state of the 12/12 ring
        _case("excited_ring12", "spectral", RING, 12, 1e5, 50, dtau=2e-3, instances=2),
        # the 20/20 ring with two-word addresses at 1e7 walkers
        _case("ring20", "solver", RING, 20, 1e7, 30, words=2, buckets=16384, table=12_000_000, spawn=40_000_000,
              grow=700),
        # the published benchmark system: the 6 x 6 lattice, importance sampled, 1e7 walkers
        _case("lattice6x6", "solver", LATTICE, 36, 1e7, 30, lx=6, t=0.1, u=1.0, g=1.0, dtau=1.5e-3, words=2,
              buckets=16384, table=30_000_000, spawn=60_000_000, grow=1500),
        # the headline run: momentum space, 16/16, 1e8 walkers
        _case("mom16", "solver", MOM, 16, 1e8, 40, u=4.0, dtau=5e-4, buckets=16384, table=19_500_000,
              spawn=200_000_000, grow=1300),
        # a scan of the interaction strength: many rings stepped together
        _case("batch_ring10", "batch", RING, 10, 1e4, 100, instances=32, **TUNED),
        # a service that solves a burst of small requests to the end
        _case("server_ring8", "server", RING, 8, 3e3, 500, instances=8, lds_slots=1024, block=256, spawn_block=256),
        # checkpoint of a running solve, and its continuation in another solver
        _case("resume_ring16", "resume", RING, 16, 1e6, 10),
    ]


def draw(rng):
    """One more case: the models over their range of sizes and walker numbers,
    the compression styles, the initiator rule, and the ways to run them."""
    kind = rng.choice(["solver"] * 6 + ["replicas", "replicas", "spectral", "batch", "server", "resume"])
    # the server runs the ring and momentum space; excited states are a real-space method here
    model = rng.choice({"server": [RING, MOM], "spectral": [RING, LATTICE]}.get(kind, [RING, MOM, LATTICE]))
    top = {"solver": 7.0, "replicas": 6.5, "spectral": 5.0, "batch": 4.5, "server": 4.0, "resume": 6.0}[kind]
    target = float(round(10 ** rng.uniform(3.0, top)))
    # the basis must be able to hold the population
    least = 6 if target < 1e4 else 9 if target < 1e5 else 12 if target < 1e6 else 14
    instances = {"replicas": rng.choice([2, 3]), "spectral": 2, "batch": rng.randint(3, 48),
                 "server": rng.randint(2, 12)}.get(kind, 1)
    more = dict(u=round(rng.uniform(1.0, 8.0), 2), instances=instances)
    if model == LATTICE:
        lx = rng.randint(2, 6)
        M = lx * max(2, -(-least // lx) + rng.randint(0, 1))
        more.update(lx=lx, t=0.1, u=1.0, g=rng.choice([0.0, 0.5, 1.0]))
        width = 0.5 * M * (M - 1) + 0.8 * M
    elif model == MOM:
        M = rng.randint(least, 15 if kind == "server" else 18)
        more["u"] = round(rng.uniform(1.0, 4.0), 2)
        width = 0.5 * more["u"] * M * (M - 1) + 4 * M
    else:
        M = rng.randint(least, 24)
        width = 0.5 * more["u"] * M * (M - 1) + 4 * M
    more["dtau"] = min(5e-4 if model == MOM else 2e-3 if kind == "spectral" else 1e-3, 1.0 / width)
    more["words"] = 2 if 2 * M - 1 > 62 or (kind != "server" and rng.random() < 0.2) else 1
    if kind in ("solver", "resume"):
        option = rng.choice(["", "", "early", "initiator"])
        more["early"] = option == "early"
        more["initiator"] = rng.choice([1.0, 3.0, 10.0]) if option == "initiator" else -1.0
    if kind == "server":
        more.update(lds_slots=1024, block=256, spawn_block=256)
    elif kind == "spectral" or kind == "batch":
        more.update(TUNED)
    steps = int(min(rng.randint(100, 300) // (2 if instances > 1 else 1), max(10, (1e8 if model == MOM else 2e8) / target / instances)))
    if kind == "server":
        steps = rng.randint(200, 800)
    elif kind == "resume":
        steps = 10
    return _case("", kind, model, M, target, steps, **more)


# ------------------------------------------------------------------ the framework's side


def _dimension(case):
    return math.comb(case["N"] + case["M"] - 1, case["N"])


def _spec(case, seed, k):
    """Keyword arguments of instance k; a batch scans u."""
    target = case["target"]
    # a sign problem lets the population overshoot while it grows
    room = 4.0 if case["model"] == MOM else 3.0
    u = case["u"]
    if case["kind"] in ("batch", "server"):
        u = round(u * (0.25 + 0.75 * (k + 1) / case["instances"]), 4)
    spec = dict(model=MODELS[case["model"]], M=case["M"], N=case["N"], t=case["t"], u=u, dtau=case["dtau"],
                target_walkers=target, seed=seed * 1000 + k, addr_words=case["words"],
                flags=fq.FLAG_EARLY_COMPRESSION if case["early"] else 0, lx=case["lx"], g=case["g"],
                initiator=None if case["initiator"] < 0 else case["initiator"],
                table_capacity=case["table"] or int(min(_dimension(case), room * target)) + 4096,
                spawn_capacity=case["spawn"] or int(2 * room * target) + 65536, buckets=case["buckets"],
                lds_slots=case["lds_slots"], block=case["block"], spawn_block=case["spawn_block"])
    return spec


def _occupations(case, k):
    """Start of instance k: the uniform state (the condensate in momentum
    space); excited-state runs after the first start one hop away."""
    M, N = case["M"], case["N"]
    if case["model"] == MOM:
        occ = [N] + [0] * (M - 1)
        if case["kind"] == "spectral" and k:
            occ[0], occ[1], occ[M - 1] = N - 2, 1, 1
        return occ
    occ = [N // M + (1 if j < N % M else 0) for j in range(M)]
    if case["kind"] == "spectral" and k:
        occ[0], occ[1] = occ[0] - 1, occ[1] + 1
    return occ


def _walkers(case):
    """On the start address: a hundredth of the target, so that the growth is short."""
    return 10.0 if case["kind"] == "server" else max(10.0, case["target"] / 100)


def _place(solver, case, k):
    a = fq.encode(_occupations(case, k), case["words"])
    solver.set_state([a], [_walkers(case)], 0.0, 0, ref=a, yref=YREF)


def prepare(case, seed):
    kind = case["kind"]
    specs = [_spec(case, seed, k) for k in range(case["instances"])]
    if kind == "server":
        sv = fq.Server(MODELS[case["model"]], int(2e9), addr_words=case["words"], lds_slots=case["lds_slots"],
                       block=case["block"], spawn_block=case["spawn_block"], max_active=64, steps_per_tick=250)
        start = fq.encode(_occupations(case, 0), case["words"])
        return dict(case=case, server=sv, specs=specs, start=start)
    if kind in ("solver", "resume"):
        solver = fq.Solver(**specs[0])
        _place(solver, case, 0)
        solver.run(case["grow"])
        state = dict(case=case, solver=solver)
        if kind == "resume":
            state["other"] = fq.Solver(**specs[0])
        return state
    batch = fq.Batch(specs)
    for k in range(case["instances"]):
        _place(batch.instance(k), case, k)
    if kind == "replicas":
        batch.run_replicas(case["grow"])
    elif kind == "spectral":
        batch.run_spectral(case["grow"])
    else:
        batch.run(case["grow"])
    return dict(case=case, batch=batch)


def _rows(stats):
    return {name: np.ascontiguousarray(stats[name]) for name in stats.dtype.names}


def _ordered(case, a, v):
    """The vector in address order, in arrays of the most entries it may have."""
    most, order = _spec(case, 0, 0)["table_capacity"], np.lexsort(a.T)
    addresses, values = np.zeros((most, a.shape[1]), np.int64), np.zeros(most)
    addresses[:len(v)], values[:len(v)] = a[order].view(np.int64), v[order]
    return dict(addresses=addresses, values=values)


def run(state):
    case = state["case"]
    kind, steps = case["kind"], case["steps"]
    if kind == "solver":
        out = dict(rows=_rows(state["solver"].run(steps)))
        if case["target"] <= STATE_UP_TO:
            a, v, _, _ = state["solver"].get_state()
            out["vector"] = _ordered(case, a, v)
        return out
    if kind == "resume":
        a, v, shift, step = state["solver"].get_state()
        start = fq.encode(_occupations(case, 0), case["words"])
        state["other"].set_state(a, v, shift, step, ref=start, yref=YREF)
        return dict(rows=_rows(state["other"].run(steps)))
    if kind == "server":
        sv = state["server"]
        ids = [sv.submit({k: v for k, v in sp.items() if k not in ("lds_slots", "block", "spawn_block")},
                         state["start"], 10.0, steps + 37 * k) for k, sp in enumerate(state["specs"])]
        while True:
            active, queued, _ = sv.tick()
            if not active and not queued:
                break
        got = [sv.poll(i) for i in ids]
        keys = ("state", "steps_done", "mean_shift", "mean_hproj", "mean_vproj", "n_mean", "walker_steps")
        out = {k: np.array([g[k] for g in got]) for k in keys}
        out["last"] = {k: np.array([g["last"][k] for g in got]) for k in got[0]["last"]}
        return out
    batch = state["batch"]
    if kind == "replicas":
        stats, overlaps, _ = batch.run_replicas(steps)
        return dict(rows=_rows(stats), overlaps=overlaps)
    if kind == "spectral":
        stats, _ = batch.run_spectral(steps)
        return dict(rows=_rows(stats))
    return dict(rows=_rows(batch.run(steps)))


def work(case):
    """Per step: the vector read and written once and every spawn event
    exchanged once (written and read); floating-point work of the diagonal,
    the spawned values and the sums.  Entries and events per walker are
    measured averages of the populated systems."""
    entries, events = {RING: (0.85, 1.15), MOM: (0.16, 0.9), LATTICE: (1.0, 1.05)}[case["model"]]
    entries = min(entries * case["target"], _dimension(case))
    events = events * case["target"] * (0.05 if case["early"] else 1.0)
    n = case["instances"] * case["steps"]
    return dict(bytes=n * (8 * case["words"] + 8) * 2 * (entries + events),
                flops=n * (entries * (2 * case["M"] + 6) + events * 6))


# ------------------------------------------------------------------ the same numbers in plain numpy


def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 of counter arrays (uint64 holding 32-bit words) under key."""
    low = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)
    c0, c1, c2, c3 = (np.asarray(c, np.uint64) & low for c in (c0, c1, c2, c3))
    k0, k1 = np.asarray(key, np.uint64) & low, np.asarray(key, np.uint64) >> s32
    for _ in range(10):
        p, q = np.uint64(0xD2511F53) * c0, np.uint64(0xCD9E8D57) * c2
        c0, c1, c2, c3 = (q >> s32) ^ c1 ^ k0, q & low, (p >> s32) ^ c3 ^ k1, p & low
        k0, k1 = (k0 + np.uint64(0x9E3779B9)) & low, (k1 + np.uint64(0xBB67AE85)) & low
    return np.stack([c0, c1, c2, c3], 1)


class _Plain:
    """One FCIQMC run over occupation numbers, sums rounded once (fsum)."""

    def __init__(self, case, spec, start):
        self.c, self.s = case, spec
        self.M, self.N = case["M"], case["N"]
        self.ref = tuple(start)
        self.occ = np.array([start], np.int64)
        self.val = np.array([_walkers(case)])
        self.shift, self.step = 0.0, 0
        self.norm = abs(float(self.val[0]))
        lx = case["lx"] or self.M
        x, y = np.arange(self.M) % lx, np.arange(self.M) // lx
        ly = self.M // lx
        hops = [(x + 1) % lx + lx * y, (x - 1) % lx + lx * y]
        if case["model"] == LATTICE:
            hops += [x + lx * ((y + 1) % ly), x + lx * ((y - 1) % ly)]
        self.hops = np.array(hops)
        self.eps = np.array([(-2.0 * case["t"]) * math.cos((2.0 * math.pi * j) / self.M) for j in range(self.M)])

    def words(self, occ):
        """Address words: the i-th boson, in mode m, is bit i + m."""
        end = np.cumsum(occ, 1)
        bit = np.arange(self.N) + (end[:, None, :] <= np.arange(self.N)[None, :, None]).sum(2)
        w = [np.where((bit >> 6) == k, np.uint64(1) << (bit & 63).astype(np.uint64), np.uint64(0)).sum(1, dtype=np.uint64)
             for k in (0, 1)]
        return w[0], w[1]

    def draws(self, occ, step, tag, block):
        a0, a1 = self.words(occ)
        return _philox(a0, a0 >> np.uint64(32), (np.asarray(tag, np.uint64) << np.uint64(28)) | np.asarray(block, np.uint64),
                       np.full(len(occ), step, np.uint64), np.uint64(self.s["seed"]) ^ a1)

    def diagonal(self, occ):
        u = self.s["u"]
        if self.c["model"] != MOM:
            return (0.5 * u) * (occ * (occ - 1)).sum(1).astype(float)
        kin = np.zeros(len(occ))
        for j in range(self.M):
            kin = kin + self.eps[j] * occ[:, j]
        return kin + (u / (2.0 * self.M)) * (2 * self.N * self.N - self.N - (occ * occ).sum(1)).astype(float)

    def hop(self, occ, k, row=False):
        """Entry k of the columns of occ (the rows when `row`) in real space."""
        n, o = len(occ), (occ > 0).sum(1)
        way = k // o
        src = (np.cumsum(occ > 0, 1) == (k - way * o + 1)[:, None]).argmax(1)
        dst = self.hops[way, src]
        at = np.arange(n)
        ns, nd = occ[at, src], occ[at, dst]
        h = (-self.c["t"]) * np.sqrt((ns * (nd + 1)).astype(float))
        if self.c["model"] == LATTICE:
            h = h * np.exp(-((self.c["g"] * self.s["u"]) * ((nd - ns + 1) * (-1.0 if row else 1.0))))
        d = occ.copy()
        d[at, src] -= 1
        d[at, dst] += 1
        return d, h

    def scatter(self, occ, p, q, r, s):
        """Momentum-space move {p, q} -> {r, s} of every row."""
        at = np.arange(len(occ))
        A = occ[at, p] * (occ[at, q] - (p == q))
        B = (occ[at, r] + 1) * (occ[at, s] + 1 + (r == s))
        cc = np.where(p == q, 1, 2) * np.where(r == s, 1, 2)
        h = (self.s["u"] / (2.0 * self.M) * cc) * (np.sqrt(A.astype(float)) * np.sqrt(B.astype(float)))
        d = occ.copy()
        for x, sign in ((p, -1), (q, -1), (r, 1), (s, 1)):
            np.add.at(d, (at, x), sign)
        return d, h

    def targets(self, p, q):
        """Destination pairs of every removal pair: arrays (n, most) and their number."""
        M = self.M
        K = (p + q) % M
        r = np.arange(M)[None, :]
        ok = (r <= K[:, None] // 2) | ((r > K[:, None]) & (r <= (K[:, None] + M) // 2))
        ok &= r != np.where(p <= K // 2, p, np.where(p > K, p, q))[:, None]
        return K, ok

    def column(self, one):
        """All off-diagonal entries of one column (of its row, for the projected energy)."""
        occ = np.array([one], np.int64)
        o = np.flatnonzero(occ[0])
        if self.c["model"] != MOM:
            m = len(self.hops) * len(o)
            return np.repeat(occ, m, 0), np.arange(m)
        p, q, r, s = [], [], [], []
        for i, x in enumerate(o):
            for y in o[i:]:
                if x == y and one[x] < 2:
                    continue
                K, ok = self.targets(np.array([x]), np.array([y]))
                for z in np.flatnonzero(ok[0]):
                    p.append(x), q.append(y), r.append(z), s.append((K[0] - z) % self.M)
        return np.repeat(occ, len(p), 0), np.array([p, q, r, s], np.int64).reshape(4, -1)

    def sizes(self, occ):
        o = (occ > 0).sum(1)
        if self.c["model"] != MOM:
            return len(self.hops) * o
        pairs = o * (o - 1) // 2 + (occ > 1).sum(1)
        if self.M & 1:
            return pairs * ((self.M - 1) // 2)
        odd = (occ[:, 1::2] > 0).sum(1)
        return pairs * (self.M // 2) - odd * (o - odd)

    def spawns(self):
        """Events of the next step: destinations, values, initiator marks, and the parents' two counts."""
        occ, c, dt, nxt = self.occ, self.val, self.c["dtau"], self.step + 1
        m = self.sizes(occ)
        full = np.abs(c) >= m
        D, V, P, A = [], [], [], []
        for i in np.flatnonzero(full):
            rep, k = self.column(occ[i])
            if len(rep):
                d, h = self.scatter(rep, *k) if self.c["model"] == MOM else self.hop(rep, k)
                D.append(d), V.append((-(dt * h)) * c[i]), P.append(np.full(len(d), i)), A.append(np.arange(len(d)))
        part = np.flatnonzero(~full)
        if len(part):
            n = np.ceil(np.abs(c[part])).astype(np.int64)
            i = np.repeat(part, n)
            k = np.arange(len(i)) - np.repeat(np.cumsum(n) - n, n)
            par, ci, ni = occ[i], c[i], np.repeat(n, n).astype(float)
            at = np.arange(len(i))
            big = np.uint64(32)
            if self.c["model"] != MOM:
                w = self.draws(par, nxt, 0, k >> 2)[at, k & 3]
                d, h = self.hop(par, ((w * m[i].astype(np.uint64)) >> big).astype(np.int64))
                v = ((-(dt * h)) * ci) * (m[i].astype(float) / ni)
            else:
                w = self.draws(par, nxt, 0, k >> 1)
                w0, w1 = w[at, 2 * (k & 1)], w[at, 2 * (k & 1) + 1]
                o, two = (par > 0).sum(1), (par > 1).sum(1)
                pairs = o * (o - 1) // 2 + two
                t = ((w0 * pairs.astype(np.uint64)) >> big).astype(np.int64)
                same = t < two
                t2 = np.where(same, 0, t - two)
                j = ((1 + np.sqrt(1.0 + 8.0 * t2)) / 2).astype(np.int64)
                lo = t2 - j * (j - 1) // 2
                cum1, cum2 = np.cumsum(par > 0, 1), np.cumsum(par > 1, 1)
                p = np.where(same, (cum2 == (t + 1)[:, None]).argmax(1), (cum1 == (lo + 1)[:, None]).argmax(1))
                q = np.where(same, p, (cum1 == (j + 1)[:, None]).argmax(1))
                K, ok = self.targets(p, q)
                R = ok.sum(1)
                e = ((w1 * R.astype(np.uint64)) >> big).astype(np.int64)
                r = (np.cumsum(ok, 1) == (e + 1)[:, None]).argmax(1)
                d, h = self.scatter(par, p, q, r, (K - r) % self.M)
                v = ((-(dt * h)) * ci) * ((pairs * R).astype(float) / ni)
            D.append(d), V.append(v), P.append(i), A.append(k)
        if not D:
            D, V, P, A = [occ[:0]], [c[:0]], [np.zeros(0, np.int64)], [np.zeros(0, np.int64)]
        D, V, P, A = (np.concatenate(x) for x in (D, V, P, A))
        if self.c["early"]:
            r = self.draws(occ[P], nxt, 4, A)[:, 0]
            V = self.compress(V, r)
            D, V, P = D[V != 0], V[V != 0], P[V != 0]
        return D, V, np.abs(c[P]) > self.c["initiator"], int(full.sum()), int((~full).sum())

    @staticmethod
    def compress(w, r):
        return np.where(np.abs(w) >= 1.0, w, np.where(r * 2.0 ** -32 < np.abs(w), np.sign(w), 0.0))

    def advance(self):
        nxt = self.step + 1
        D, V, strong, n_full, n_part = self.spawns()
        events = len(V)
        w = self.val * (1.0 + self.c["dtau"] * (self.shift - self.diagonal(self.occ)))
        if self.c["early"]:
            w = self.compress(w, self.draws(self.occ, nxt, 2, 0)[:, 0])
        held = set(map(tuple, self.occ.tolist())) if self.c["initiator"] >= 0 else None
        sums = {}
        for key, x in zip(map(tuple, self.occ.tolist()), w.tolist()):
            sums[key] = [x]
        for key, x, ok in zip(map(tuple, D.tolist()), V.tolist(), strong.tolist()):
            if held is None or ok or key in held:
                sums.setdefault(key, []).append(x)
        occ = np.array(list(sums), np.int64).reshape(-1, self.M)
        val = np.array([math.fsum(x) for x in sums.values()])
        if not self.c["early"]:
            val = self.compress(val, self.draws(occ, nxt, 1, 0)[:, 0])
        self.occ, self.val = occ[val != 0], val[val != 0]
        norm = math.fsum(np.abs(self.val).tolist())
        # the projected energy
        now = dict(zip(map(tuple, self.occ.tolist()), self.val.tolist()))
        rep, k = self.column(self.ref)
        d, h = self.scatter(rep, *k) if self.c["model"] == MOM else self.hop(rep, k, row=True)
        terms = [YREF * (float(self.diagonal(np.array([self.ref]))[0]) * now.get(self.ref, 0.0))]
        terms += [YREF * (x * now.get(key, 0.0)) for key, x in zip(map(tuple, d.tolist()), h.tolist())]
        dt, zeta = self.c["dtau"], 0.08
        self.shift = (self.shift - zeta / dt * math.log(norm / self.norm)) - (zeta * zeta / 4) / dt * math.log(
            norm / self.c["target"])
        row = (nxt, len(self.val), n_full, n_part, events, self.shift, norm, math.fsum(terms),
               YREF * now.get(self.ref, 0.0), 0)
        self.step, self.norm, self.now = nxt, norm, now
        return row


def exact(case, seed):
    """Rows, overlaps and vector of a small solver or replica set, computed
    over occupation numbers; None for larger ones and for the other kinds."""
    size = case["target"] * (case["grow"] + case["steps"]) * case["instances"]
    if case["kind"] not in ("solver", "replicas") or size > (1.5e6 if case["model"] == MOM else 3.2e6):
        return None
    if case["early"] and case["model"] == MOM:
        return None
    runs = [_Plain(case, _spec(case, seed, k), _occupations(case, k)) for k in range(case["instances"])]
    rows = [[] for _ in runs]
    overlaps = []
    for n in range(case["grow"] + case["steps"]):
        got = [r.advance() for r in runs]
        if n < case["grow"]:
            continue
        for k, row in enumerate(got):
            rows[k].append(row)
        overlaps.append([math.fsum(x * b.now[key] for key, x in a.now.items() if key in b.now)
                         for i, a in enumerate(runs) for b in runs[i + 1:]])
    stats = np.array([[tuple(x) for x in r] for r in rows], dtype=fq.STATS_DTYPE)
    if case["kind"] == "replicas":
        return dict(rows=_rows(stats), overlaps=np.array(overlaps))
    out = dict(rows=_rows(stats[0]))
    if case["target"] <= STATE_UP_TO:
        w0, w1 = runs[0].words(runs[0].occ)
        a = np.stack([w0, w1][:case["words"]], 1)
        out["vector"] = _ordered(case, a, runs[0].val)
    return out
