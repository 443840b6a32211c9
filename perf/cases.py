"""Performance cases of the simulator: the calls that its users make, over the
sizes they make them at, each with its inputs, one pass through the public
entry points, the work that pass cannot do without, and a plain 64-bit
evaluation of the computed numbers.

Families ("kind" of a case):
  rounds   run_rounds (and the decoder, where the logical error rate is what
           is wanted): whole trajectories of one job
  batch    run_batch: many small-distance trajectories with parameters of
           their own
  gates    a noisy stabilizer circuit applied gate by gate to a register,
           ending in the measurement and reset of the ancilla
  fused    dense k-qubit matrices on a register
  serving  a burst of mixed jobs through the job server
"""
import math

import numpy as np
import torch

import paper_2204_11404_amd as qs

_FLAGS = ("xbasis", "idle", "twirl", "virtual_z", "zz_plaquette")


def _rounds(name, d, gateset, rounds, n_traj, dtype, p, eps=0.0, theta=0.0, zeta=0.0, p1=False, states=False,
            decode=False, flag=""):
    c = dict(kind="rounds", d=d, gateset=gateset, rounds=rounds, n_traj=n_traj, dtype=dtype, p=p, eps=eps,
             theta=theta, zeta=zeta, p1=p1, states=states, decode=decode, flag=flag)
    return dict(c, name=name) if name else c


def _batch(name, d, gateset, n_traj, dtype, max_rounds, ragged, eps=0.0, theta=0.0, zeta=0.0):
    c = dict(kind="batch", d=d, gateset=gateset, n_traj=n_traj, dtype=dtype, max_rounds=max_rounds, ragged=ragged,
             eps=eps, theta=theta, zeta=zeta)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: four trajectories of a d=3 code with everything
        # asked for (the library's own smoke check); latency and launches
        _rounds("smoke_d3_c128", 3, "cr", 2, 4, "c128", 0.02, eps=0.02, zeta=0.01, p1=True, states=True),
        # a study of final registers at d=4: X-basis memory with crosstalk,
        # probabilities and registers back on the host
        _rounds("xbasis_d4_c128", 4, "cr", 3, 6, "c128", 0.01, theta=0.05, zeta=0.01, p1=True, states=True,
                flag="xbasis"),
        # the small code's curve of a threshold plot: logical error rate at
        # d=3, one point's chunk of trajectories, decoded
        _rounds("sweep_d3_c64", 3, "cr", 5, 500, "c64", 2e-3, eps=0.02, decode=True),
        # the paper's experiment: logical error rate at d=5, five rounds,
        # coherent over-rotation c = 0.5, decoded
        _rounds("sweep_d5_c64", 5, "cr", 5, 8, "c64", 2e-3, eps=0.5 * math.sqrt(2e-3), decode=True),
        # the same register in double precision, angles per gate site,
        # probabilities wanted
        _rounds("coherent_d5_c128", 5, "cr", 5, 2, "c128", 1e-3, theta=0.05, p1=True),
        # the benchmark's workload: d=5 with ZZ crosstalk between data qubits
        _rounds("crosstalk_d5_c128", 5, "cr", 5, 2, "c128", 1e-3, theta=0.05, zeta=0.01, p1=True),
        # the textbook circuit at d=3, 1000 equal trajectories in one launch
        _batch("textbook_d3_c128", 3, "textbook", 1000, "c128", 3, False, eps=0.02),
        # large batched launches of ragged small-distance trajectories
        _batch("batch_d3_c64", 3, "cr", 65536, "c64", 9, True, theta=0.05),
        _batch("batch_d4_c64", 4, "cr", 4096, "c64", 9, True, theta=0.05),
        # a noise model outside the built-in family: one stabilizer circuit
        # gate by gate on 26 qubits, measured and reset
        dict(kind="gates", n=26, dtype="c128", gates=6, name="gates_n26_c128"),
        # runs of gates multiplied into dense matrices on the host
        dict(kind="fused", n=26, dtype="c64", k=5, low=True, name="fused_n26_c64"),
        # a burst of mixed jobs as a service sees them
        dict(kind="serving", jobs=24, big=2, name="serving_burst"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rounds", "rounds", "rounds5", "batch", "batch", "gates", "fused", "serving"])
    gateset = rng.choice(["cr", "cr", "textbook"])
    dtype = rng.choice(["c64", "c128"])
    p = round(math.exp(rng.uniform(math.log(5e-4), math.log(2e-2))), 6)
    theta = rng.choice([0.0, round(rng.uniform(0.01, 0.06), 4)])
    eps = 0.0 if theta else round(rng.uniform(0.0, 0.03), 4)
    zeta = rng.choice([0.0, 0.0, round(rng.uniform(0.005, 0.02), 4)])
    if kind == "rounds":  # d = 2..4, options in turn
        d = rng.choice([2, 3, 3, 4])
        flag = rng.choice(["", "", "", *_FLAGS])
        if flag in ("virtual_z", "twirl", "zz_plaquette"):
            gateset = "cr"
        if flag == "zz_plaquette":
            zeta = zeta or 0.01
        # numbers back on the host (few trajectories), or records to decode
        if rng.random() < 0.5:
            return _rounds(None, d, gateset, rng.randint(1, 6), rng.randint(1, 9), dtype, p, eps, theta, zeta,
                           p1=dtype == "c128", states=True, flag=flag)
        return _rounds(None, d, gateset, rng.randint(1, 6), _log(rng, 10, 500 if d < 4 else 60), dtype, p, eps,
                       theta, zeta, decode=p < 5e-3, flag=flag)
    if kind == "rounds5":
        return _rounds(None, 5, gateset, rng.randint(1, 5), rng.randint(1, 3), dtype, min(p, 5e-3), eps, theta, zeta,
                       p1=dtype == "c128", flag=rng.choice(["", "", "", "xbasis", "idle"]))
    if kind == "batch":
        d = rng.choice([2, 3, 3, 4])
        n = _log(rng, 1, 65536) if d < 4 else _log(rng, 1, 2048 if dtype == "c128" else 4096)
        return _batch(None, d, gateset, n, dtype, rng.randint(1, 9), rng.random() < 0.7, eps, theta, zeta)
    if kind == "gates":
        return dict(kind="gates", n=rng.randint(10, 26), dtype=dtype, gates=rng.randint(2, 6))
    if kind == "fused":
        return dict(kind="fused", n=rng.randint(10, 26), dtype=dtype, k=rng.randint(1, 5), low=rng.random() < 0.3)
    return dict(kind="serving", jobs=rng.randint(3, 24), big=rng.randint(0, 2))


# ------------------------------------------------------------------ inputs --
def _eps_sites(c, seed, n):
    """Over-rotation exponents per gate site (eps = theta / 2, theta uniform)."""
    n_sites = qs.template_info(c["d"], c["gateset"])[1]
    r = np.random.default_rng([seed, 11])
    v = r.uniform(0.0, c["theta"], size=(n, n_sites)) / 2.0 if n else r.uniform(0.0, c["theta"], size=n_sites) / 2.0
    return v


def _unitary(k, rng):
    a = rng.normal(size=(1 << k, 1 << k)) + 1j * rng.normal(size=(1 << k, 1 << k))
    q, r = np.linalg.qr(a)
    return q * (np.diag(r) / np.abs(np.diag(r)))


def _register(c, seed):
    """A random normalised register as a torch tensor on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    real = torch.float64 if c["dtype"] == "c128" else torch.float32
    v = torch.randn((1 << c["n"], 2), generator=g, device="cuda", dtype=real)
    v /= math.sqrt(2.0) * 2.0 ** (c["n"] / 2)
    return torch.view_as_complex(v)


def _circuit(c, seed):
    """The gates of a "gates" pass: one-qubit and two-qubit unitaries between
    the ancilla (the top qubit) and data qubits, a phase layer, the draw."""
    r = np.random.default_rng([seed, 12])
    n, out = c["n"], []
    anc = n - 1
    for i in range(c["gates"]):
        q = int(r.integers(0, n - 1))
        out.append(("gate", [anc], _unitary(1, r)) if i % 3 == 0 else ("gate", [q, anc], _unitary(2, r)))
    q = sorted(int(x) for x in r.choice(n - 1, size=4, replace=False))
    out.append(("diag", q, np.exp(1j * r.uniform(0, 2 * np.pi, size=16))))
    out.append(("measure", anc, float(r.uniform(0.1, 0.9))))
    return out


def _matrices(c, seed):
    r = np.random.default_rng([seed, 13])
    n, k = c["n"], c["k"]
    low = list(range(k))
    rand = [int(x) for x in r.choice(n, size=k, replace=False)]
    top = list(range(n - k, n))
    return [(q, _unitary(k, r)) for q in ([low] if c["low"] else []) + [top, rand]]


def _jobs(c, seed):
    sizes = np.random.default_rng([c["jobs"], c["big"], 14])  # the burst's jobs; their noise and draws by the seed
    r = np.random.default_rng([seed, 14])
    out = []
    for i in range(c["jobs"]):
        big = i < c["big"]
        d = 5 if big else (4 if sizes.random() < 0.3 else 3)
        n = 1 if big else int(round(math.exp(sizes.uniform(math.log(10.0), math.log(1000.0 if d == 3 else 100.0)))))
        out.append(dict(tag=i, d=d, gateset="cr", rounds=int(sizes.integers(1, 4 if big else 9)), n_traj=n,
                        seed=int(r.integers(0, 2 ** 62)), p=float(r.uniform(5e-4, 5e-3)),
                        eps_site=r.uniform(0.0, 0.05, size=qs.template_info(d, "cr")[1]) / 2.0, zeta=0.0,
                        dtype="c64" if sizes.random() < 0.5 else "c128", traj0=0))
    return out


def prepare(case, seed):
    c = case
    if c["kind"] == "rounds":
        kw = dict(d=c["d"], gateset=c["gateset"], rounds=c["rounds"], n_traj=c["n_traj"], seed=seed, p=c["p"],
                  eps=c["eps"], zeta=c["zeta"], dtype=c["dtype"], want_p1=c["p1"], want_states=c["states"])
        if c["theta"]:
            kw["eps_site"] = _eps_sites(c, seed, 0)
        if c["flag"]:
            kw["idle_noise" if c["flag"] == "idle" else c["flag"]] = True
        return dict(case=c, kw=kw)
    if c["kind"] == "batch":
        r = np.random.default_rng([seed, 15])
        n = c["n_traj"]
        rounds = r.integers(1, c["max_rounds"] + 1, size=n) if c["ragged"] else np.full(n, c["max_rounds"])
        kw = dict(d=c["d"], gateset=c["gateset"], rounds=rounds.astype(np.int32),
                  p=r.uniform(5e-4, 5e-3, size=n) if c["ragged"] else np.full(n, 1e-3), seed=seed, eps=c["eps"],
                  zeta=c["zeta"], dtype=c["dtype"], max_rounds=c["max_rounds"])
        if c["theta"]:
            kw["eps_site"] = _eps_sites(c, seed, n)
        return dict(case=c, kw=kw)
    if c["kind"] in ("gates", "fused"):
        t = _register(c, seed)
        s = qs.State(c["n"], c["dtype"], stream=torch.cuda.current_stream(), tensor=t)
        return dict(case=c, tensor=t, state=s, ops=_circuit(c, seed) if c["kind"] == "gates" else _matrices(c, seed))
    return dict(case=c, jobs=_jobs(c, seed), server=qs.Server(hbm_budget=64 << 30, big_streams=2))


def run(state):
    c = state["case"]
    if c["kind"] == "rounds":
        g = qs.run_rounds(**state["kw"])
        out = dict(records=g["records"], final_bits=g["final_bits"], p1=g["p1"], states=g["states"])
        if c["decode"]:
            f = qs.decode_x if c["flag"] == "xbasis" else qs.decode_z
            out.update(f(c["d"], c["gateset"], g["records"], g["final_bits"]))
        return out
    if c["kind"] == "batch":
        g = qs.run_batch(**state["kw"])
        return dict(records=g["records"], final_bits=g["final_bits"])
    if c["kind"] == "gates":
        s, m = state["state"], None
        for op, q, v in state["ops"]:
            if op == "gate":
                s.apply_gate(q, v)
            elif op == "diag":
                s.apply_diag(q, v)
            else:
                m = s.measure_reset(q, v)
        return dict(register=state["tensor"], outcome=m[0], p1=m[1] if c["dtype"] == "c128" else None)
    if c["kind"] == "fused":
        for q, m in state["ops"]:
            state["state"].apply_fused(q, m)
        return dict(register=state["tensor"])
    srv = state["server"]
    for j in state["jobs"]:
        srv.submit(**j)
    srv.wait_idle(60.0)
    done = sorted(srv.poll(), key=lambda x: x["tag"])
    return dict(status=np.array([x["status"] for x in done]),
                records=np.concatenate([x["records"].reshape(-1) for x in done]),
                final_bits=np.concatenate([x["final_bits"].reshape(-1) for x in done]))


# -------------------------------------------------------------------- work --
_FLOPS = 40.0  # per amplitude and stabilizer circuit: two transforms, a diagonal, two weighted norms


def _trajectory(d, rounds, dtype, zeta):
    """(bytes, flops) of one trajectory.  A register that does not fit a
    compute unit (d >= 4) is read and written once for the X checks and once
    for the Z checks of a round (their outcomes are decided from sums over it),
    with the crosstalk layer between X checks once for each of those; and
    written and read once more.  Smaller ones stay on the chip."""
    n, amp = d * d, 16 if dtype == "c128" else 8
    n_x = (n - 1) // 2 + ((n - 1) & 1)
    passes = rounds * ((n_x if zeta else 1) + 1) + 1 if d >= 4 else 0
    return passes * 2.0 * amp * 2 ** n + rounds * (n - 1) + n, _FLOPS * 2 ** n * rounds * (n - 1)


def work(case):
    c = case
    if c["kind"] == "rounds":
        b, f = _trajectory(c["d"], c["rounds"], c["dtype"], c["zeta"])
        amp = 16 if c["dtype"] == "c128" else 8
        if c["states"]:
            b += amp * 2.0 ** (c["d"] ** 2)
        if c["p1"]:
            b += 8.0 * c["rounds"] * (c["d"] ** 2 - 1)
        return dict(bytes=c["n_traj"] * b, flops=c["n_traj"] * f)
    if c["kind"] == "batch":
        rounds = (c["max_rounds"] + 1) / 2 if c["ragged"] else c["max_rounds"]
        b, f = _trajectory(c["d"], rounds, c["dtype"], c["zeta"])
        per_traj = 12 + (8 * qs.template_info(c["d"], c["gateset"])[1] if c["theta"] else 0)
        return dict(bytes=c["n_traj"] * (b + per_traj), flops=c["n_traj"] * f)
    if c["kind"] in ("gates", "fused"):
        size = (16.0 if c["dtype"] == "c128" else 8.0) * 2 ** c["n"]
        # each call is a pass over the register; the measurement reads it for
        # the two norms and then keeps one half of it
        calls = c["gates"] + 1 if c["kind"] == "gates" else 2 + int(c["low"])
        k = 2 if c["kind"] == "gates" else c["k"]
        extra = 2.5 * size if c["kind"] == "gates" else 0.0
        return dict(bytes=2.0 * size * calls + extra, flops=8.0 * 2 ** k * 2 ** c["n"] * calls)
    b = f = 0.0
    for j in _jobs(c, 0):
        x, y = _trajectory(j["d"], j["rounds"], j["dtype"], 0.0)
        b, f = b + j["n_traj"] * x, f + j["n_traj"] * y
    return dict(bytes=b, flops=f)


# ------------------------------------------------- plain 64-bit evaluation --
def _uniform(seed, t, k):
    """Philox4x32-10 (key: seed, counter: (k, t)), 53 bits in [0, 1)."""
    m = 0xFFFFFFFF
    x, y, z, w = k & m, k >> 32, t & m, t >> 32
    k0, k1 = seed & m, seed >> 32
    for _ in range(10):
        a, b = 0xD2511F53 * x, 0xCD9E8D57 * z
        x, y, z, w = (b >> 32) ^ y ^ k0, b & m, (a >> 32) ^ w ^ k1, a & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return (((y << 32) | x) >> 11) / 9007199254740992.0


def _layout(d):
    """Checks in the paper's order: ("X" / "Z", data qubit or None per slot)."""
    def q(r, c):
        return r * d + c if 0 <= r < d and 0 <= c < d else None

    out = []
    for r in range(-1, d):
        for c in range(-1, d):
            if (r + c) % 2 and ((0 <= r < d - 1 and 0 <= c < d - 1) or (r in (-1, d - 1) and 0 <= c < d - 1)):
                out.append(("X", [q(r + 1, c + 1), q(r + 1, c), q(r, c), q(r, c + 1)]))
    for c in range(-1, d):
        for r in range(d - 1, -2, -1):
            if (r + c) % 2 == 0 and ((0 <= r < d - 1 and 0 <= c < d - 1) or (c in (-1, d - 1) and 0 <= r < d - 1)):
                out.append(("Z", [q(r, c + 1), q(r + 1, c + 1), q(r + 1, c), q(r, c)]))
    return out


def _x(v, q):
    return v.reshape(-1, 2, 1 << q).flip(1).reshape(-1)


def _z(v, q):
    return v * torch.tensor([1.0, -1.0], device=v.device, dtype=torch.float64).reshape(1, 2, 1).expand(
        v.numel() >> (q + 1), 2, 1 << q).reshape(-1)


def _clamp(p1):
    return 0.0 if p1 < 1e-10 else (1.0 if p1 > 1 - 1e-10 else p1)


class _Plain:
    """One trajectory gate by gate: amplitudes with the ancilla 0 and 1."""

    def __init__(self, c, kw, t, dev):
        self.c, self.seed, self.t, self.dev = c, kw["seed"], t, dev
        self.d, self.n = c["d"], c["d"] ** 2
        self.lay = _layout(self.d)
        self.eps = kw.get("eps_site")
        idx = torch.arange(1 << self.n, device=dev, dtype=torch.int64)

        def odd(mask):
            v = idx & mask
            for s in (16, 8, 4, 2, 1):
                v = v ^ (v >> s)
            return (v & 1).bool()

        want = "Z" if c["flag"] == "xbasis" else "X"
        # logical |+>: even parity on every Z check; logical |0>: the orbit of
        # 0 under the X checks, i.e. even parity on every Z check and on Z_L
        masks = [sum(1 << q for q in s if q is not None) for k, s in self.lay if k == "Z"]
        masks += [] if want == "Z" else [(1 << self.d) - 1]
        ok = torch.ones(1 << self.n, device=dev, dtype=torch.bool)
        for m in masks:
            ok &= ~odd(m)
        self.a = ok.to(torch.complex128)
        self.a /= math.sqrt(float(ok.sum()))
        self.b = torch.zeros_like(self.a)
        self.zz = None
        if c["zeta"]:
            e = torch.zeros(1 << self.n, device=dev, dtype=torch.float64)
            for i in range(self.n):
                for j in ([i + 1] if i % self.d != self.d - 1 else []) + ([i + self.d] if i + self.d < self.n else []):
                    e += 1.0 - 2.0 * (((idx >> i) ^ (idx >> j)) & 1)
            self.zz = torch.polar(torch.ones_like(e), -c["zeta"] * e)
        self.k = 0

    def u(self):
        self.k += 1
        return _uniform(self.seed, self.t, self.k - 1)

    def anc(self, P):
        if P == 1:
            self.a, self.b = self.b, self.a
        elif P == 2:
            self.a, self.b = -1j * self.b, 1j * self.a
        elif P == 3:
            self.b = -self.b

    def data(self, P, q):
        for s in ("a", "b"):
            v = getattr(self, s)
            setattr(self, s, _x(v, q) if P == 1 else _z(v, q) if P == 3 else 1j * _x(_z(v, q), q) if P == 2 else v)

    def n1(self, q):  # q None: the ancilla
        u, p = self.u(), self.c["p"]
        P = next((j for j in (1, 2, 3) if u < j * p / 3.0), 0)
        if P:
            self.anc(P) if q is None else self.data(P, q)

    def n2(self, q, data_first):
        u, p = self.u(), self.c["p"]
        P = next((j for j in range(1, 16) if u < j * p / 15.0), 0)
        f, s = P >> 2, P & 3
        self.anc(s if data_first else f)
        self.data(f if data_first else s, q)

    def rot(self, site, base, kind, q, sgn=1.0, exact=False):
        """exp(-i (base + eps) sgn A), A by kind; twirled: base, then A by a draw."""
        e = float(self.eps[site]) if self.eps is not None else self.c["eps"]
        twirl = self.c["flag"] == "twirl" and not exact
        th = sgn * (base + (0.0 if exact or twirl else e))
        C, S = math.cos(th), math.sin(th)
        a, b = self.a, self.b
        if kind == "anc":  # X on the ancilla
            self.a, self.b = C * a - 1j * S * b, C * b - 1j * S * a
        elif kind == "x":
            self.a, self.b = C * a - 1j * S * _x(a, q), C * b - 1j * S * _x(b, q)
        elif kind == "z":
            self.a, self.b = C * a - 1j * S * _z(a, q), C * b - 1j * S * _z(b, q)
        elif kind == "ad":  # Z on the ancilla, X on q
            self.a, self.b = C * a - 1j * S * _x(a, q), C * b + 1j * S * _x(b, q)
        else:  # Z on q, X on the ancilla
            self.a, self.b = C * a - 1j * S * _z(b, q), C * b - 1j * S * _z(a, q)
        if twirl and self.u() < math.sin(e) * math.sin(e):
            if kind in ("anc", "da"):
                self.anc(1)
            elif kind == "ad":
                self.anc(3)
            if kind in ("x", "ad"):
                self.data(1, q)
            elif kind in ("z", "da"):
                self.data(3, q)

    def step(self, qs_, busy, rest=False):
        """End of a step: idle noise on the waiting data qubits, crosstalk."""
        if self.c["flag"] == "idle" and not rest:
            for q in qs_:
                if q != busy:
                    self.n1(q)
        if self.c["flag"] == "zz_plaquette":
            C, S = math.cos(self.c["zeta"]), math.sin(self.c["zeta"])
            for q in qs_:
                self.a, self.b = C * self.a - 1j * S * _z(self.a, q), C * self.b + 1j * S * _z(self.b, q)

    def h(self):
        self.a, self.b = (self.a + self.b) / math.sqrt(2.0), (self.a - self.b) / math.sqrt(2.0)

    def check(self, kind, slots, site):
        """One check's circuit; returns the next gate site."""
        qd = [q for q in slots if q is not None]
        quarter = math.pi / 4
        if self.c["gateset"] == "textbook":
            for last in (False, True):
                self.h()
                self.rot(site, 0.0, "anc", None)
                site += 1
                self.n1(None)
                self.step(qd, None)
                for q in [] if last else qd:
                    if kind == "X":
                        self.b = _x(self.b, q)
                    else:
                        self.b = _z(self.b, q)
                    self.n2(q, False)
                    self.step(qd, q)
            return site
        if kind == "X":
            self.rot(site, quarter, "anc", None, sgn=-1.0)
            site += 1
            self.n1(None)
            self.step(qd, None)
        for q in slots:
            if q is None:
                self.n1(None)
            else:
                self.rot(site, quarter, "ad" if kind == "X" else "da", q)
                site += 1
                self.n2(q, kind == "Z")
            self.step(qd, q)
        if kind == "X":
            self.rot(site, quarter, "anc", None)
            site += 1
            self.n1(None)
        for q in qd:
            self.rot(site, quarter, "x" if kind == "X" else "z", q, exact=kind == "Z" and self.c["flag"] == "virtual_z")
            site += 1
            self.n1(q)
        if kind == "Z" and self.c["flag"] == "idle":
            self.n1(None)
        self.step(qd, None, rest=True)
        return site

    def trajectory(self):
        p1s = []
        for _ in range(self.c["rounds"]):
            site, row = 0, []
            for kind, slots in self.lay:
                site = self.check(kind, slots, site)
                if self.zz is not None:
                    self.a, self.b = self.a * self.zz, self.b * self.zz
                s0, s1 = (float(torch.linalg.vector_norm(v)) ** 2 for v in (self.a, self.b))
                row.append(_clamp(s1 / (s0 + s1)))
                m = self.u() < row[-1]
                self.a = self.b / math.sqrt(s1) if m else self.a / math.sqrt(s0)
                self.b = torch.zeros_like(self.a)
            p1s.append(row)
        return p1s, self.a


def _matrix_on(v, n, qubits, m):
    """Matrix m on the given qubits of v (bit j of its index: qubits[j])."""
    k = len(qubits)
    order = sorted(range(k), key=lambda j: -qubits[j])  # axes from the highest qubit down
    shape, last = [], n
    for j in order:
        shape += [1 << (last - qubits[j] - 1), 2]
        last = qubits[j]
    shape.append(1 << last)
    t = v.reshape(shape)
    at = {j: 2 * i + 1 for i, j in enumerate(order)}
    front = [at[j] for j in reversed(range(k))]  # the matrix's own order, highest bit first
    rest = [i for i in range(len(shape)) if i not in front]
    t = t.permute(front + rest)
    kept = t.shape
    w = torch.as_tensor(m, dtype=torch.complex128, device=v.device) @ t.reshape(1 << k, -1)
    back = [0] * len(shape)
    for i, a in enumerate(front + rest):
        back[a] = i
    return w.reshape(kept).permute(back).reshape(-1)


def exact(case, seed):
    c = case
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if c["kind"] == "rounds" and (c["p1"] or c["states"]):
        s = prepare(c, seed)
        p1, states = [], []
        for t in range(c["n_traj"]):
            a, v = _Plain(c, s["kw"], t, dev).trajectory()
            p1.append(a)
            if c["states"]:
                states.append(v.cpu().numpy())
        return dict(records=None, final_bits=None, p1=np.array(p1) if c["p1"] else None,
                    states=np.stack(states) if c["states"] else None)
    if c["kind"] == "gates":
        v, p1 = _register(c, seed).to(torch.complex128), None
        for op, q, m in _circuit(c, seed):
            if op == "gate":
                v = _matrix_on(v, c["n"], q, m)
            elif op == "diag":
                idx = torch.arange(v.numel(), device=v.device)
                loc = sum(((idx >> b) & 1) << i for i, b in enumerate(q))
                v = v * torch.as_tensor(m, device=v.device)[loc]
            else:
                w = v.reshape(2, -1)  # the ancilla is the top qubit
                s0, s1 = (float(torch.linalg.vector_norm(x)) ** 2 for x in w)
                p1 = _clamp(s1 / (s0 + s1))
                keep = w[1] / math.sqrt(s1) if m < p1 else w[0] / math.sqrt(s0)
                v = torch.cat([keep, torch.zeros_like(keep)])
        return dict(register=v, outcome=None, p1=p1 if c["dtype"] == "c128" else None)
    if c["kind"] == "fused":
        v = _register(c, seed).to(torch.complex128)
        for q, m in _matrices(c, seed):
            v = _matrix_on(v, c["n"], q, m)
        return dict(register=v)
    return None
