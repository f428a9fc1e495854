"""Work that programs give this library, as measurable cases.

A case is a plain dict; `kind` says which public entry points its pass goes
through:

  batch    qs_run_batched: many small mixed-unitary circuits in one launch,
           bitstrings and Kraus choices out (the serving loop's batch lane,
           the 12-qubit chain)
  traj     qs_run_trajectories (one state) or its concurrent form (several
           states on their own streams): noisy trajectories, or one noiseless
           state; the Kraus choices and the last trajectory's amplitudes out
  sample   qs_sample_measurements on a state in device memory
  observe  qs_norm, qs_expectation_z and qs_expectation on such a state
  gates    qs_copy_state, then qs_apply_fused_gate / qs_apply_channel one by
           one and qs_flush: a program that drives the state itself

Amplitudes are complex64 everywhere; that is the library's only state type.

`traj` cases take no bitstrings: which index a draw lands on in a state of
2^20 or more amplitudes hangs on the last bits of the complex64 arithmetic,
so the pass returns the amplitudes themselves, and sampling is measured on
given states (`sample`), where every bitstring is determined.  `max_fuse` is
the one the workloads' own records carry (4, batched launches 3) rather than
the autotuner's, whose choice depends on timing.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2111_02396_amd as qs
import workloads as W


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # The smallest batched request: one 10-qubit circuit, four shots of one
        # sample each, as a serving loop meets it when nothing else waits.
        dict(name="batch-10q-4", kind="batch", layout="grid", circuits=1, n_lo=10, n_hi=10,
             d_lo=10, d_hi=10, traj=4, shots=1, p_dep=1e-3, readout=0.0),
        # The 12-qubit chain: 100 trajectories of 1000 samples.
        dict(name="batch-chain12", kind="batch", layout="chain", circuits=1, n_lo=12, n_hi=12,
             d_lo=20, d_hi=20, traj=100, shots=1000, p_dep=1e-3, readout=0.0),
        # A full batch of mixed sizes: 64 circuits of 12 to 18 qubits and 10 to
        # 40 cycles, 16 trajectories each.
        dict(name="batch-mixed", kind="batch", layout="grid", circuits=64, n_lo=12, n_hi=18,
             d_lo=10, d_hi=40, traj=16, shots=1, p_dep=1e-3, readout=0.02),
        # The smallest trajectory call: one 10-qubit trajectory with amplitude
        # damping (latency of one request outside the batch lane).
        dict(name="traj-10q-1", kind="traj", n=10, depth=10, p_dep=1e-3, gamma=1e-3, lam=0.0,
             traj=1, states=1),
        # A serving request of odd size: 15 qubits, 25 cycles, 20 trajectories.
        dict(name="traj-15q-20", kind="traj", n=15, depth=25, p_dep=3e-3, gamma=1e-3, lam=0.0,
             traj=20, states=1),
        # Phase damping at 0.01 after every gate, 20 qubits on one state: many
        # channels need inner products.
        dict(name="traj-phase20", kind="traj", n=20, depth=20, p_dep=0.0, gamma=0.0, lam=1e-2,
             traj=20, states=1),
        # The headline workload: 24-qubit 4x6 grid, depolarizing 1e-3 and
        # amplitude damping 1e-3, two states side by side.
        dict(name="traj-grid24", kind="traj", n=24, depth=20, p_dep=1e-3, gamma=1e-3, lam=0.0,
             traj=16, states=2),
        # One noiseless 28-qubit state of depth 20 (2 GiB, past every cache).
        dict(name="traj-28q-noiseless", kind="traj", n=28, depth=20, p_dep=0.0, gamma=0.0, lam=0.0,
             traj=1, states=1),
        # A large noisy request: one 30-qubit trajectory (8 GiB).
        dict(name="traj-30q", kind="traj", n=30, depth=12, p_dep=1e-3, gamma=1e-3, lam=0.0,
             traj=1, states=1),
        # 10^5 readings of a 28-qubit state, with readout error.
        dict(name="sample-28q", kind="sample", n=28, shots=100000, readout=0.02),
        # Norm, every <Z_q>, and one- and two-qubit observables of a 26-qubit state.
        dict(name="observe-26q", kind="observe", n=26, pairs=4),
        # A program that drives a 22-qubit state itself: 24 fused gates of one
        # to five qubits on scattered targets, with amplitude damping between.
        dict(name="gates-22q", kind="gates", n=22, count=24, k_max=5, gamma=0.01),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["batch", "batch", "traj", "traj", "traj", "sample", "observe", "gates"])
    if kind == "batch":
        lo = rng.randint(6, 18)
        hi = rng.randint(lo, 18)
        d = rng.randint(5, 40)
        circuits = _log_int(rng, 1, 64)
        return dict(kind="batch", layout=rng.choice(["grid", "grid", "chain"]), circuits=circuits,
                    n_lo=lo, n_hi=hi, d_lo=d, d_hi=rng.randint(d, 40),
                    traj=_log_int(rng, 1, max(1, 1024 // circuits)),
                    shots=_log_int(rng, 1, 100), p_dep=10.0 ** rng.uniform(-4, -2),
                    readout=rng.choice([0.0, 0.02]))
    if kind == "traj":
        n = rng.randint(4, 28)
        noise = rng.choice(["mixture", "damping", "phase", "none"])
        states = 1 if n > 26 else rng.choice([1, 1, 2, 3])
        most = max(1, min(64, 1 << max(0, 28 - n)))
        return dict(kind="traj", n=n, depth=rng.randint(5, 40 if n < 26 else 20),
                    p_dep=10.0 ** rng.uniform(-4, -2) if noise in ("mixture", "damping") else 0.0,
                    gamma=10.0 ** rng.uniform(-4, -2.5) if noise == "damping" else 0.0,
                    lam=10.0 ** rng.uniform(-4, -1.5) if noise == "phase" else 0.0,
                    traj=1 if noise == "none" else max(states, _log_int(rng, 1, most)), states=states)
    if kind == "sample":
        n = rng.randint(8, 28)
        return dict(kind="sample", n=n, shots=_log_int(rng, 1, 100000), readout=rng.choice([0.0, 0.02]))
    if kind == "observe":
        return dict(kind="observe", n=rng.randint(8, 28), pairs=rng.randint(1, 8))
    n = rng.randint(6, 26)
    return dict(kind="gates", n=n, count=rng.randint(4, 32), k_max=rng.randint(1, 5),
                gamma=rng.choice([0.0, 0.01, 0.05]))


# ---------------------------------------------------------------- inputs

def _traj_circuit(case, seed):
    """The noisy grid; with `lam`, phase damping after every gate instead."""
    n = case["n"]
    if not case["lam"]:
        return W.generic_grid_circuit(n, case["depth"], p_dep=case["p_dep"] or None,
                                      gamma=case["gamma"] or None, seed=seed)
    damp = W.phase_damp(case["lam"])
    ops = []
    for op in W.generic_grid_circuit(n, case["depth"], seed=seed).ops:
        ops.append(op)
        ops += [W.Op(W.CHANNEL, (q,), damp, op.moment, "phase_damp") for q in op.qubits]
    return W.Circuit(n, ops, "phase-damped")


def _spread(lo, hi, count, i):
    """The i-th of `count` whole numbers spread over lo..hi."""
    return lo if count == 1 else lo + (i * 7919 % count) * (hi - lo + 1) // count


def _batch_workloads(case, seed):
    out = []
    for i in range(case["circuits"]):
        n = _spread(case["n_lo"], case["n_hi"], case["circuits"], i)
        d = _spread(case["d_lo"], case["d_hi"], case["circuits"], 3 * i + 1)
        build = W.chain_circuit if case["layout"] == "chain" else W.generic_grid_circuit
        c = build(n, d, p_dep=case["p_dep"], seed=seed * 4099 + i)
        e0 = e1 = None
        if case["readout"]:
            e0, e1 = W.readout_arrays(n, case["readout"], case["readout"])
        out.append(W.TrajectoryWorkload(f"c{i}", c, n_traj=case["traj"], seed=seed, circuit_id=i,
                                        n_samples=case["shots"], e0=e0, e1=e1, max_fuse=3))
    return out


def _random_state(n, seed):
    """A normalised random state: what a deep circuit leaves behind."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    v = torch.randn(1 << n, dtype=torch.complex64, device="cuda", generator=g)
    return v.mul_(2.0 ** (-0.5 * n))


def _gate_program(case, seed):
    """(targets, matrix) for gates and (targets, Kraus list) for channels, in order."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n = case["n"]
    prog = []
    for i in range(case["count"]):
        k = 1 + i % min(case["k_max"], n)
        prog.append(("gate", tuple(int(x) for x in rng.choice(n, size=k, replace=False)),
                     W.random_unitary(k, rng)))
        if case["gamma"] and i % 4 == 3:
            prog.append(("channel", (int(rng.integers(n)),), W.amplitude_damp(case["gamma"])))
    return prog


def _state_on(buf, n, stream=None):
    return qs.State(n, buf.data_ptr(), buf.numel() * buf.element_size(), stream)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return dict(kind=kind, batch=qs.PreparedBatch(_batch_workloads(case, seed)))
    n = case["n"]
    if kind == "traj":
        mc = qs.MarshalledCircuit(_traj_circuit(case, seed))
        bufs = [torch.zeros(1 << n, dtype=torch.complex64, device="cuda") for _ in range(case["states"])]
        streams = [torch.cuda.Stream() for _ in bufs] if len(bufs) > 1 else [None]
        torch.cuda.synchronize()  # the streams' first work follows the buffers' clearing
        states = [_state_on(b, n, s.cuda_stream if s is not None else None) for b, s in zip(bufs, streams)]
        return dict(kind=kind, mc=mc, bufs=bufs, streams=streams, states=states, seed=seed, traj=case["traj"])
    buf = torch.zeros(1 << n, dtype=torch.complex64, device="cuda")
    given = _state_on(buf, n)  # a new handle starts as |0...0>; the program puts its state there
    buf.copy_(_random_state(n, seed))
    if kind == "sample":
        e = W.readout_arrays(n, case["readout"], case["readout"]) if case["readout"] else (None, None)
        return dict(kind=kind, buf=buf, state=given, seed=seed, shots=case["shots"], e=e)
    if kind == "observe":
        return dict(kind=kind, buf=buf, state=given, obs=_observables(case, seed))
    out = torch.zeros_like(buf)
    return dict(kind=kind, buf=buf, out=out, src=given, state=_state_on(out, n), seed=seed,
                prog=_gate_program(case, seed))


def _observables(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    out = []
    for i in range(case["pairs"]):
        k = 1 + i % 2
        m = W.random_matrix(k, rng)
        out.append((tuple(int(x) for x in rng.choice(case["n"], size=k, replace=False)), m + m.conj().T))
    return out


# ---------------------------------------------------------------- one pass

def run(state):
    kind = state["kind"]
    if kind == "batch":
        results, _ = qs.qs_run_batched(state["batch"], max_fuse=3, copy=False)
        # one array for all circuits, as a program collects them
        return {"samples": np.concatenate([r["samples"].ravel() for r in results]),
                "choices": np.concatenate([r["choices"].ravel() for r in results])}
    if kind == "traj":
        hs = [s.h for s in state["states"]]
        r = qs.qs_run_trajectories(hs if len(hs) > 1 else hs[0], None, state["traj"], seed=state["seed"],
                                   max_fuse=4, marshalled=state["mc"])
        # the range is cut into contiguous chunks, so the last state that got
        # a trajectory holds the range's last one
        last = min(len(hs), state["traj"]) - 1
        return {"state": state["bufs"][last], "choices": r["choices"], "paths": r["paths"],
                "n_slow": r["n_slow"]}
    h = state["state"].h
    if kind == "sample":
        return qs.qs_sample_measurements(h, state["seed"], 0, state["shots"], *state["e"])
    if kind == "observe":
        return {"norm": qs.qs_norm(h), "z": qs.qs_expectation_z(h),
                "obs": [qs.qs_expectation(h, t, m) for t, m in state["obs"]]}
    qs.qs_copy_state(h, state["src"].h)
    picks = []
    for i, (what, targets, m) in enumerate(state["prog"]):
        if what == "gate":
            qs.qs_apply_fused_gate(h, targets, m)
        else:
            picks.append(qs.qs_apply_channel(h, targets, m, state["seed"], 0, i)[0])
    qs.qs_flush(h)
    return {"state": state["out"], "picks": np.array(picks + [-1], dtype=np.int32)}


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Bytes: the result (and a given state) once.  Flops: every dense gate of
    the circuit once, 8 * 2^k - 2 per amplitude (the sign flips of the CZ
    layers and the picks that commute into a gate's matrix are free)."""
    kind = case["kind"]
    if kind == "batch":
        flops = out = 0.0
        for i in range(case["circuits"]):
            n = _spread(case["n_lo"], case["n_hi"], case["circuits"], i)
            d = _spread(case["d_lo"], case["d_hi"], case["circuits"], 3 * i + 1)
            flops += 14.0 * n * d * 2.0 ** n * case["traj"]
            out += case["traj"] * (8.0 * case["shots"] + n * d)
        return {"bytes": out, "flops": flops}
    dim = 2.0 ** case["n"]
    if kind == "traj":
        return {"bytes": 8.0 * dim, "flops": 14.0 * case["n"] * case["depth"] * dim * case["traj"]}
    if kind == "sample":
        return {"bytes": 8.0 * dim + 8.0 * case["shots"], "flops": 4.0 * dim}
    if kind == "observe":
        return {"bytes": 8.0 * dim, "flops": 4.0 * dim}
    ks = [1 + i % min(case["k_max"], case["n"]) for i in range(case["count"])]
    return {"bytes": 16.0 * dim, "flops": sum(8.0 * 2 ** k - 2 for k in ks) * dim}


# ---------------------------------------------------------------- the same in 64 bits

def _philox(counter, key):
    """Philox4x32-10 (Salmon et al., SC'11)."""
    c, (k0, k1) = list(counter), key
    for _ in range(10):
        a, b = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(b >> 32) ^ c[1] ^ k0, b & 0xFFFFFFFF, (a >> 32) ^ c[3] ^ k1, a & 0xFFFFFFFF]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _channel_draw(seed, index, traj):
    w = _philox((index, traj, 0, 0), (seed & 0xFFFFFFFF, seed >> 32))
    return (((w[1] << 32) | w[0]) >> 11) * 2.0 ** -53


class _Exact:
    """A complex128 state; one-qubit operators wait until a wider one, or an
    inner product, touches their qubit."""

    def __init__(self, n, v):
        self.n, self.v, self.pending = n, v, {}

    def _one(self, q, m):
        lo = 1 << q
        x = self.v.view(-1, 2, lo)
        if m[0, 1] == 0 and m[1, 0] == 0:
            x[:, 0].mul_(complex(m[0, 0]))
            x[:, 1].mul_(complex(m[1, 1]))
            return
        flat = max(1, (1 << 27) // (2 * lo))  # bounded temporaries
        for part in (x.split(flat) if x.shape[0] > flat else [x]):
            for w in part.split(1 << 27, dim=2):
                a, b = w[:, 0].clone(), w[:, 1].clone()
                w[:, 0] = a * complex(m[0, 0]) + b * complex(m[0, 1])
                w[:, 1] = a * complex(m[1, 0]) + b * complex(m[1, 1])

    def flush(self, qubits=None):
        for q in list(self.pending) if qubits is None else qubits:
            if q in self.pending:
                self._one(q, self.pending.pop(q))

    def apply(self, targets, m):
        k = len(targets)
        if k == 1:
            q = targets[0]
            self.pending[q] = m @ self.pending[q] if q in self.pending else m
            return
        self.flush(targets)
        d = np.diag(m)
        if k == 2 and np.array_equal(m, np.diag(d)):
            hi, lo = max(targets), min(targets)
            x = self.v.view(-1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
            for j in range(4):
                if d[j] != 1:
                    bit = {targets[0]: j & 1, targets[1]: j >> 1}
                    x[:, bit[hi], :, bit[lo], :].mul_(complex(d[j]))
            return
        dims = [self.n - 1 - t for t in reversed(targets)]  # most significant matrix bit first
        rest = [i for i in range(self.n) if i not in dims]
        x = self.v.view([2] * self.n).permute(dims + rest).reshape(1 << k, -1)
        x = torch.tensor(m, dtype=torch.complex128, device=self.v.device) @ x
        back = [0] * self.n
        for i, p in enumerate(dims + rest):
            back[p] = i
        self.v = x.view([2] * self.n).permute(back).reshape(-1)

    def density(self, targets):
        """R[j, l] = sum of v_j conj(v_l) over the rest of the index."""
        k = len(targets)
        dims = [self.n - 1 - t for t in reversed(targets)]
        rest = [i for i in range(self.n) if i not in dims]
        if k == 1:
            x = self.v.view(-1, 2, 1 << targets[0])
            parts = [x[:, 0].reshape(-1), x[:, 1].reshape(-1)]
        else:
            y = self.v.view([2] * self.n).permute(dims + rest).reshape(1 << k, -1)
            parts = [y[j] for j in range(1 << k)]
        return np.array([[complex(torch.vdot(parts[l], parts[j])) for l in range(1 << k)] for j in range(1 << k)])

    def channel(self, targets, kraus, r):
        """Algorithm 2 with lazy normalisation: a pick from the bounds leaves
        the norm as K_i leaves it (a mixture's K_i is taken as its unitary),
        a pick after inner products divides by sqrt(p_i N)."""
        grams = [K.conj().T @ K for K in kraus]
        pbar = [max(float(np.linalg.eigvalsh(g)[0]), 0.0) for g in grams]
        mixture = all(np.allclose(g, g[0, 0] * np.eye(len(g)), atol=1e-12) for g in grams)
        pick = None
        for i, p in enumerate(pbar):
            if r < p:
                pick = i
                break
            r -= p
        if pick is None and mixture:
            pick = max(i for i, p in enumerate(pbar) if p > 0)
        if pick is not None:
            K = kraus[pick] / math.sqrt(pbar[pick]) if mixture else kraus[pick]
            if not np.allclose(K, K[0, 0] * np.eye(len(K)), atol=1e-14):
                self.apply(targets, K)
            return
        self.flush()
        R = self.density(targets)
        N = float(np.trace(R).real)
        e = [float(np.trace((g - p * np.eye(len(g))) @ R).real) / N for g, p in zip(grams, pbar)]
        pick = max((i for i, x in enumerate(e) if x > 0), default=len(e) - 1)
        for i, x in enumerate(e):
            if r < x:
                pick = i
                break
            r -= x
        self.apply(targets, kraus[pick] / math.sqrt((pbar[pick] + e[pick]) * N))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "sample"):
        return None  # whole numbers
    n = case["n"]
    if kind == "observe":
        v = _random_state(n, seed)
        p = torch.view_as_real(v).double().square().sum(-1)
        N = float(p.sum())
        z = []
        for q in range(n):
            x = p.view(-1, 2, 1 << q).sum(dim=(0, 2))
            z.append(float(x[0] - x[1]) / N)
        s = _Exact(n, v.to(torch.complex128))
        obs = [float(np.trace(m @ s.density(t)).real) / N for t, m in _observables(case, seed)]
        return {"norm": N, "z": np.array(z), "obs": obs}
    if kind == "gates":
        s = _Exact(n, _random_state(n, seed).to(torch.complex128))
        for i, (what, targets, m) in enumerate(_gate_program(case, seed)):
            if what == "gate":
                s.apply(targets, m)
            else:
                s.channel(targets, m, _channel_draw(seed, i, 0))
        s.flush()
        return {"state": s.v, "picks": None}
    v = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    v[0] = 1.0
    s, ordinal = _Exact(n, v), 0
    for op in _traj_circuit(case, seed).ops:
        if op.kind == W.GATE:
            s.apply(op.qubits, op.mats[0])
        else:
            s.channel(op.qubits, op.mats, _channel_draw(seed, ordinal, case["traj"] - 1))
            ordinal += 1
    s.flush()
    return {"state": s.v, "choices": None, "paths": None, "n_slow": None}
