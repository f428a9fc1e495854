"""Trajectories run side by side (resident states up to 13 qubits, shared
sweep launches from 14) against the same trajectories one by one, which the
driver does when it times its kernels."""

import torch  # noqa: F401  (imported at collection: the first import can be slow)

import numpy as np
import pytest

import workloads as W
from gpu_helpers import AMP_TOL, rel_l2

pytestmark = pytest.mark.gpu


def _circuit(n, depth, two_qubit):
    """A noisy grid with mixtures and inner-product channels; with
    `two_qubit`, damping on pairs as one two-qubit channel, too."""
    c = W.generic_grid_circuit(n, depth, p_dep=0.02, gamma=0.01, seed=40 + n)
    if not two_qubit:
        return c
    k = W.amplitude_damp(0.02)
    pair = [np.kron(a, b) for a in k for b in k]
    ops = []
    for i, op in enumerate(c.ops):
        ops.append(op)
        if op.kind == W.GATE and len(op.qubits) == 2 and i % 3 == 0:
            ops.append(W.Op(W.CHANNEL, tuple(reversed(op.qubits)), pair, op.moment, "pair_damp"))
    return W.Circuit(n, ops, "pairs")


@pytest.mark.parametrize("n,depth,f,two_qubit,n_traj,states", [
    (1, 6, 4, False, 90, 1), (2, 8, 2, True, 60, 1), (5, 8, 5, True, 20, 2), (9, 8, 4, True, 11, 1),
    (10, 10, 4, False, 12, 1), (11, 8, 3, True, 7, 1), (13, 6, 4, True, 300, 1), (13, 6, 5, False, 3, 2),
    (14, 8, 4, False, 70, 1), (14, 6, 4, True, 4, 1), (15, 6, 5, False, 3, 1), (16, 6, 1, False, 9, 3),
    (19, 5, 4, False, 20, 1), (21, 4, 3, False, 6, 1)])
def test_side_by_side_equals_one_by_one(qs, n, depth, f, two_qubit, n_traj, states):
    c = _circuit(n, depth, two_qubit)
    e0, e1 = W.readout_arrays(n, 0.01, 0.02)
    kw = dict(seed=5, traj_offset=3, circuit_id=2, max_fuse=f, n_samples=7, p0to1=e0, p1to0=e1, return_state=True,
              z_expect=True)
    handles = [qs.State(n) for _ in range(states)]
    try:
        hs = [h.h for h in handles]
        got = qs.qs_run_trajectories(hs if states > 1 else hs[0], c, n_traj, **kw)
        ref = qs.qs_run_trajectories(hs[0], c, n_traj, time_kernels=True, **kw)
    finally:
        for h in handles:
            h.close()
    assert ref["n_slow"].sum() > 0
    for key in ("choices", "paths", "n_slow"):
        assert np.array_equal(got[key], ref[key]), key
    # from 10 qubits on both run the same blocks in the same order on the same
    # units; below, the one-by-one path multiplies in another order
    assert np.abs(got["z_expect"] - ref["z_expect"]).max() < 2 * AMP_TOL
    assert rel_l2(got["state"], ref["state"]) < AMP_TOL
    if n >= 10:
        assert np.array_equal(got["samples"], ref["samples"])
        assert got["gate_sweeps"] == ref["gate_sweeps"]


def test_range_split_keeps_results(qs):
    """The same range in one call, in pieces and one by one through
    traj_offset; a 14-qubit piece of one trajectory takes the other path."""
    for n in (8, 14):
        c = _circuit(n, 6, False)
        with qs.State(n) as st:
            whole = qs.qs_run_trajectories(st.h, c, 9, seed=1, max_fuse=4, return_state=True)
            for first, count in ((0, 4), (4, 4), (8, 1)):
                part = qs.qs_run_trajectories(st.h, c, count, seed=1, max_fuse=4, traj_offset=first, return_state=True)
                assert np.array_equal(part["choices"], whole["choices"][first:first + count])
        assert np.array_equal(part["state"], whole["state"])


@pytest.mark.parametrize("n,n_traj,states", [(13, 2, 1), (13, 9, 2), (14, 2, 1), (14, 3, 2), (16, 5, 1),
                                             (21, 2, 1), (21, 3, 2)])
def test_tuned_calls_keep_the_widths_that_run_side_by_side(qs, n, n_traj, states):
    """With both widths left to the tuner, a call that can run side by side is
    tuned over the fusion width alone (at most four qubits from 14 qubits on),
    and equals the one-by-one run with the same widths."""
    c = _circuit(n, 5, False)
    kw = dict(seed=6, traj_offset=1, n_samples=9, return_state=True)
    handles = [qs.State(n) for _ in range(states)]
    try:
        hs = [h.h for h in handles]
        got = qs.qs_run_trajectories(hs if states > 1 else hs[0], c, n_traj, max_fuse=0, **kw)
        f, tb = got["max_fuse_used"], got["tile_bits_used"]
        again = qs.qs_run_trajectories(hs[0], c, n_traj, max_fuse=0, **kw)
        ref = qs.qs_run_trajectories(hs[0], c, n_traj, max_fuse=f, tile_bits=tb, time_kernels=True, **kw)
    finally:
        for h in handles:
            h.close()
    assert tb == 13 and (n == 13 or f <= 4)
    assert again["tune_ms"] == 0.0
    for key in ("choices", "paths", "samples"):
        assert np.array_equal(got[key], ref[key]), key
        assert np.array_equal(got[key], again[key]), key
    assert rel_l2(got["state"], ref["state"]) < AMP_TOL


@pytest.mark.parametrize("n,n_traj,noise", [(11, 1, 0.0), (11, 4, 0.01), (12, 1, 0.01), (12, 3, 0.0), (13, 1, 0.0),
                                            (13, 2, 0.01)])
def test_few_trajectories_of_five_qubit_blocks_stay_on_the_matrix_units(qs, n, n_traj, noise):
    """A workgroup per trajectory multiplies 5-qubit blocks on VALU, three
    times as slow for a single one; such a call runs as the timed one does,
    bit for bit."""
    c = W.generic_grid_circuit(n, 12, p_dep=noise or None, gamma=noise or None, seed=n)
    kw = dict(seed=4, max_fuse=5, n_samples=3, return_state=True)
    with qs.State(n) as st:
        got = qs.qs_run_trajectories(st.h, c, n_traj, **kw)
        ref = qs.qs_run_trajectories(st.h, c, n_traj, time_kernels=True, **kw)
    assert got["gate_k_launches"][5] > 0
    for key in ("choices", "samples", "state"):
        assert np.array_equal(got[key], ref[key]), key


def test_staging_grows_with_the_calls(qs):
    """One small trajectory, then many, then one by one on one handle: each
    equals the call on a handle of its own."""
    c = _circuit(9, 8, True)
    calls = [(1, {}), (120, {}), (3, dict(time_kernels=True)), (2, {})]
    kw = dict(seed=8, max_fuse=4, n_samples=5, return_state=True, z_expect=True)
    with qs.State(9) as st:
        for count, more in calls:
            got = qs.qs_run_trajectories(st.h, c, count, **kw, **more)
            with qs.State(9) as own:
                ref = qs.qs_run_trajectories(own.h, c, count, **kw, **more)
            for key in ("choices", "samples", "state", "z_expect"):
                assert np.array_equal(got[key], ref[key]), (count, key)


@pytest.mark.parametrize("n,f,n_traj,states", [(7, 5, 3, 3), (8, 5, 5, 4), (11, 5, 6, 3), (12, 5, 4, 2), (13, 5, 5, 4),
                                               (13, 3, 2, 2), (14, 4, 3, 3), (16, 4, 5, 4)])
def test_chunks_round_as_the_whole_call(qs, n, f, n_traj, states):
    """A concurrent call's chunks take the path that one state would take for
    the whole range, however few trajectories each has."""
    c = W.generic_grid_circuit(n, 8, p_dep=0.01, gamma=0.002 if n > 13 else None, seed=n)
    kw = dict(seed=11, max_fuse=f, n_samples=3, return_state=True, z_expect=True)
    handles = [qs.State(n) for _ in range(states)]
    try:
        got = qs.qs_run_trajectories([h.h for h in handles], c, n_traj, **kw)
        ref = qs.qs_run_trajectories(handles[0].h, c, n_traj, **kw)
    finally:
        for h in handles:
            h.close()
    for key in ("choices", "samples", "z_expect", "state"):
        assert np.array_equal(got[key], ref[key]), key


def test_path_does_not_depend_on_what_the_state_did_before(qs):
    """More samples than a flush holds run one by one, also on a handle whose
    sample buffer an earlier call made larger (5-qubit blocks of 11 qubits
    round differently side by side)."""
    c = W.generic_grid_circuit(11, 8, p_dep=0.02, seed=3)
    kw = dict(seed=2, max_fuse=5, n_samples=900000, return_state=True, record_choices=False)
    with qs.State(11) as st, qs.State(11) as used:
        qs.qs_sample_measurements(used.h, 1, 0, 5000000)
        a = qs.qs_run_trajectories(st.h, c, 5, **kw)
        b = qs.qs_run_trajectories(used.h, c, 5, **kw)
        side = qs.qs_run_trajectories(st.h, c, 5, **dict(kw, n_samples=0))
    assert not np.array_equal(side["state"], a["state"])
    assert np.array_equal(a["state"], b["state"])
    assert np.array_equal(a["samples"], b["samples"])
    assert rel_l2(side["state"], a["state"]) < AMP_TOL


def test_tuner_times_the_kind_of_call_it_tunes(qs):
    """One trajectory in a workgroup, many side by side and timed passes of one
    state have choices of their own; a circuit with a 5-qubit gate above 13
    qubits always runs as passes of one state and shares theirs."""
    c = W.generic_grid_circuit(9, 7, p_dep=0.01, gamma=0.003, seed=21)
    with qs.State(9) as st:
        def tune_ms(n_traj, **kw):
            return qs.qs_run_trajectories(st.h, c, n_traj, seed=1, max_fuse=0, **kw)["tune_ms"]

        assert tune_ms(1) > 0.0
        assert tune_ms(40) > 0.0
        assert tune_ms(3, time_kernels=True) > 0.0
        assert [tune_ms(1), tune_ms(64), tune_ms(1, time_kernels=True)] == [0.0] * 3
    ops = list(W.generic_grid_circuit(14, 4, p_dep=0.01, seed=22).ops)
    wide = W.random_unitary(5, np.random.Generator(np.random.PCG64(2)))
    ops.insert(20, W.Op(W.GATE, (1, 4, 7, 10, 13), [wide], ops[20].moment, "wide"))
    c = W.Circuit(14, ops, "wide")
    with qs.State(14) as st:
        one = qs.qs_run_trajectories(st.h, c, 1, seed=1, max_fuse=0)
        four = qs.qs_run_trajectories(st.h, c, 4, seed=1, max_fuse=0)
    assert one["tune_ms"] > 0.0 and four["tune_ms"] == 0.0
    assert (one["max_fuse_used"], one["tile_bits_used"]) == (four["max_fuse_used"], four["tile_bits_used"])


@pytest.mark.parametrize("n,f", [(5, 4), (9, 4), (11, 5), (12, 5), (13, 5)])
def test_both_ways_round_within_the_blocks_errors(qs, n, f):
    """Where the workgroup's kernels differ from the one-by-one path's (below
    10 qubits, and 5-qubit blocks of 11 to 13), the states differ by no more
    than the two paths' rounding: an output of a block sums 2^f products of
    complex numbers in FP32, so at most 2^f + 2 roundings of 2^-24 of its norm
    a block and path."""
    c = W.generic_grid_circuit(n, 10, p_dep=0.02, seed=n)
    kw = dict(seed=3, max_fuse=f, return_state=True)
    with qs.State(n) as st:
        side = qs.qs_run_trajectories(st.h, c, 6, **kw)
        alone = qs.qs_run_trajectories(st.h, c, 6, time_kernels=True, **kw)
    assert np.array_equal(side["choices"], alone["choices"])
    blocks = sum(alone["gate_k_launches"]) / 6
    assert rel_l2(side["state"], alone["state"]) < 2 * blocks * (2 ** f + 2) * 2.0 ** -24
