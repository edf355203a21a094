"""Step launches with two waves per tile against the one-wave form that larger batches run, at
the sizes where the split of tiles over blocks changes and at the limits of their rules."""
import numpy as np
import pytest

import synth
from paper_2503_09203_amd import mgx

from test_gpu_parity import fins_class, make_batch

pytestmark = pytest.mark.gpu

ONE_WAVE = 65600      # more tiles than the device has SIMDs


def _class(body):
    base = synth.plain_class()
    return {"plain": lambda: base, "shaped": lambda: synth.propeller_variants(base), "payload": synth.payload_class,
            "fins": lambda: fins_class(8)}[body]()


@pytest.mark.parametrize("body,precision", [("plain", mgx.FP32), ("shaped", mgx.FP32), ("payload", mgx.FP32),
                                            ("fins", mgx.FP32), ("plain", mgx.FP64), ("shaped", mgx.FP64),
                                            ("payload", mgx.FP64)])
def test_two_wave_states_equal_the_one_wave_form(body, precision):
    """One tile per block, two, three and four, the last block full or partly empty; one tile
    per compute unit and one more; hand-over groups cut by the last step: the states of the same
    environments in a batch too large for two waves, bit for bit (the same operations)."""
    import torch as t
    steps, got = (4, 5, 33), {}
    for n in (ONE_WAVE, 1, 65, 16384, 16385, 33000, 49153):
        w = synth.mixed([_class(body)], [n], steps=33, hold=3)
        b = make_batch(w, precision)
        s0 = b.get_state()
        acts = b.gen_actions(12, seed=4)
        for K in steps:
            b.set_state(s0)
            b.t = 0
            b.step(acts, K, hold=3)
            x = t.as_tensor(b.unpack_state(b.get_state())[0])
            assert b.check() == (0, 0)
            if n == ONE_WAVE:
                got[K] = x
            else:
                assert t.equal(x, got[K][:, :n]), (n, K)
        b.close()
    assert not t.equal(got[4], got[5])


@pytest.mark.parametrize("m,body", [(1, "shaped"), (6, "shaped"), (6, "payload"), (8, "shaped"), (8, "payload")])
def test_two_wave_outputs_equal_the_one_wave_form(m, body):
    """Launches with trajectory and wrenches on both sides of the two-wave form's limits (33
    steps; the longest hold per actuator count; two tiles per compute unit): states, trajectories
    and wrenches of a batch too large for it, bit for bit."""
    import torch as t
    from dataclasses import replace
    cls = synth.draw_class(m)
    cls = synth.propeller_variants(cls) if body == "shaped" else replace(cls, rg=np.array([0.015625, -0.0078125, 0.015625]))
    cases, got = ((32, 1), (33, 1), (34, 2), (35, 8), (35, 9), (35, 16), (36, 17), (33, 100)), {}
    for n in (ONE_WAVE, 65, 16385, 32768, 32769):
        w = synth.mixed([cls], [n], steps=36, hold=1)
        b = make_batch(w)
        s0 = b.get_state()
        acts = b.gen_actions(36, seed=4)
        L = b.layout
        for K, hold in cases:
            b.set_state(s0)
            b.t = 0
            traj = t.zeros((K, L.state_elems), device=b.device)
            forces = t.zeros((K, L.force_row_elems), device=b.device)
            b.step(acts, K, hold=hold, traj=traj, forces=forces)
            x = [t.as_tensor(b.unpack_state(b.get_state())[0]), traj.view(K, 13 + m, -1), forces.view(K, 12, -1)]
            assert b.check() == (0, 0)
            if n == ONE_WAVE:
                got[K, hold] = x = [y[..., :32769].clone() for y in x]
                assert x[1].abs().max() > 0 and x[2].abs().max() > 0
            else:
                assert all(t.equal(y[..., :n], z[..., :n]) for y, z in zip(x, got[K, hold])), (n, K, hold)
        b.close()


@pytest.mark.parametrize("body,precision", [("plain", mgx.FP64), ("shaped", mgx.FP64), ("payload", mgx.FP64),
                                            ("fins", mgx.FP64), ("fins", mgx.FP32), ("payload", mgx.FP32)])
@pytest.mark.parametrize("n,K,n_steps", [(70, 2, 7), (130, 16, 100), (33000, 3, 17)])
def test_joined_stretches_equal_their_launches(n, K, n_steps, body, precision):
    """A captured chunk without statistics, whose stretches share launches, against its K-step
    launches, replayed twice; attitudes start off the unit sphere, so that the drift checks
    between the stretches renormalise."""
    import torch as t
    w = synth.mixed([_class(body)], [n])
    got = []
    for captured in (True, False):
        b = make_batch(w, precision)
        x = np.array(b.unpack_state(b.get_state().cpu().numpy())[0])
        x[3:7] *= 1.2
        b.set_state(t.tensor(b.pack_state([x]), dtype=b.dtype, device=b.device))
        acts = b.gen_actions((2 * n_steps + 4) // 5, seed=4)
        if captured:
            g = b.capture(acts, n_steps, K, hold=5)
            g.replay()
            g.replay()
        else:
            for r in range(2):
                for k in range(0, n_steps, K):
                    b.step(acts, min(K, n_steps - k), hold=5)
        got.append((b.get_state(), b.t))
        assert b.check() == (0, 0)
        b.close()
    assert got[0][1] == got[1][1] == 2 * n_steps and t.equal(got[0][0], got[1][0])


@pytest.mark.parametrize("body,precision", [("plain", mgx.FP32), ("payload fins", mgx.FP64)])
def test_single_steps_replayed_at_other_steps(body, precision):
    """Single steps captured by the caller carry the steps of their capture; replayed later, they
    start again on the rows that the device counter names. Against the same steps one by one."""
    import torch as t
    from dataclasses import replace
    cls = synth.plain_class() if body == "plain" else replace(fins_class(8), rg=np.array([0.015625, -0.0078125, 0.015625]))
    w = synth.mixed([cls], [130], steps=8, hold=1)
    got, side = [], t.cuda.Stream()
    for captured in (True, False):
        with t.cuda.stream(side):
            b = make_batch(w, precision)
            acts = b.gen_actions(8, seed=4)
            t.cuda.synchronize()
            if captured:
                g = t.cuda.CUDAGraph()
                with t.cuda.graph(g, stream=side):
                    b.step(acts, 1, hold=1)
                    b.step(acts, 1, hold=1)
                for _ in range(4):
                    g.replay()
            else:
                for _ in range(8):
                    b.step(acts, 1, hold=1)
            state = b.get_state().clone()
        t.cuda.synchronize()
        got.append(state)
        assert b.check() == (0, 0)
        b.close()
    assert t.equal(got[0], got[1])


def test_fin_blocks_are_resident_together():
    """Eight actuators with fins hold the most LDS per tile. A launch of two tiles for some
    compute units may not run its blocks in two rounds: it takes about as long as one of a tile
    each (two rounds take twice as long; the bound is half way)."""
    import torch as t
    times = []
    for n in (16384, 20000):
        w = synth.mixed([fins_class(8)], [n], steps=1, hold=1)
        b = make_batch(w)
        acts = b.gen_actions(1, seed=4)
        best = np.inf
        for _ in range(6):
            e0, e1 = t.cuda.Event(enable_timing=True), t.cuda.Event(enable_timing=True)
            e0.record()
            b.step(acts, 200, hold=1 << 20)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1))
        times.append(best)
        b.close()
    assert times[1] < 1.5 * times[0], times
