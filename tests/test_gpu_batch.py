"""Batched simulations (abs_batch_*): a simulation's result must not depend on what else is in its
batch.  Linear rounds are bitwise those of an unbatched run; softmax rounds sum the gradient per
upload first (another rounding order than abs_round), so they are bitwise those of a batch of one
and agree with the unbatched run and with the CPU oracle to the parity bar."""
import numpy as np
import pytest

import workloads
import paper_2301_08895_amd as lib
from parity_util import assert_models_close, assert_matches_oracle, LOSS_WORD, KNEXT_WORD

pytestmark = pytest.mark.gpu


def _variants(base, S):
    """S settings of one shape: different simulation seeds, a, K0, step sizes and methods."""
    names = ["abs", "adasync", "sa_abs", "k_async", "abs_fixed_tau"]
    out = []
    for i in range(S):
        p = workloads.method_preset(base, names[i % len(names)])
        p.update(seed_sim=base["seed_sim"] + 17 * i, lr=base["lr"] * (1.0 + 0.1 * (i % 4)),
                 K0=1 + i % base["N"])
        if p["tau_mode"] == 0:
            p["a"] = p["tau_cap"] - base["N"] // base["K0"] - (i % 2)
        out.append(p)
    return out


def _same_schedule(tr, want):
    """Traces agree in everything but the loss words (False: an adaptive-K decision flipped on a
    last-bit loss difference, which the unbatched parity tests cover)."""
    keep = np.ones(tr.shape[1], bool)
    keep[LOSS_WORD] = False
    if np.any(tr[:, KNEXT_WORD] != want[:, KNEXT_WORD]):
        return False
    assert np.array_equal(tr[:, keep], want[:, keep])
    return True


def _rerun_as_batch_of_one(d):
    def rerun(q, k_replay):
        sim = lib.Simulation(q, d, k_replay=k_replay)
        one = lib.Batch([sim])
        one.round(len(k_replay))
        one.close()
        out = (sim.model().copy(), sim.trace().copy())
        sim.close()
        return out
    return rerun


def _run(base, S, T, tol, loss_rtol, oracle_for=(0, 1), bitwise_alone=True):
    d = workloads.make_inputs(base)
    ps = _variants(base, S)
    sims = [lib.Simulation(p, d) for p in ps]
    batch = lib.Batch(sims)
    batch.round(T // 2)
    mid = [s.model().copy() for s in sims]            # handles stay usable between batch calls
    batch.round(T - T // 2)
    got = [(s.model().copy(), s.trace().copy()) for s in sims]
    batch.close()
    for s in sims:
        s.close()
    assert len({m.tobytes() for m in mid}) > 1        # the simulations really differ
    compared = 0
    for i, p in enumerate(ps):
        alone = lib.Simulation(p, d)
        if bitwise_alone:
            alone.round(T)
            assert np.array_equal(alone.model(), got[i][0]), f"simulation {i} differs from its unbatched run"
            assert np.array_equal(alone.trace(), got[i][1]), f"trace of simulation {i} differs from its unbatched run"
        else:
            one = lib.Batch([alone])
            one.round(T)
            one.close()
            assert np.array_equal(alone.model(), got[i][0]), f"simulation {i} differs from a batch of one"
            assert np.array_equal(alone.trace(), got[i][1]), f"trace of simulation {i} differs from a batch of one"
            plain = lib.Simulation(p, d)
            plain.round(T)
            if _same_schedule(got[i][1], plain.trace()):
                compared += 1
                assert_models_close(p, got[i][0], plain.model(), d["w0"], tol, T, where=f"simulation {i} against its unbatched run")
            plain.close()
        alone.close()
    assert bitwise_alone or compared >= S // 2
    for i in oracle_for:
        assert_matches_oracle(ps[i], d, got[i][0], got[i][1], T, tol, _rerun_as_batch_of_one(d), where=f"simulation {i}")


def test_linear_batch():
    _run(workloads.scaled_preset(1, M=4000), 12, 60, 1e-5, 1e-4)


def test_linear_batch_wide():
    _run(workloads.scaled_preset(1, M=4000, dims=[300, 1], N=16, B=20, tau_cap=3), 70, 30, 1e-5, 1e-4, oracle_for=(3,))


def test_softmax_batch():
    _run(workloads.scaled_preset(2, M=6000), 6, 40, 1e-5, 1e-4, bitwise_alone=False)
    _run(workloads.scaled_preset(2, M=4000, dims=[52, 3], n_classes=3, N=6, B=10, K0=2, tau_cap=2, lr=5e-3), 9, 50,
         1e-5, 1e-4, bitwise_alone=False)
    # the widest model the register-resident form takes (all 56 blocks of 16 features in use)
    _run(workloads.scaled_preset(2, M=3000, dims=[892, 10], N=5, B=37, lr=2e-4), 3, 10, 1e-5, 1e-4,
         oracle_for=(0,), bitwise_alone=False)
    # all 16 class columns in use
    _run(workloads.scaled_preset(2, M=3000, dims=[320, 16], n_classes=16, N=6, B=23, lr=5e-4), 4, 10, 1e-5, 1e-4,
         oracle_for=(0,), bitwise_alone=False)
    # wider ones keep the model in LDS: 8-row tiles with two workgroups per CU (1000 x 4) ...
    _run(workloads.scaled_preset(2, M=3000, dims=[1000, 4], n_classes=4, N=4, B=21, lr=2e-4), 3, 10, 1e-5, 1e-4,
         oracle_for=(0,), bitwise_alone=False)
    # ... or 16-row tiles (16 classes and 1024 features), a ragged last tile; 8 features (fewer chunks than lanes)
    _run(workloads.scaled_preset(2, M=4000, dims=[1024, 16], n_classes=16, N=4, B=70, lr=2e-4), 3, 12, 1e-5, 1e-4,
         oracle_for=(0,), bitwise_alone=False)
    _run(workloads.scaled_preset(2, M=2000, dims=[8, 2], n_classes=2, N=16, B=5, lr=2e-2), 20, 30, 1e-5, 1e-4,
         oracle_for=(0,), bitwise_alone=False)


def test_batches_that_advance_as_groups():
    """Large batches run as two to four groups staggered in time, each on its own stream (softmax:
    two from 4 simulations, three from 64, four from 128; linear: two from 32): results must not
    change, also when a call is split in two."""
    _run(workloads.scaled_preset(2, M=2000, dims=[20, 4], n_classes=4, N=5, B=17, K0=2, lr=1e-2), 131, 14, 1e-5, 1e-4,
         oracle_for=(0, 130), bitwise_alone=False)
    _run(workloads.scaled_preset(2, M=2000, dims=[12, 3], n_classes=3, N=6, B=9, K0=2, lr=1e-2), 67, 21, 1e-5, 1e-4,
         oracle_for=(0, 66), bitwise_alone=False)
    _run(workloads.scaled_preset(1, M=2000, dims=[20, 1], N=5, B=6, K0=2), 515, 11, 1e-5, 1e-4, oracle_for=(0, 514))


def test_softmax_batch_of_many_simulations():
    """Launches of more than a thousand uploads (4 groups of 130 simulations x up to 8 uploads; wait
    counts differ between the simulations): bitwise the batch of one.  Three tiles with a ragged last
    one, a single tile per upload, and all feature blocks in use."""
    _run(workloads.scaled_preset(2, M=2000, dims=[20, 4], n_classes=4, N=8, B=37, K0=2, lr=1e-2), 520, 8, 1e-5, 1e-4,
         oracle_for=(0, 259, 519), bitwise_alone=False)
    _run(workloads.scaled_preset(2, M=2000, dims=[36, 10], N=8, B=9, K0=2, lr=1e-2), 520, 6, 1e-5, 1e-4,
         oracle_for=(7, 518), bitwise_alone=False)
    _run(workloads.scaled_preset(2, M=3000, dims=[892, 10], N=8, B=16, lr=2e-4), 520, 4, 1e-5, 1e-4,
         oracle_for=(0, 300), bitwise_alone=False)


def test_local_sgd_batches():
    """U > 1 in batched rounds: the local-SGD kernels with one column of workgroups per simulation,
    bitwise the unbatched rounds (also as groups)."""
    _run(workloads.scaled_preset(1, M=3000, dims=[40, 1], N=6, B=8, K0=2, U=3), 9, 30, 1e-5, 1e-4)
    _run(workloads.scaled_preset(2, M=3000, dims=[24, 5], n_classes=5, N=7, B=6, K0=3, U=4, lr=1e-2), 66, 16,
         1e-5, 1e-4, oracle_for=(0, 65))
    a = lib.Simulation(workloads.scaled_preset(1, M=2000, U=2), workloads.make_inputs(workloads.scaled_preset(1, M=2000, U=2)))
    b = lib.Simulation(workloads.scaled_preset(1, M=2000), workloads.make_inputs(workloads.scaled_preset(1, M=2000)))
    with pytest.raises(lib.AbsError):
        lib.Batch([a, b])                      # U must agree
    a.close()
    b.close()


def test_softmax_batch_of_long_minibatches():
    """B > 1024: batched softmax rounds run the kernels of abs_round, one column per simulation."""
    _run(workloads.scaled_preset(2, M=6000, dims=[16, 4], n_classes=4, N=3, B=1030, K0=1, lr=5e-3), 3, 10, 1e-5, 1e-4,
         oracle_for=(0,))


def test_batch_rejects_mixed_shapes_and_models():
    d1 = workloads.make_inputs(workloads.scaled_preset(1, M=2000))
    a = lib.Simulation(workloads.scaled_preset(1, M=2000), d1)
    p2 = workloads.scaled_preset(1, M=2000, B=16)
    b = lib.Simulation(p2, d1)
    with pytest.raises(lib.AbsError):
        lib.Batch([a, b])
    with pytest.raises(lib.AbsError):
        lib.Batch([a, a])
    pm = workloads.scaled_preset(3, M=2048, dims=[128, 64, 10], N=4, B=32, n_slow=1)
    m = lib.Simulation(pm, workloads.make_inputs(pm))
    with pytest.raises(lib.AbsError):
        lib.Batch([a, m])                      # one model kind per batch
    for s in (a, b, m):
        s.close()


def test_batch_device_memory_comes_from_the_caller():
    """The batch's device scratch is a workspace of abs_batch_workspace_size() bytes that the caller
    brings: too small or missing is an error, MLP handles need none."""
    import torch
    p = workloads.scaled_preset(2, M=3000, dims=[32, 5], n_classes=5, N=8, B=12, lr=2e-2)
    d = workloads.make_inputs(p)
    sims = [lib.Simulation(dict(p, seed_sim=p["seed_sim"] + i), d) for i in range(3)]
    handles = [s.handle for s in sims]
    need = lib.abs_batch_workspace_size(handles)
    assert need > 3 * (16 + 8 * 16) and need % 256 == 0
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    ptr = (ws.data_ptr() + 255) // 256 * 256
    for args in ((0, 0), (ptr, need - 256), (ptr + 8, need)):
        with pytest.raises(lib.AbsError) as e:
            lib.abs_batch_create(handles, *args)
        assert e.value.code in (-1, -2)
    b = lib.abs_batch_create(handles, ptr, need)
    lib.abs_batch_round(b, 5)
    lib.abs_batch_destroy(b)
    one = lib.Simulation(dict(p, seed_sim=p["seed_sim"] + 1), d)
    b1 = lib.Batch([one])
    b1.round(5)
    b1.close()
    assert np.array_equal(one.model(), sims[1].model())
    for s in sims + [one]:
        s.close()
    pm = workloads.scaled_preset(3, M=2048, dims=[128, 64, 10], N=4, B=32, n_slow=1)
    m = lib.Simulation(pm, workloads.make_inputs(pm))
    assert lib.abs_batch_workspace_size([m.handle]) == 0
    bm = lib.abs_batch_create([m.handle])
    lib.abs_batch_destroy(bm)
    m.close()


def test_mlp_batch():
    """MLP simulations of a batch run side by side, each through its own rounds on a stream of the
    batch: bitwise the unbatched runs, also with more simulations than streams and over two calls."""
    base = workloads.scaled_preset(3, M=4096, dims=[256, 128, 10], N=6, B=32, n_slow=1, K0=2, tau_cap=3)
    d = workloads.make_inputs(base)
    S, T = 6, 14
    ps = [dict(base, seed_sim=base["seed_sim"] + 101 * i, lr=base["lr"] * (1 + 0.25 * (i % 3)), sa_penalty=i % 2)
          for i in range(S)]
    sims = [lib.Simulation(p, d) for p in ps]
    batch = lib.Batch(sims)
    batch.round(T // 2)
    mid = [s.model().copy() for s in sims]
    batch.round(T - T // 2)
    got = [(s.model().copy(), s.trace().copy()) for s in sims]
    batch.close()
    for s in sims:
        s.close()
    assert len({m.tobytes() for m in mid}) == S
    for i, p in enumerate(ps):
        alone = lib.Simulation(p, d)
        alone.round(T)
        assert np.array_equal(alone.model(), got[i][0]), f"simulation {i} differs from its unbatched run"
        assert np.array_equal(alone.trace(), got[i][1])
        alone.close()
    assert_matches_oracle(ps[1], d, got[1][0], got[1][1], T, 2e-2, _rerun_as_batch_of_one(d), where="simulation 1")


def test_batch_of_simulations_on_different_datasets():
    """Only the shape has to agree: every simulation may bring its own dataset."""
    base = workloads.scaled_preset(2, M=3000, dims=[32, 5], n_classes=5, N=8, B=12, lr=2e-2)
    ps = [dict(base, seed_data=base["seed_data"] + 5 * i, seed_sim=base["seed_sim"] + i) for i in range(5)]
    ds = [workloads.make_inputs(p) for p in ps]
    sims = [lib.Simulation(p, d) for p, d in zip(ps, ds)]
    batch = lib.Batch(sims)
    batch.round(40)
    got = [(s.model().copy(), s.trace().copy()) for s in sims]
    batch.close()
    for s in sims:
        s.close()
    for p, d, (m, tr) in zip(ps, ds, got):
        alone = lib.Simulation(p, d)
        one = lib.Batch([alone])
        one.round(40)
        one.close()
        assert np.array_equal(alone.model(), m) and np.array_equal(alone.trace(), tr)
        alone.close()
        assert_matches_oracle(p, d, m, tr, 40, 1e-5, _rerun_as_batch_of_one(d), where=f"dataset seed {p['seed_data']}")


def test_batch_error_leaves_every_simulation_consistent():
    """One simulation of a large batch runs out of its K replay: the call names it, rounds already on
    the device are completed (so the simulations end within a round of each other), and every other
    handle carries on, alone, exactly as if nothing had happened (linear model: bitwise)."""
    base = dict(workloads.scaled_preset(1, M=2000, dims=[20, 1], N=5, B=6, K0=2), k_mode=2)
    d = workloads.make_inputs(base)
    S, bad, T = 515, 300, 12
    ok_replay = np.tile(np.array([2, 3, 1, 5, 4], np.int32), 4)
    ps = [dict(base, seed_sim=base["seed_sim"] + 13 * i) for i in range(S)]
    sims = [lib.Simulation(p, d, k_replay=ok_replay[:7] if i == bad else ok_replay) for i, p in enumerate(ps)]
    batch = lib.Batch(sims)
    with pytest.raises(lib.AbsError) as err:
        batch.round(T)
    assert f"simulation {bad}" in str(err.value)
    batch.close()
    done = np.array([lib.abs_rounds_done(s.handle) for s in sims])
    assert done[bad] in (6, 7)
    assert np.all(np.abs(done - done[bad]) <= 1)
    assert len(set(done[:S // 2])) == 1 and len(set(np.delete(done, bad)[S // 2:])) == 1
    for i in (0, 1, S // 2 - 1, S // 2, bad - 1, bad + 1, S - 1):
        sims[i].round(T - int(done[i]))
        alone = lib.Simulation(ps[i], d, k_replay=ok_replay)
        alone.round(T)
        assert np.array_equal(alone.model(), sims[i].model()) and np.array_equal(alone.trace(), sims[i].trace())
        alone.close()
    for s in sims:
        s.close()


def test_mlp_batch_error_does_not_stop_the_others():
    """MLP simulations of a batch advance independently: the one that runs out of its K replay is
    reported, all the others complete their rounds."""
    base = dict(workloads.scaled_preset(3, M=4096, dims=[256, 128, 10], N=6, B=32, n_slow=1, K0=2, tau_cap=3), k_mode=2)
    d = workloads.make_inputs(base)
    S, bad, T = 6, 2, 10
    replay = np.tile(np.array([2, 3, 1, 6, 4], np.int32), 2)
    ps = [dict(base, seed_sim=base["seed_sim"] + 7 * i) for i in range(S)]
    sims = [lib.Simulation(p, d, k_replay=replay[:4] if i == bad else replay) for i, p in enumerate(ps)]
    batch = lib.Batch(sims)
    with pytest.raises(lib.AbsError) as err:
        batch.round(T)
    assert f"simulation {bad}" in str(err.value)
    batch.close()
    done = [lib.abs_rounds_done(s.handle) for s in sims]
    assert done[bad] == 4 and all(n == T for i, n in enumerate(done) if i != bad)
    for i in (0, S - 1):
        alone = lib.Simulation(ps[i], d, k_replay=replay)
        alone.round(T)
        assert np.array_equal(alone.model(), sims[i].model()) and np.array_equal(alone.trace(), sims[i].trace())
        alone.close()
    for s in sims:
        s.close()


def test_softmax_batch_random_shapes():
    """Seeded random shapes (features, classes, workers, minibatch, batch size) of batched softmax
    rounds: batch-of-one bitwise, oracle to the parity bar."""
    rng = np.random.default_rng(20240607)
    for case in range(10):
        d_ = int(rng.integers(1, 257)) * 4
        C = int(rng.integers(2, 17))
        N = int(rng.integers(1, 17))
        B = int(rng.choice([1, 3, 7, 8, 9, 15, 16, 17, 31, 40, 64, 100, 130, 257]))
        S = int(rng.choice([1, 2, 5, 33, 70]))
        p = workloads.scaled_preset(2, M=max(N * 20, 600), dims=[d_, C], n_classes=C, N=N, B=B,
                                    K0=int(rng.integers(1, N + 1)), tau_cap=int(rng.integers(1, 5)),
                                    lr=float(0.2 / d_), sa_penalty=int(rng.integers(0, 2)))
        print(f"case {case}: d={d_} C={C} N={N} B={B} S={S}", flush=True)
        d = workloads.make_inputs(p)
        ps = [dict(p, seed_sim=p["seed_sim"] + 31 * k) for k in range(S)]
        sims = [lib.Simulation(q, d) for q in ps]
        batch = lib.Batch(sims)
        batch.round(8)
        batch.close()
        got = [(s.model().copy(), s.trace().copy()) for s in sims]
        for s in sims:
            s.close()
        for k in sorted({0, S - 1}):
            one = lib.Simulation(ps[k], d)
            b1 = lib.Batch([one])
            b1.round(8)
            b1.close()
            assert np.array_equal(one.model(), got[k][0]) and np.array_equal(one.trace(), got[k][1]), (case, k)
            one.close()
            assert_matches_oracle(ps[k], d, got[k][0], got[k][1], 8, 1e-5, _rerun_as_batch_of_one(d),
                                  where=f"case {case} simulation {k}")


@pytest.mark.parametrize("S", [1, 63, 64, 67])
def test_many_short_calls_equal_one_long_call(S):
    """The batch's host threads sleep between calls and take up the next one (none below 64 simulations)."""
    base = workloads.scaled_preset(1, M=1000, dims=[12, 1], N=5, B=4, K0=2)
    d = workloads.make_inputs(base)
    out = []
    for calls in ([1] * 12, [0, 12]):
        sims = [lib.Simulation(p, d) for p in _variants(base, S)]
        batch = lib.Batch(sims)
        for n in calls:
            batch.round(n)
        batch.close()
        out.append([(s.model().copy(), s.trace().copy()) for s in sims])
        for s in sims:
            s.close()
    for (m0, t0), (m1, t1) in zip(*out):
        assert np.array_equal(m0, m1) and np.array_equal(t0, t1)


def test_batches_driven_from_several_threads_at_once():
    """Calls that run side by side share the process's budget of host threads (a call's number of them changes
    while it runs); results are those of the batches driven one after the other."""
    import threading
    import torch
    base = workloads.scaled_preset(1, M=1000, dims=[12, 1], N=5, B=4, K0=2)
    d = workloads.make_inputs(base)
    out = []
    for at_once in (False, True):
        batches, sims = [], []
        for b in range(4):
            with torch.cuda.stream(torch.cuda.Stream()):
                sims.append([lib.Simulation(dict(p, seed_sim=p["seed_sim"] + 1000 * b), d) for p in _variants(base, 64 + b)])
                batches.append(lib.Batch(sims[-1]))

        def drive(b):
            for n in (1, 7, 40):
                batches[b].round(n)
        threads = [threading.Thread(target=drive, args=(b,)) for b in range(4)]
        for t in threads:
            t.start()
            if not at_once:
                t.join()
        for t in threads:
            t.join()
        out.append([(s.model().copy(), s.trace().copy()) for ss in sims for s in ss])
        for b in batches:
            b.close()
        for ss in sims:
            for s in ss:
                s.close()
    assert len(out[0]) == len(out[1]) == 4 * 64 + 6
    for (m0, t0), (m1, t1) in zip(*out):
        assert np.array_equal(m0, m1) and np.array_equal(t0, t1)
