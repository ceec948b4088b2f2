"""Driver of test_gpu_failed_calls.py: calls of abs_round that give up waiting (ABS_MAILBOX_TIMEOUT_MS is a few
microseconds in this process) because the stream is busy with other work, and what the handle does afterwards."""
import sys

import numpy as np
import torch

import paper_2301_08895_amd as lib
import workloads

E_HIP, E_VERSION = -3, -4


def steady(sim, n):
    """n rounds, over whatever time-outs."""
    end = lib.abs_rounds_done(sim.handle) + n
    while lib.abs_rounds_done(sim.handle) < end:
        torch.cuda.synchronize()
        try:
            sim.round(1)
        except lib.AbsError as e:
            assert e.code == E_HIP, e


def history(p, data, T):
    """Every version's model and the trace, from a handle that takes a round's losses before it starts the next."""
    sim = lib.Simulation(p, data, profile=1)
    models = [sim.model()]
    for _ in range(T):
        steady(sim, 1)
        models.append(sim.model())
    trace = sim.trace()
    sim.close()
    return models, trace


def check_ring(sim, models, p, readable_from, evaluation):
    """What can be read is that version, by both read-outs alike; what is gone is refused."""
    t = lib.abs_rounds_done(sim.handle)
    for v in range(max(0, t - p["tau_cap"] - 4), t + 3):
        ok = []
        for read in (lambda: sim.model(v), lambda: sim.evaluate(*evaluation, version=v)):
            try:
                got = read()
                ok.append(True)
                if len(ok) == 1:
                    assert np.array_equal(got, models[v]), f"version {v} after round {t}"
            except lib.AbsError as e:
                assert e.code == E_VERSION, e
                ok.append(False)
        assert ok[0] == ok[1] == (max(0, readable_from) <= v <= t), (v, t, readable_from, ok)


def main(preset, in_batch):
    over = {1: dict(M=4000, N=8, B=32, K0=2, tau_cap=3), 2: dict(M=4000, dims=[784, 10], N=8, B=16, K0=2, tau_cap=2),
            3: dict(M=2000, dims=[64, 40, 5], n_classes=5, N=8, B=20, K0=2, tau_cap=2)}[preset]
    p = workloads.scaled_preset(preset, k_mode=1, n_slow=0, **over)
    data = workloads.make_inputs(p)
    evaluation = (data["X"][:50], data["y"][:50])
    calls, R = 40, p["tau_cap"] + 3
    models, trace = history(p, data, 4 * calls + 4)
    if in_batch:
        q = dict(p, seed_sim=p["seed_sim"] + 1)
        models2, trace2 = history(q, data, 4 * calls + 4)
        other = lib.Simulation(q, data)
    sim = lib.Simulation(p, data)
    steady(sim, 3)                                   # (the kernels are loaded)
    if in_batch:
        steady(other, 3)
        batch = lib.Batch([other, sim])
    busy = torch.zeros(1 << 28, device="cuda")
    given_up = stale = 0
    launched = 3
    for call in range(calls):
        torch.cuda.synchronize()
        t = lib.abs_rounds_done(sim.handle)
        for again in (3, 1 + call % 2) if call % 3 == 0 else (3,):
            first = lib.abs_rounds_done(sim.handle)
            for _ in range(8):
                busy.add_(1.0)                       # some 0.4 ms each
            try:
                sim.round(again)
                launched = max(launched, first + again)
            except lib.AbsError as e:
                assert e.code == E_HIP, e
                failed = lib.abs_rounds_done(sim.handle)
                launched = max(launched, min(failed + 2, first + again))       # the round behind it had been started too
                given_up += 1
                stale += launched == failed + 2 and int(trace[failed][12 + 2 * p["K0"]:12 + 3 * p["K0"]].max()) == p["tau_cap"] + 1
            check_ring(sim, models, p, launched + 1 - R, evaluation)
        torch.cuda.synchronize()
        if in_batch and call % 2:
            try:
                batch.round(1)
            except lib.AbsError as e:
                assert e.code == E_HIP, e
            torch.cuda.synchronize()
        while lib.abs_rounds_done(sim.handle) < t + 3:
            steady(sim, 1)
        launched = lib.abs_rounds_done(sim.handle)
        check_ring(sim, models, p, launched + 1 - R, evaluation)
    T = lib.abs_rounds_done(sim.handle)
    assert np.array_equal(sim.trace(), trace[:T])
    if in_batch:
        T2 = lib.abs_rounds_done(other.handle)
        assert T2 > 3 and np.array_equal(other.trace(), trace2[:T2]) and np.array_equal(other.model(), models2[T2])
        batch.close(); other.close()
    sim.close()
    assert given_up >= calls // 2, given_up
    assert stale >= 3, stale
    print(f"ok: preset {preset}, batch {in_batch}: {given_up} calls given up, {stale} at a round that reads the oldest version", flush=True)


if __name__ == "__main__":
    main(int(sys.argv[1]), int(sys.argv[2]))
