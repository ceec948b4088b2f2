"""After a call that failed, a handle is where it was: the rounds that had been started are not lost and not taken
from models that were overwritten meanwhile, and a version that is gone is refused."""
import os
import subprocess
import sys

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("preset,in_batch", [(1, 0), (1, 1), (2, 0), (3, 0), (3, 1)])
def test_rounds_after_a_call_that_gave_up_waiting(preset, in_batch):
    env = dict(os.environ, ABS_MAILBOX_TIMEOUT_MS="0.01", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-u", os.path.join(ROOT, "tests", "failed_calls_main.py"), str(preset), str(in_batch)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, env=env, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().splitlines()[-1].startswith("ok: "), r.stdout[-3000:]


@pytest.mark.parametrize("preset", [1, 2])
@pytest.mark.parametrize("ahead", [True, False])
def test_versions_after_a_loss_that_is_not_finite(preset, ahead):
    """The round that failed and the one started behind it have overwritten the ring's oldest versions: those are refused, also
    after the round has been asked for again, alone and in a batch; all others are what they were."""
    import paper_2301_08895_amd as lib
    p = workloads.scaled_preset(preset, M=4000, N=4, B=4, K0=2, k_mode=1, tau_cap=3, a=1, n_slow=0)
    R = p["tau_cap"] + 3
    data = workloads.make_inputs(p)
    data["X"][1234] = np.nan
    ref = lib.Simulation(p, data, profile=1)
    models = [ref.model()]
    with pytest.raises(lib.AbsError):
        while True:
            ref.round(1)
            models.append(ref.model())
    t = len(models) - 1
    assert t > 10
    sim = lib.Simulation(p, data)
    batch = lib.Batch([sim])
    sim.round(t)

    def check(oldest):
        assert lib.abs_rounds_done(sim.handle) == t
        for v in range(t - R - 1, t + 3):
            if max(0, oldest) <= v <= t:
                assert np.array_equal(sim.model(v), models[v]), v
                sim.evaluate(data["X"][:8], data["y"][:8], version=v)
            elif v >= 0:
                for read in (lambda: sim.model(v), lambda: sim.evaluate(data["X"][:8], data["y"][:8], version=v)):
                    with pytest.raises(lib.AbsError) as e:
                        read()
                    assert e.value.code == -4, v

    check(t + 1 - R)
    for call in (lambda: sim.round(3 if ahead else 1), lambda: sim.round(1), lambda: batch.round(2), lambda: sim.round(1)):
        with pytest.raises(lib.AbsError) as e:
            call()
        assert e.value.code == -5
        check(t + 3 - R if ahead else t + 2 - R)
    batch.close(); sim.close(); ref.close()
