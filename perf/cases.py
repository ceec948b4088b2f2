"""The work a user of libabs has it do, as cases that can be timed and compared.

A case is a simulation (or a batch of simulations, or a held-out evaluation) on seeded synthetic data,
driven through the C entry points as a training program drives them: the handle, its workspace and the
dataset exist, and one pass advances it by a few parameter-server rounds (abs_round / abs_batch_round) or
reads the held-out loss and accuracy (abs_evaluate).  What comes back is the new global model, left where
the library keeps it (the ring of model versions at the head of the caller's workspace), and the event
trace of the rounds.

The wait count K^t is held constant (k_mode 1), so a pass is the same amount of work whenever it is
timed; worker times, minibatches, staleness and forced restarts vary from round to round as in any run.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2301_08895_amd as lib

LINEAR, SOFTMAX, MLP, CNN = 0, 1, 2, 3
MODEL_OF = {"linear": LINEAR, "softmax": SOFTMAX, "mlp": MLP, "cnn": CNN}
HEADER, LOSS_WORD = 12, 10


def _case(name, model, dims, M, N, B, K, rounds, *, U=1, S=1, rows=0, tau_cap=4, sa=0, times="exp", slow=0):
    """model, dims: as abs_config (dims as text, a case holds plain values); M dataset rows; N workers of
    minibatch B, K uploads per round; U local steps; S simulations in a batch; rounds per pass;
    rows > 0: the pass evaluates that many held-out rows instead of training."""
    return dict(name=name, model=model, dims=" ".join(str(d) for d in dims), M=M, N=N, B=B, K=K, U=U, S=S,
                rounds=rounds, rows=rows, tau_cap=tau_cap, sa=sa, times=times, slow=slow)


def listed():
    wide = [3072, 2048, 2048, 100]
    image = [3 * 32 * 32, 6, 16, 120, 84, 10, 3, 5]
    return [
        # the smallest round there is: least squares, two uploads of 32 rows; latency and launches only
        _case("linear", "linear", [100, 1], 10_000, 8, 32, 2, 20, tau_cap=3),
        # softmax regression on 784 features, one simulation: a round of a few hundred rows
        _case("softmax", "softmax", [784, 10], 60_000, 16, 64, 4, 20),
        # the same with ten local steps per job, every worker waited for (synchronous local SGD)
        _case("softmax local", "softmax", [784, 10], 60_000, 16, 64, 16, 10, U=10),
        # a sweep: 64 softmax simulations advanced as one batch
        _case("softmax sweep", "softmax", [784, 10], 60_000, 16, 64, 8, 10, S=64),
        # one hidden layer of 512, a fifth of the workers slowed down, a quarter of them waited for
        _case("mlp 512", "mlp", [3072, 512, 10], 50_000, 32, 128, 8, 10, times="slow", slow=6),
        # two hidden layers of 1024, staleness-aware steps, half of the workers waited for
        _case("mlp 1024", "mlp", [3072, 1024, 1024, 10], 50_000, 64, 128, 32, 6, tau_cap=6, sa=1),
        # two hidden layers of 2048, 100 classes, Pareto times: the first rounds of a run (K = N / 4) ...
        _case("mlp 2048", "mlp", wide, 100_000, 128, 256, 32, 6, tau_cap=8, times="pareto"),
        # ... and its last ones, when every worker is waited for: the largest round
        _case("mlp 2048 all", "mlp", wide, 100_000, 128, 256, 128, 3, tau_cap=8, times="pareto"),
        # nothing a multiple of a tile: widths, minibatch, classes
        _case("mlp ragged", "mlp", [1000, 520, 300, 26], 30_000, 24, 90, 9, 10, tau_cap=3),
        # local SGD on the network with one hidden layer: ten steps on a private model per upload
        _case("mlp local", "mlp", [3072, 512, 10], 50_000, 32, 128, 8, 1, U=10, times="slow", slow=6),
        # two convolutional and three dense layers on 32 x 32 colour images, 5 of 20 workers
        _case("cnn", "cnn", image, 50_000, 20, 32, 5, 5, tau_cap=2),
        # held-out loss and accuracy of the wide network over a test set of 10 000 rows
        _case("mlp evaluate", "mlp", wide, 100_000, 128, 256, 32, 0, rows=10_000, tau_cap=8, times="pareto"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(x, m, hi):
    return min(hi, max(m, (x + m // 2) // m * m))


def draw(rng):
    """One more case: any model, with and without local steps, alone, in a batch or evaluated, with sizes
    spread over the ranges the listed cases span."""
    kind = rng.choice(["linear", "softmax", "softmax local", "softmax sweep", "linear sweep", "mlp", "mlp", "mlp",
                       "mlp local", "mlp sweep", "cnn", "evaluate"])
    model = {"linear sweep": "linear", "evaluate": rng.choice(["mlp", "mlp", "softmax", "cnn"])}.get(kind, kind.split()[0])
    times = rng.choice(["exp", "pareto", "slow"])
    sa, tau_cap = int(rng.random() < 0.3), rng.randint(2, 8)
    U, S, rows = 1, 1, 0
    if kind == "evaluate":
        rows = _log(rng, 1000, 20_000)
    if model == "linear":
        N, B = _log(rng, 4, 64), _log(rng, 8, 128)
        dims, M = [_log(rng, 16, 512), 1], _log(rng, 5000, 60_000)
        rounds = 20
        if kind == "linear sweep":
            S, N = _log(rng, 16, 256), min(N, 16)
    elif model == "softmax":
        N, B = _log(rng, 4, 64), _log(rng, 8, 256)
        dims, M = [_mult(_log(rng, 32, 1024), 4, 1024), rng.randint(2, 16)], _log(rng, 5000, 60_000)
        rounds = 20
        if kind == "softmax local":
            U, rounds = rng.randint(2, 12), 8
        elif kind == "softmax sweep":
            S, N, rounds = _log(rng, 8, 128), min(N, 16), 10
    elif model == "cnn":
        S_k = rng.choice([(32, 5), (28, 5), (18, 3), (22, 3)])
        C0 = rng.choice([1, 3])
        N, B = _log(rng, 4, 32), _log(rng, 8, 48)
        dims = [C0 * S_k[0] ** 2, rng.randint(4, 10), rng.randint(8, 20), _log(rng, 40, 200), _log(rng, 24, 100),
                rng.randint(2, 20), C0, S_k[1]]
        M, rounds = _log(rng, 5000, 50_000), 5
        if rng.random() < 0.3:
            U, rounds = rng.randint(2, 6), 1
    else:
        N, B = _log(rng, 4, 128), _log(rng, 16, 256)
        depth = rng.randint(2, 4)
        tile = rng.choice([1, 1, 128, 256])          # half of the networks have widths of whole tiles
        dims = [_mult(_log(rng, 256, 3072), max(8, tile), 3072)]
        dims += [_mult(_log(rng, 64, 2048), tile, 2048) for _ in range(depth - 1)] + [rng.choice([10, 100, rng.randint(2, 128)])]
        M = _log(rng, 10_000, 60_000)
        rounds = 6
        if kind == "mlp local":
            U, rounds, N = rng.randint(2, 10), 1, min(N, 32)
        elif kind == "mlp sweep":
            S, N, rounds = rng.randint(2, 6), min(N, 32), 4
    M = max(M, 4 * N)
    K = max(1, min(N, int(round(N * rng.choice([0.125, 0.25, 0.25, 0.5, 1.0])))))
    slow = max(1, N // 5) if times == "slow" else 0
    c = _case("", model, dims, M, N, B, K, 0 if rows else rounds, U=U, S=S, rows=rows, tau_cap=tau_cap, sa=sa, times=times, slow=slow)
    del c["name"]
    return c


def _shapes(case):
    """[(rows, columns)] of the weight matrices in the model vector."""
    d = [int(x) for x in case["dims"].split()]
    if case["model"] == "linear":
        return [(d[0], 1)]
    if case["model"] == "cnn":
        d0, C1, C2, F1, F2, C, C0, k = d
        S2 = (((math.isqrt(d0 // C0) - k + 1) // 2) - k + 1) // 2
        return [(C0 * k * k, C1), (C1 * k * k, C2), (C2 * S2 * S2, F1), (F1, F2), (F2, C)]
    return [(d[l], d[l + 1]) for l in range(len(d) - 1)]


def _params(case):
    return sum(r * c + (0 if case["model"] == "linear" else c) for r, c in _shapes(case))


def _classes(case):
    d = [int(x) for x in case["dims"].split()]
    return d[5] if case["model"] == "cnn" else d[-1]


def _data(case, n, gen, mu):
    """n rows of the workload: a Gaussian mixture with unit variance around the class means (bf16 for the
    MLP), or standard normal rows with noisy linear targets."""
    d0 = int(case["dims"].split()[0])
    if case["model"] == "linear":
        X = torch.randn(n, d0, generator=gen, device="cuda")
        return X, X @ mu + 0.01 * torch.randn(n, generator=gen, device="cuda")
    y = torch.randint(0, _classes(case), (n,), generator=gen, device="cuda", dtype=torch.int32)
    X = torch.empty(n, d0, device="cuda", dtype=torch.bfloat16 if case["model"] == "mlp" else torch.float32)
    for lo in range(0, n, 20_000):
        hi = min(n, lo + 20_000)
        X[lo:hi] = torch.randn(hi - lo, d0, generator=gen, device="cuda") + mu[y[lo:hi].long()]
    return X, y


def _learning_rate(case):
    """Steps that learn and stay stable on inputs that are not normalised: inversely to a row's squared norm."""
    d = [int(x) for x in case["dims"].split()]
    if case["model"] == "linear":
        return 1.0 / d[0]
    if case["model"] == "softmax":
        return 0.8 / d[0]
    return 0.003 * min(1.0, 3072 / d[0]) if case["model"] == "cnn" else 0.6 / max(d[:-1])


class _State:
    """What a training program holds: dataset, workspace and handles."""

    def __init__(self, case, seed):
        self.case = case
        self.handles, self.batch = [], None
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        d = [int(x) for x in case["dims"].split()]
        shapes = _shapes(case)
        if case["model"] == "linear":
            mu = torch.randn(d[0], generator=gen, device="cuda")
        else:
            mu = torch.randn(_classes(case), d[0], generator=gen, device="cuda")
        self.X, self.y = _data(case, case["M"], gen, mu)
        if case["rows"]:
            self.X_eval, self.y_eval = _data(case, case["rows"], gen, mu)
        parts = []
        for r, c in shapes:
            if case["model"] in ("linear", "softmax"):
                parts.append(torch.zeros(r * c, device="cuda"))
            else:
                parts.append(torch.randn(r * c, generator=gen, device="cuda") * math.sqrt(2.0 / r))
            if case["model"] != "linear":
                parts.append(torch.zeros(c, device="cuda"))
        self.w0 = torch.cat(parts)
        self.P = self.w0.numel()
        K, N = case["K"], case["N"]
        cfgs = []
        for s in range(case["S"]):
            cfgs.append(lib.make_config(dict(
                model=MODEL_OF[case["model"]], dims=d, x_dtype=1 if case["model"] == "mlp" else 0, N=N, M=case["M"],
                B=case["B"], K0=K, k_mode=1, tau_mode=0, tau_cap=case["tau_cap"], a=case["tau_cap"] - N // K,
                lr=_learning_rate(case), sa_penalty=case["sa"], time_dist=1 if case["times"] == "pareto" else 0,
                time_param=1.5 if case["times"] == "pareto" else 0.0, n_slow=case["slow"],
                slow_factor=5.0 if case["slow"] else 1.0, seed_sim=seed * 4099 + 17 * s + 1, U=case["U"])))
        need = (lib.abs_workspace_size(cfgs[0]) + 255) // 256 * 256
        self.ring = case["tau_cap"] + 3                       # model versions kept; round t's model is version t
        self.slot = (self.P + 63) // 64 * 64                  # floats between them
        self.ws = torch.empty(case["S"], need, dtype=torch.uint8, device="cuda")
        stream = torch.cuda.current_stream().cuda_stream
        torch.cuda.synchronize()
        for s, cfg in enumerate(cfgs):
            self.handles.append(lib.abs_create(cfg, self.X.data_ptr(), self.y.data_ptr(), self.w0.data_ptr(),
                                               self.ws[s].data_ptr(), need, stream))
        if case["S"] > 1:
            n = lib.abs_batch_workspace_size(self.handles)
            self.batch_ws = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
            self.batch = lib.abs_batch_create(self.handles, self.batch_ws.data_ptr() if n else 0, n)
        if case["rows"]:
            # the model that is evaluated has a few rounds behind it
            lib.abs_round(self.handles[0], 3)
        self.t = lib.abs_rounds_done(self.handles[0])
        self.models = self.ws.view(torch.float32)[:, :self.ring * self.slot].view(case["S"], self.ring, self.slot)

    def __del__(self):
        if self.batch is not None:
            lib.abs_batch_destroy(self.batch)
        for h in self.handles:
            lib.abs_destroy(h)


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    case = s.case
    if case["rows"]:
        return lib.abs_evaluate(s.handles[0], -1, s.X_eval.data_ptr(), s.y_eval.data_ptr(), case["rows"])
    n = case["rounds"]
    if s.batch is not None:
        lib.abs_batch_round(s.batch, n)
        s.t += n
        return s.models[:, s.t % s.ring, :s.P]
    lib.abs_round(s.handles[0], n)
    t0, s.t = s.t, s.t + n
    trace = lib.abs_trace(s.handles[0], t0, s.t, case["N"])
    losses = trace[:, LOSS_WORD].copy().view(np.float32)      # the one word of a record that is a float
    trace[:, LOSS_WORD] = 0
    return s.models[0, s.t % s.ring, :s.P], trace, losses


def work(case):
    """Every minibatch row read once, the model of each round read and written once; the products of the
    forward and backward pass."""
    d = [int(x) for x in case["dims"].split()]
    shapes = _shapes(case)
    row_bytes = d[0] * (2 if case["model"] == "mlp" else 4) + 4
    P = _params(case)
    if case["model"] == "cnn":
        C0, k = d[6], d[7]
        S = math.isqrt(d[0] // C0)
        o1 = S - k + 1
        o2 = o1 // 2 - k + 1
        macs = [o1 * o1 * shapes[0][0] * d[1], o2 * o2 * shapes[1][0] * d[2]] + [r * c for r, c in shapes[2:]]
        # backward: the gradient of a pooled map reaches one position of each window
        train = 2.0 * (sum(macs) + macs[0] / 4 + 2 * macs[1] / 4 + 2 * sum(macs[2:]))
    else:
        macs = [r * c for r, c in shapes]
        train = 2.0 * (3 * sum(macs) - macs[0])
    if case["rows"]:
        return {"bytes": float(case["rows"] * row_bytes + P * (2 if case["model"] == "mlp" else 4)),
                "flops": 2.0 * case["rows"] * sum(macs)}
    samples = case["rounds"] * case["S"] * case["K"] * case["B"] * case["U"]
    return {"bytes": float(samples * row_bytes + case["rounds"] * case["S"] * 8.0 * P), "flops": samples * train}


def tolerance(case):
    """Four times what the same path shows with its sums in another order (contractions walked backwards,
    other splits, reductions and uploads in reverse), the largest of 54 cases: fp32 regression 1e-7, the
    convolutional model 2e-6 (elements 8e-5: a pooling window at a tie), bf16 networks 4e-5 (a sum that
    lands on the other side of a rounding point moves an activation by one bf16 step).  An evaluation
    also counts hits: one row at a tie is 1 / rows of the accuracy."""
    rel, most = {"linear": (4e-7, 2e-6), "softmax": (4e-7, 2e-6), "cnn": (1e-5, 4e-4), "mlp": (1.6e-4, 1e-3)}[case["model"]]
    if case["rows"]:
        rel = most = max(rel, 4.0 / case["rows"])
    return {"rel": rel, "max": most}
