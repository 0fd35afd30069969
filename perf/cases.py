"""Performance cases of the library: the work its users have it do, through the
public Python entry points, from the smallest training run to the largest
fitness evaluation.

A case is a dict of plain values.  Its "kind" names the call:

  run        a whole training run of a small problem: init_population, run
  step       one generation of a large run from a given population: step
  screened   one generation with a fitness surrogate attached: step
  fitness    the errors of a population over the training set: Game.fitness
  batch      many independent runs of uneven sizes together: Batch.init, run
  predict    model outputs of chromosomes on new patterns: Game.predict
  classify   class counts of chromosomes on new patterns: Game.classify
  rescore    float64 errors on a validation set: Game.rescore64
  trig_sums  per-pattern sums of the shared-gene model: game_trig_sums

Sizes follow the workloads of bench.py and paper_1304_0597_amd/datagen.py
(2,000 x 7; the paper-shaped 2,100 x 11 and its replicated sizes;
200,000 x 20; 1,000,000 x 32; the batched runs).
"""
import math
import random

import torch

from paper_1304_0597_amd import game as gg

BASES = {"chebyshev": 0, "legendre": 1, "power": 2, "trig": 3}
ERRORS = {"mse": 0, "rmse": 1, "tmse": 2}
SELECTIONS = {"tournament": 0, "ranking": 1, "roulette": 2}
TMSE_R = 0.49


def listed():
    return [
        # A whole training run on a small catalogue (the smallest workload of
        # bench.py): each generation is microseconds of arithmetic, so
        # launches and latency count.
        dict(name="run small", kind="run", basis="chebyshev", degree=4, patterns=2000, features=7,
             population=50, error="mse", generations=100, selection="tournament"),
        # The paper's own training run: the shared-gene trigonometric model
        # (degree 4: 8 per-pattern sums) on 2,100 sources, 23 chromosomes,
        # thresholded error.
        dict(name="run shared", kind="run", basis="power", degree=1, patterns=2100, features=8,
             population=23, error="tmse", generations=1000, selection="tournament"),
        # One generation of the same model on the paper's largest replicated
        # set (512 MB; degree 8: 16 sums): reading the data set counts.
        dict(name="step shared large", kind="step", basis="power", degree=1, patterns=7168000,
             features=16, population=23, error="tmse", selection="tournament", spread=0.05),
        # One generation of the throughput workload: 200,000 x 20, Legendre
        # degree 8 (161 genes), population 2,048.
        dict(name="step scale", kind="step", basis="legendre", degree=8, patterns=200000,
             features=20, population=2048, error="mse", selection="tournament", spread=0.2),
        # A population's errors under the paper's trigonometric expansion, at
        # sizes that are multiples of nothing.
        dict(name="fitness trig ragged", kind="fitness", basis="trig", degree=5, patterns=100003,
             features=13, population=777, n=777, error="rmse", precision="fp32", spread=0.1),
        # The precision form at its full size: 1,000,000 x 32, Chebyshev
        # degree 8 (257 genes), population 4,096, bfloat16 operands.
        dict(name="fitness bf16", kind="fitness", basis="chebyshev", degree=8, patterns=1000000,
             features=32, population=4096, n=4096, error="mse", precision="bf16", spread=0.2),
        # Independent runs of uneven sizes trained together (sizes drawn as
        # the batched workload's).
        dict(name="batch", kind="batch", runs=48, shapes=3, generations=10),
        # The model's outputs on a large new catalogue: the best chromosome
        # and its runners-up.
        dict(name="predict", kind="predict", basis="legendre", degree=8, patterns=1000000,
             features=20, population=64, n=8, spread=0.1),
        # Figures of merit of a small trained population on a held-out set.
        dict(name="classify", kind="classify", basis="trig", degree=4, patterns=2100, features=11,
             population=23, n=23, spread=0.1),
        # Validation of a run's best chromosome in float64, as every few
        # generations of a run to a validation target.
        dict(name="rescore", kind="rescore", basis="chebyshev", degree=8, patterns=250000,
             features=32, population=64, n=1, error="mse", spread=0.1),
        # One surrogate-screened generation: archive, 48 training steps,
        # oversampled offspring, audit, screening.
        dict(name="screened", kind="screened", basis="chebyshev", degree=8, patterns=200000,
             features=20, population=2048, error="mse", precision="bf16", spread=0.05),
        # The gene-independent sums of the shared model, once per data set
        # (the paper's 128 MB size, degree 4).
        dict(name="trig sums", kind="trig_sums", patterns=1792000, features=11, degree=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; sizes log-uniform, mostly odd."""
    kind = rng.choice(["run", "run", "step", "step", "fitness", "fitness", "batch", "predict",
                       "classify", "rescore", "screened", "trig_sums"])
    basis = rng.choice(["chebyshev", "legendre", "power", "trig"])
    selection = rng.choice(["tournament", "tournament", "ranking", "roulette"])
    error = rng.choice(["mse", "mse", "rmse", "tmse"])
    spread = round(math.exp(rng.uniform(math.log(0.03), math.log(0.3))), 3)
    if kind == "run":
        return dict(kind=kind, basis=basis, degree=rng.randint(1, 6), features=rng.randint(3, 16),
                    patterns=_log(rng, 500, 20000), population=_log(rng, 20, 300), error=error,
                    generations=_log(rng, 50, 1000), selection=selection)
    if kind == "batch":
        return dict(kind=kind, runs=rng.randint(4, 48), shapes=rng.randint(4, 10 ** 6),
                    generations=rng.randint(4, 10))
    if kind == "trig_sums":
        return dict(kind=kind, patterns=_log(rng, 2000, 1792000), features=rng.randint(4, 20),
                    degree=rng.randint(1, 10))
    if kind == "screened":
        return dict(kind=kind, basis=rng.choice(["chebyshev", "legendre"]), degree=rng.randint(3, 8),
                    patterns=_log(rng, 10000, 200000), features=rng.randint(5, 20),
                    population=_log(rng, 512, 2048), error="mse", precision="bf16", spread=spread)
    terms = {"trig": 2}.get(basis, 1)
    degree = rng.randint(1, 10)
    features = rng.randint(4, max(5, min(40, 320 // (terms * degree))))
    shape = dict(kind=kind, basis=basis, degree=degree, features=features, spread=spread)
    if kind in ("predict", "classify"):
        return dict(shape, patterns=_log(rng, 1000, 1000000), population=64, n=_log(rng, 1, 24))
    if kind == "rescore":
        return dict(shape, patterns=_log(rng, 1000, 250000), population=64, n=rng.randint(1, 4),
                    error=error)
    population = _log(rng, 100, 3000)
    patterns = min(_log(rng, 2000, 500000),
                   int(3.0e11 / (2.0 * population * terms * degree * features)))
    shape.update(patterns=max(patterns, 500), population=population, error=error)
    if kind == "step":
        return dict(shape, selection=selection)
    n = population if rng.random() < 0.6 else rng.randint(1, population)
    return dict(shape, n=n, precision=rng.choice(["fp32", "fp32", "bf16"]))


# ------------------------------------------------------------------ inputs
def _terms(case):
    return (2 if case["basis"] == "trig" else 1) * case["features"] * case["degree"]


def _expand(X, basis, degree):
    """Expansion of X in float64, [rows, terms] in the order of the genes."""
    x = X.double()
    if basis == "trig":
        j = torch.arange(1, degree + 1, device=X.device, dtype=torch.float64)
        ang = x[:, :, None] * j
        return torch.cat([ang.cos(), ang.sin()], dim=2).reshape(X.shape[0], -1)
    cols, prev, cur = [], torch.ones_like(x), x
    for j in range(1, degree + 1):
        cols.append(cur)
        if basis == "chebyshev":
            nxt = 2 * x * cur - prev
        elif basis == "legendre":
            nxt = ((2 * j + 1) * x * cur - j * prev) / (j + 1)
        else:
            nxt = x * cur
        prev, cur = cur, nxt
    return torch.stack(cols, dim=2).reshape(X.shape[0], -1)


def _outputs(X, genes, basis, degree, rows=65536):
    """Model outputs in float64, [rows, chromosomes], block by block."""
    w = genes.double()
    for r in range(0, X.shape[0], rows):
        yield r, w[:, 0] + _expand(X[r:r + rows], basis, degree) @ w[:, 1:].T.contiguous()


def _errors(X, t, genes, basis, degree, error):
    """Errors of the chromosomes over (X, t) in float64."""
    total = torch.zeros(genes.shape[0], dtype=torch.float64, device=X.device)
    rows = max(1024, min(65536, (1 << 28) // genes.shape[0]))
    for r, out in _outputs(X, genes, basis, degree, rows):
        res = out - t[r:r + rows, None].double()
        sq = res * res
        if error == "tmse":
            sq = torch.where(res.abs() > TMSE_R, sq, torch.zeros_like(sq))
        total += sq.sum(0)
    mean = total / X.shape[0]
    return mean.sqrt() if error == "rmse" else mean


def _data(gen, patterns, features, basis, degree, error, binary=False):
    """Patterns, targets and the teacher's genes: features in [-1, 1] (in
    radians up to pi for the trigonometric expansion), targets a random
    teacher plus noise, or its 0/1 labels with 5 % flips."""
    dev = "cuda"
    X = torch.rand((patterns, features), generator=gen, device=dev) * 2 - 1
    if basis == "trig":
        X *= math.pi
    terms = (2 if basis == "trig" else 1) * features * degree
    teacher = torch.rand(terms + 1, generator=gen, device=dev) * 2 - 1
    t = torch.empty(patterns, device=dev)
    for r, out in _outputs(X, teacher[None], basis, degree):
        t[r:r + out.shape[0]] = out[:, 0].float()
    if binary or error == "tmse":
        flip = torch.rand(patterns, generator=gen, device=dev) < 0.05
        t = ((t > t.mean()) ^ flip).float()
        teacher = teacher * (0.3 / math.sqrt(terms))
        teacher[0] = 0.5
    else:
        t += 0.05 * torch.randn(patterns, generator=gen, device=dev)
    return X, t, teacher


def _population(gen, teacher, n, spread):
    """Chromosomes of a run under way: scattered about the teacher."""
    noise = torch.randn((n, teacher.numel()), generator=gen, device="cuda")
    return (teacher + spread * noise).clamp(-1, 1).contiguous()


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


def _config(case, **kw):
    return gg.config(basis=BASES[case["basis"]], degree=case["degree"],
                     population=case["population"], error_fn=ERRORS[case.get("error", "mse")],
                     precision=gg.GAME_BF16 if case.get("precision") == "bf16" else gg.GAME_FP32,
                     selection=SELECTIONS[case.get("selection", "tournament")],
                     tmse_R=TMSE_R, target=-1.0, **kw)


def _shapes(case):
    """Sizes of a batch's runs, as the batched workload draws them."""
    rng = random.Random(case["shapes"])
    out = []
    for _ in range(case["runs"]):
        patterns = _log(rng, 1000, 200000)
        features, degree = rng.randint(4, 64), rng.randint(2, 10)
        out.append(dict(patterns=patterns, features=features, degree=degree,
                        population=rng.randint(32, 1024),
                        basis=rng.choice(["chebyshev", "power"]), error="mse"))
    return out


def _inputs(case, seed):
    """Data set and chromosomes of a case, from the seed alone."""
    gen = _generator(seed)
    binary = case["kind"] == "classify"
    X, t, teacher = _data(gen, case["patterns"], case["features"], case["basis"], case["degree"],
                          case.get("error", "mse"), binary)
    n = case.get("n", case["population"])
    return X, t, _population(gen, teacher, n, case["spread"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "trig_sums":
        X = torch.rand((case["patterns"], case["features"]), generator=_generator(seed),
                       device="cuda") * 2 - 1
        return dict(case=case, X=X)
    if kind == "batch":
        gen = _generator(seed)
        problems, cfgs = [], []
        for i, s in enumerate(_shapes(case)):
            X, t, _ = _data(gen, s["patterns"], s["features"], s["basis"], s["degree"], "mse")
            problems.append((X, t))
            cfgs.append(_config(s, seed=seed * 1000 + i, max_generations=case["generations"]))
        return dict(case=case, batch=gg.Batch(problems, cfgs))
    if kind == "run":
        X, t, _ = _data(_generator(seed), case["patterns"], case["features"], case["basis"],
                        case["degree"], case["error"])
        cfg = _config(case, seed=seed, tournament_k=4, max_generations=case["generations"])
        return dict(case=case, game=gg.Game(cfg, X, t))
    X, t, genes = _inputs(case, seed)
    state = dict(case=case, genes=genes, X=X, t=t)
    if kind in ("predict", "classify", "rescore"):
        # a trained model's handle (over its own small training set) and the
        # new patterns it is applied to
        state["game"] = gg.Game(_config(case), X[:500].contiguous(), t[:500].contiguous())
        return state
    cfg = _config(case, seed=seed, max_generations=1 << 30)
    state["game"] = gg.Game(cfg, X, t)
    if kind == "screened":
        P, E = case["population"], cfg.elitism
        sc = gg.surrogate_config(seed=seed, min_archive=256, audit=min(256, P))
        state["surrogate"] = gg.Surrogate(sc, _terms(case) + 1, sc.oversample * (P - E))
        gg.game_attach_surrogate(state["game"].h, state["surrogate"].h)
    return state


# --------------------------------------------------------------------- run
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "trig_sums":
        return gg.game_trig_sums(state["X"], case["degree"])
    if kind == "batch":
        batch = state["batch"]
        batch.init()
        generations, _ = batch.run()
        trained = [batch.population(i) for i in range(case["runs"])]
        return {"generations": generations,
                "genes": torch.cat([g.reshape(-1) for g, _ in trained]),
                "fitness": torch.cat([f for _, f in trained])}
    game = state["game"]
    if kind == "run":
        game.init_population()
        generations, best, _ = game.run()
        genes, fitness = game.population()
        return {"generations": generations, "best": best, "genes": genes, "fitness": fitness}
    if kind in ("step", "screened"):
        game.set_population(state["genes"], 7)
        game.step()
        genes, fitness = game.population()
        return {"genes": genes, "fitness": fitness}
    if kind == "fitness":
        return game.fitness(state["genes"])
    if kind == "predict":
        return game.predict(state["genes"], state["X"])
    if kind == "classify":
        return game.classify(state["genes"], state["X"], state["t"])
    return game.rescore64(state["genes"], state["X"], state["t"])


# ----------------------------------------------------------- work and truth
def _evaluation(case, n):
    """Bytes and operations of the errors of n chromosomes over a data set:
    the contraction with the expansion, or for squared errors, where it is
    less, the quadratic form of the expansion's (symmetric) moment matrix."""
    K, rows = _terms(case) + 1, case["patterns"]
    flops = 2.0 * (K - 1) * n * rows
    if case.get("error", "mse") != "tmse":
        flops = min(flops, 1.0 * rows * (K + 1) ** 2 + 2.0 * n * (K + 1) ** 2)
    return {"bytes": 4.0 * (rows * (case["features"] + 1) + n * K + n), "flops": flops}


def _generations(case, count):
    """`count` generations in one call: the data set is read once at least;
    a generation reads its population and writes the next one."""
    one = _evaluation(case, case["population"])
    K, rows, P = _terms(case) + 1, case["patterns"], case["population"]
    flops = count * 2.0 * (K - 1) * P * rows
    if case["error"] != "tmse":
        flops = min(flops, 1.0 * rows * (K + 1) ** 2 + count * 2.0 * P * (K + 1) ** 2)
    return {"bytes": one["bytes"] + count * 8.0 * P * K, "flops": flops}


def work(case):
    kind = case["kind"]
    if kind == "trig_sums":
        rows, N, d = case["patterns"], case["features"], case["degree"]
        return {"bytes": 4.0 * rows * (N + 2 * d), "flops": rows * N * (40.0 + 6.0 * d)}
    if kind == "batch":
        each = [_generations(s, case["generations"] + 1) for s in _shapes(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    if kind == "run":
        return _generations(case, case["generations"] + 1)
    if kind == "step":
        return _generations(case, 1)
    if kind == "screened":
        w = _generations(case, 1)
        K, H = _terms(case) + 1, 256
        # 48 training steps of 1,024 rows (forward, two backward products)
        # and the network over 8 children per kept one
        w["flops"] += 2.0 * (K * H + H * H) * (3 * 48 * 1024 + 8 * case["population"])
        w["bytes"] += 8 * 4.0 * case["population"] * K + 48 * 4.0 * (1024 * K + 3 * (K + H) * H)
        return w
    K, rows, n = _terms(case) + 1, case["patterns"], case["n"]
    if kind == "fitness":
        return _evaluation(case, n)
    if kind == "rescore":
        return {"bytes": 4.0 * (rows * (case["features"] + 1) + n * K) + 8.0 * n,
                "flops": 2.0 * (K - 1) * n * rows}
    out = 4.0 * n * rows if kind == "predict" else 4.0 * rows + 32.0 * n
    return {"bytes": 4.0 * (rows * case["features"] + n * K) + out, "flops": 2.0 * (K - 1) * n * rows}


def exact(case, seed):
    """What run() returns, in float64; None for evolved genes (they follow
    from draws and comparisons) and for whole numbers."""
    kind = case["kind"]
    if kind in ("batch", "run", "classify"):
        return None
    if kind == "trig_sums":
        X = prepare(case, seed)["X"].double()
        cols = [(X * j).cos().sum(1) for j in range(1, case["degree"] + 1)]
        cols += [(X * j).sin().sum(1) for j in range(1, case["degree"] + 1)]
        return torch.stack(cols, dim=1)
    X, t, genes = _inputs(case, seed)
    if kind == "predict":
        blocks = [out.T for _, out in _outputs(X, genes, case["basis"], case["degree"])]
        return torch.cat(blocks, dim=1).contiguous()
    err = _errors(X, t, genes, case["basis"], case["degree"], case["error"])
    if kind in ("step", "screened"):
        return {"genes": None, "fitness": err}
    return err
