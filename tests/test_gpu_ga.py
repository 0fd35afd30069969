"""Bit-exactness of the device genetic operators against the oracle given the
same inputs, and the device training loop against the oracle driven by the
device's own fitness vectors."""
import numpy as np
import pytest

from fitness_plan import plan
from oracle import ga as oga
from oracle import game as og
from paper_1304_0597_amd import datagen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gg():
    from paper_1304_0597_amd import game
    game.lib()
    return game


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def oracle_cfg(c):
    return oga.GAConfig(population=c.population, tournament_k=c.tournament_k, elitism=c.elitism,
                        elite_mode=c.elite_mode, p_crossover=c.p_crossover,
                        p_mutation=c.p_mutation, sigma_mutation=c.sigma_mutation, seed=c.seed,
                        init_mode=c.init_mode, selection=c.selection)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("P,K", [(1, 1), (50, 29), (130, 161), (7, 700)])
def test_init_bit_exact(gg, mode, P, K):
    c = gg.config(population=max(P, 2), init_mode=mode, seed=12345)
    c.population = P
    out = torch.empty((P, K), dtype=torch.float32, device="cuda")
    gg.game_init_genes(c, K, out)
    torch.cuda.synchronize()
    ref = oga.init_population(P, K, 12345, mode)
    assert np.array_equal(bits(out.cpu().numpy()), bits(ref))


@pytest.mark.parametrize("n", [1, 2, 3, 50, 1000, 2048, 4096, 8192])
def test_rank_bit_exact(gg, n):
    rng = np.random.default_rng(n)
    f = rng.choice(np.array([0.5, 0.25, 1.0, 2.0, np.inf], np.float32), n) if n > 10 else \
        rng.uniform(0, 1, n).astype(np.float32)
    if n > 10:
        f[rng.choice(n, n // 3, replace=False)] = rng.uniform(0, 3, n // 3).astype(np.float32)
        f[rng.choice(n, max(1, n // 50), replace=False)] = np.nan
        f[rng.choice(n, max(1, n // 50), replace=False)] = -0.0
    fd = torch.from_numpy(f).cuda()
    order = torch.empty(n, dtype=torch.int32, device="cuda")
    gg.game_rank(fd, n, order)
    torch.cuda.synchronize()
    assert np.array_equal(order.cpu().numpy(), oga.rank_order(f))


GA_CASES = [
    # P, K, k, E, mode, pc, pm, sigma
    (50, 29, 3, 2, 0, 0.9, 0.05, 0.1),
    (51, 29, 3, 2, 1, 0.9, 0.05, 0.1),
    (2048, 161, 3, 2, 0, 0.9, 0.05, 0.1),
    (4096, 257, 4, 2, 0, 0.9, 0.2, 0.1),
    (33, 2, 1, 0, 0, 1.0, 1.0, 2.0),
    (40, 700, 4, 5, 1, 0.0, 0.0, 0.1),
    (40, 13, 40, 1, 0, 1.0, 0.0, 0.1),
    (9, 17, 64 // 8, 3, 1, 0.5, 0.5, 0.7),
    # tournaments longer than one Philox block of words, up to k = P
    (200, 31, 100, 2, 0, 0.9, 0.05, 0.1),
    (70, 9, 70, 1, 1, 1.0, 0.5, 0.3),
]


@pytest.mark.parametrize("case", GA_CASES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("generation", [1, 7])
def test_ga_next_bit_exact(gg, case, generation):
    P, K, k, E, mode, pc, pm, sigma = case
    rng = np.random.default_rng(P * K + generation)
    pop = rng.uniform(-1, 1, (P, K)).astype(np.float32)
    fit = rng.uniform(0, 1, P).astype(np.float32)
    fit[rng.choice(P, max(1, P // 10), replace=False)] = fit[0]          # ties
    fit[rng.choice(P, max(1, P // 20), replace=False)] = np.nan          # NaN
    c = gg.config(population=P, tournament_k=k, elitism=E, elite_mode=mode, p_crossover=pc,
                  p_mutation=pm, sigma_mutation=sigma, seed=777)
    ws = torch.empty(gg.game_ga_workspace_size(c), dtype=torch.uint8, device="cuda")
    out = torch.empty((P, K), dtype=torch.float32, device="cuda")
    gg.game_ga_next(c, K, torch.from_numpy(pop).cuda(), torch.from_numpy(fit).cuda(),
                    generation, out, ws)
    torch.cuda.synchronize()
    ref = oga.ga_next(pop, fit, generation, oracle_cfg(c))
    got = out.cpu().numpy()
    assert np.array_equal(bits(got), bits(ref)), np.argwhere(bits(got) != bits(ref))[:5]


def _small_game(gg, **kw):
    prob = datagen.small()
    c = gg.config(basis=prob.basis, degree=prob.degree, population=prob.population, seed=3,
                  max_generations=100, target=0.0)
    for k, v in kw.items():
        setattr(c, k, v)
    g = gg.Game(c, torch.from_numpy(prob.X).cuda(), torch.from_numpy(prob.t).cuda())
    return prob, c, g


def test_steps_follow_oracle_given_device_fitness(gg):
    """Each generation built on the device equals the oracle's generation
    built from the same population and the device's fitness vector; the
    device fitness matches the float64 oracle."""
    prob, c, g = _small_game(gg)
    g.init_population()
    pop0, _ = g.population()
    ref0 = oga.init_population(c.population, g.n_genes, c.seed, c.init_mode)
    assert np.array_equal(bits(pop0.cpu().numpy()), bits(ref0))
    ocfg = oracle_cfg(c)
    for gen in range(12):
        pop_g, _ = g.population()
        g.step()
        _, fit_g = g.population()
        pop_next, _ = g.population()
        pop_g, fit_g, pop_next = (x.cpu().numpy() for x in (pop_g, fit_g, pop_next))
        ref_f = og.fitness(prob.X, prob.t, pop_g, prob.basis, prob.degree)
        assert np.all(np.abs(fit_g - ref_f) <= 1e-5 * ref_f + 1e-7)
        ref_next = oga.ga_next(pop_g, fit_g, gen + 1, ocfg)
        assert np.array_equal(bits(pop_next), bits(ref_next)), gen
    st = g.state()
    assert st["generation"] == 12 and st["stopped"] == 0
    g.close()


def test_graph_run_equals_eager_steps(gg):
    _, c, g1 = _small_game(gg)
    g1.init_population()
    gens, best, err = g1.run(max_generations=30, target=0.0)
    assert gens == 30
    _, _, g2 = _small_game(gg, max_generations=30)
    g2.init_population()
    for _ in range(31):
        g2.step()
    p1, f1 = g1.population()
    p2, f2 = g2.population()
    assert np.array_equal(bits(p1.cpu().numpy()), bits(p2.cpu().numpy()))
    assert np.array_equal(bits(f1.cpu().numpy()), bits(f2.cpu().numpy()))
    st = g2.state()
    assert st["stopped"] == 1 and st["generation"] == 30
    assert abs(st["best_error"] - err) == 0.0
    assert np.array_equal(bits(best), bits(p1.cpu().numpy()[st["best_index"]]))
    g1.close()
    g2.close()


def test_run_improves_and_keeps_elite(gg):
    prob, c, g = _small_game(gg)
    g.init_population()
    hist = []
    for _ in range(20):
        g.step()
        hist.append(g.state()["best_error"])
    assert all(b <= a for a, b in zip(hist, hist[1:]))
    assert hist[-1] < hist[0]
    g.close()


def test_target_stops_at_generation_zero(gg):
    _, c, g = _small_game(gg)
    g.init_population()
    gens, _, err = g.run(max_generations=50, target=1e9)
    assert gens == 0 and err < 1e9
    g.close()


def test_resume_is_bit_exact(gg):
    _, c, g1 = _small_game(gg)
    g1.init_population()
    g1.run(max_generations=20, target=0.0)
    pop_full, _ = g1.population()
    _, _, g2 = _small_game(gg)
    g2.init_population()
    g2.run(max_generations=10, target=0.0)
    saved, _ = g2.population()
    saved = saved.clone()
    _, _, g3 = _small_game(gg)
    g3.set_population(saved, 10)
    gens, _, _ = g3.run(max_generations=20, target=0.0)
    pop_res, _ = g3.population()
    assert gens == 20
    assert np.array_equal(bits(pop_res.cpu().numpy()), bits(pop_full.cpu().numpy()))
    for g in (g1, g2, g3):
        g.close()


def test_run_resumes_when_limits_are_raised(gg):
    """A run stopped by its generation limit continues, under a higher
    limit, exactly as one uninterrupted run: run(10) then run(20) ends where
    run(20) ends, bit for bit; a second call whose limits still hold does
    nothing."""
    _, _, g1 = _small_game(gg)
    g1.init_population()
    gens1, best1, err1 = g1.run(max_generations=20, target=0.0)
    _, _, g2 = _small_game(gg)
    g2.init_population()
    assert g2.run(max_generations=10, target=0.0)[0] == 10
    assert g2.run(max_generations=10, target=0.0)[0] == 10          # still stopped
    assert g2.state()["stopped"] == 1
    gens2, best2, err2 = g2.run(max_generations=20, target=0.0)
    assert gens1 == gens2 == 20 and err1 == err2
    assert np.array_equal(bits(best1), bits(best2))
    for a, b in zip(g1.population(), g2.population()):
        assert np.array_equal(bits(a.cpu().numpy()), bits(b.cpu().numpy()))
    # a target that the stopped run's best already meets: nothing runs
    gens3, _, err3 = g2.run(max_generations=40, target=err2 * 2)
    assert gens3 == 20 and err3 == err2
    g1.close()
    g2.close()


def test_run_stops_queuing_after_an_early_stop(gg):
    """A target reached long before the generation limit: the run stops at
    the same generation as single steps do, and a very large limit does not
    make game_run queue work for every remaining generation (it returns in
    well under the time that would take)."""
    import time
    _, _, g1 = _small_game(gg)
    g1.init_population()
    g1.run(max_generations=30, target=0.0)
    target = g1.state()["best_error"]
    _, _, g2 = _small_game(gg)
    g2.init_population()
    t0 = time.perf_counter()
    gens, _, err = g2.run(max_generations=(1 << 31) - 1, target=target)
    elapsed = time.perf_counter() - t0
    assert gens <= 30 and err <= target
    assert elapsed < 20.0
    g1.close()
    g2.close()


SELECTION_CASES = [
    # P, K, E, mode, pc, pm, sigma
    (50, 29, 2, 0, 0.9, 0.05, 0.1),
    (2048, 161, 2, 1, 0.9, 0.05, 0.1),
    (4096, 257, 2, 0, 0.9, 0.2, 0.1),
    (33, 5, 0, 0, 1.0, 1.0, 2.0),
    (7, 11, 3, 1, 0.5, 0.5, 0.7),
]


@pytest.mark.parametrize("selection", [1, 2])
@pytest.mark.parametrize("case", SELECTION_CASES, ids=lambda c: "-".join(map(str, c)))
def test_ranking_and_roulette_bit_exact(gg, selection, case):
    P, K, E, mode, pc, pm, sigma = case
    rng = np.random.default_rng(P + K + selection)
    pop = rng.uniform(-1, 1, (P, K)).astype(np.float32)
    fit = rng.uniform(0, 1, P).astype(np.float32) ** 3
    fit[rng.choice(P, max(1, P // 10), replace=False)] = fit[0]          # ties
    fit[rng.choice(P, max(1, P // 20), replace=False)] = np.inf
    fit[rng.choice(P, max(1, P // 20), replace=False)] = np.nan
    c = gg.config(population=P, elitism=E, elite_mode=mode, p_crossover=pc, p_mutation=pm,
                  sigma_mutation=sigma, seed=99, selection=selection)
    ws = torch.empty(gg.game_ga_workspace_size(c), dtype=torch.uint8, device="cuda")
    out = torch.empty((P, K), dtype=torch.float32, device="cuda")
    gg.game_ga_next(c, K, torch.from_numpy(pop).cuda(), torch.from_numpy(fit).cuda(), 3, out, ws)
    torch.cuda.synchronize()
    ref = oga.ga_next(pop, fit, 3, oracle_cfg(c))
    assert np.array_equal(bits(out.cpu().numpy()), bits(ref))


def test_roulette_all_infinite_is_uniform_and_exact(gg):
    P, K = 40, 9
    pop = np.random.default_rng(1).uniform(-1, 1, (P, K)).astype(np.float32)
    fit = np.full(P, np.inf, np.float32)
    c = gg.config(population=P, elitism=1, seed=5, selection=2)
    ws = torch.empty(gg.game_ga_workspace_size(c), dtype=torch.uint8, device="cuda")
    out = torch.empty((P, K), dtype=torch.float32, device="cuda")
    gg.game_ga_next(c, K, torch.from_numpy(pop).cuda(), torch.from_numpy(fit).cuda(), 1, out, ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(out.cpu().numpy()), bits(oga.ga_next(pop, fit, 1, oracle_cfg(c))))


@pytest.mark.parametrize("selection", [1, 2])
def test_selection_modes_in_the_loop(gg, selection):
    prob, c, g = _small_game(gg, selection=selection)
    g.init_population()
    ocfg = oracle_cfg(c)
    for gen in range(6):
        pop_g, _ = g.population()
        g.step()
        _, fit_g = g.population()
        pop_next, _ = g.population()
        pop_g, fit_g, pop_next = (x.cpu().numpy() for x in (pop_g, fit_g, pop_next))
        ref_next = oga.ga_next(pop_g, fit_g, gen + 1, ocfg)
        assert np.array_equal(bits(pop_next), bits(ref_next)), gen
    g.close()


# (NP, N, d, P) and the pattern splits the plan gives them: at most 64 and
# more than 64, with 32-, 64- and (40,000 patterns) 128-chromosome tiles, ragged
# last workgroups.
SPLIT_SHAPES = [((2000, 7, 4, 50), "8-splits"), ((5000, 8, 4, 300), "20-splits-128-wide"),
                ((100000, 5, 3, 50), "391-splits"), ((40000, 8, 4, 300), "79-splits-128-wide")]


@pytest.mark.parametrize("error_fn", [0, 1], ids=["MSE", "RMSE"])
@pytest.mark.parametrize("shape", [s for s, _ in SPLIT_SHAPES], ids=[i for _, i in SPLIT_SHAPES])
def test_step_errors_are_the_fitness_launch_bits(gg, shape, error_fn):
    """The errors a generation records (its split partials reduced by the
    evaluation epilogue) equal game_fitness on the same population bit for
    bit: both add the same partials in the same order, on the path for at
    most 64 splits and on the one for more."""
    NP, N, d, P = shape
    rng = np.random.default_rng(NP + P)
    X = torch.from_numpy(rng.uniform(-1, 1, (NP, N)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(0, 1, NP).astype(np.float32)).cuda()
    c = gg.config(basis=1, degree=d, population=P, seed=5, max_generations=100, target=0.0,
                  error_fn=error_fn)
    g = gg.Game(c, X, t)
    g.init_population()
    for _ in range(2):
        pop, _ = g.population()
        g.step()
        _, fit = g.population()
        ref = g.fitness(pop)
        assert np.array_equal(bits(fit.cpu().numpy()), bits(ref.cpu().numpy()))
    g.close()


@pytest.mark.parametrize("case", [
    # (NP, N, d, P): smallest, odd population, the limits of the one-launch
    # tail (16,384 genes, 512 chromosomes, tournaments of 7) and one past each,
    # more than 64 pattern splits
    (1, 1, 1, 2, {}), (300, 5, 2, 23, dict(tournament_k=7)),
    (300, 5, 2, 23, dict(tournament_k=8)), (700, 31, 1, 512, dict(elitism=0)),
    (700, 31, 1, 511, dict(elite_mode=1, elitism=5)), (500, 63, 2, 129, dict(selection=1)),
    (500, 64, 2, 129, dict(selection=1)), (900, 3, 2, 513, dict(selection=2)),
    (20001, 8, 1, 23, dict(selection=2, elitism=1, elite_mode=1)),
    (20001, 8, 1, 23, dict(error_fn=2, p_mutation=1.0))],
    ids=lambda c: f"{c[0]}x{c[1]}-d{c[2]}-P{c[3]}-" + "-".join(f"{k}{v}" for k, v in c[4].items()))
def test_generation_tail_at_its_edges(gg, case):
    """Every generation equals the oracle's built from the device's errors,
    stepped and in a captured run; those errors are game_fitness's bits."""
    NP, N, d, P, kw = case
    rng = np.random.default_rng(NP + P)
    X = torch.from_numpy(rng.uniform(-1, 1, (NP, N)).astype(np.float32)).cuda()
    t = torch.from_numpy((rng.random(NP) < 0.5).astype(np.float32)).cuda()
    kw = dict(dict(tournament_k=min(3, P), elitism=min(2, P - 1)), **kw)
    c = gg.config(basis=0, degree=d, population=P, seed=7, max_generations=3, target=-1.0, **kw)
    g = gg.Game(c, X, t)
    g.init_population()
    for gen in range(3):
        pop, _ = g.population()
        ref = g.fitness(pop)
        g.step()
        nxt, fit = g.population()
        pop, ref, nxt, fit = (x.cpu().numpy() for x in (pop, ref, nxt, fit))
        assert np.array_equal(bits(fit), bits(ref)), gen
        assert np.array_equal(bits(nxt), bits(oga.ga_next(pop, fit, gen + 1, oracle_cfg(c)))), gen
    g.init_population()
    gens, _, _ = g.run()
    assert gens == 3
    assert np.array_equal(bits(g.population()[0].cpu().numpy()), bits(nxt))
    g.close()


@pytest.mark.parametrize("case", [
    # (NP, N, d, basis, P, generations): ends of 64-row units and 256-row tiles,
    # one and two column tiles, an odd last feature, 1 to 30 tiles, more genes
    # than threads, more generations than a launch, every basis and option
    (1, 1, 1, 0, 2, 3, {}), (64, 3, 2, 1, 32, 9, dict(selection=1)),
    (65, 2, 3, 3, 33, 9, dict(selection=2, elitism=0)),
    (256, 5, 1, 2, 64, 9, dict(error_fn=2)), (257, 4, 2, 3, 63, 9, dict(error_fn=1, elitism=5)),
    (2100, 8, 1, 2, 23, 1030, dict(error_fn=2)), (300, 7, 4, 0, 50, 9, dict(elite_mode=1)),
    (7500, 2, 1, 2, 5, 9, dict(tournament_k=5)), (4096, 1, 1, 2, 5, 9, dict(error_fn=3)),
    (100, 31, 1, 1, 40, 9, dict(tournament_k=7, p_mutation=1.0))],
    ids=lambda c: "x".join(map(str, c[:6])) + "-" + "-".join(f"{k}{v}" for k, v in c[6].items()))
def test_whole_runs_equal_their_generations(gg, case):
    """game_run ends with the bits that game_step reaches, on a first run, a
    continued one and one stopped by its target."""
    NP, N, d, basis, P, gens, kw = case
    rng = np.random.default_rng(NP + P)
    X = torch.from_numpy(rng.uniform(-1, 1, (NP, N)).astype(np.float32)).cuda()
    t = torch.from_numpy((rng.random(NP) < 0.5).astype(np.float32)).cuda()
    kw = dict(dict(tournament_k=min(3, P), elitism=min(2, P - 1)), **kw)
    c = gg.config(basis=basis, degree=d, population=P, seed=5, max_generations=gens, target=-1.0,
                  **kw)
    a, b = gg.Game(c, X, t), gg.Game(c, X, t)

    def same():
        (pa, fa), (pb, fb) = a.population(), b.population()
        assert np.array_equal(bits(pa.cpu().numpy()), bits(pb.cpu().numpy()))
        assert np.array_equal(bits(fa.cpu().numpy()), bits(fb.cpu().numpy()))

    a.init_population()
    b.init_population()
    done, _, _ = a.run()
    for _ in range(gens + 1):
        b.step()
    assert done == gens and a.state() == b.state()
    same()
    done, _, _ = a.run(max_generations=gens + 4)
    assert done == gens + 4
    # the continued run again, from the evaluated population by steps
    e = gg.Game(gg.config(basis=basis, degree=d, population=P, seed=5, max_generations=gens + 4,
                          target=-1.0, **kw), X, t)
    e.set_population(b.population()[0], gens)
    for _ in range(5):
        e.step()
    (pa, fa), (pe, fe) = a.population(), e.population()
    assert np.array_equal(bits(pa.cpu().numpy()), bits(pe.cpu().numpy()))
    assert np.array_equal(bits(fa.cpu().numpy()), bits(fe.cpu().numpy()))
    # a target that the first population meets
    a.init_population()
    done, _, _ = a.run(target=1e30)
    assert done == 0 and a.state()["stopped"]
    a.close()
    b.close()
    e.close()


@pytest.mark.parametrize("case", [
    # the largest population whose rank order is made inside the one-launch tail,
    # and one past it: ranking selection, the best kept, and both
    (700, 20, 4, 192, dict(selection=1)), (700, 20, 4, 193, dict(selection=1)),
    (700, 20, 4, 192, dict(elite_mode=1, elitism=3)), (700, 20, 4, 193, dict(elite_mode=1, elitism=3)),
    (700, 20, 4, 192, dict(selection=1, elite_mode=1, elitism=2)),
    (700, 20, 4, 193, dict(elite_mode=1, elitism=0))],
    ids=lambda c: f"{c[0]}x{c[1]}-d{c[2]}-P{c[3]}-" + "-".join(f"{k}{v}" for k, v in c[4].items()))
def test_generation_tail_with_its_rank_order(gg, case):
    test_generation_tail_at_its_edges(gg, case)


@pytest.mark.parametrize("case", [
    # partials summed inside the one-launch tail by 64 lanes a chromosome: 33, 47 and
    # 64 splits, the last with four rounds of the workgroup full
    (8193, 8, 1, 50, {}), (12000, 8, 1, 50, dict(error_fn=2)),
    (16384, 7, 2, 64, dict(selection=2)), (8200, 3, 2, 63, dict(selection=1, error_fn=1))],
    ids=lambda c: f"{c[0]}x{c[1]}-d{c[2]}-P{c[3]}-" + "-".join(f"{k}{v}" for k, v in c[4].items()))
def test_generation_tail_with_64_lanes_a_sum(gg, case):
    assert 33 <= plan(*case[:4]).splits <= 64
    test_generation_tail_at_its_edges(gg, case)
