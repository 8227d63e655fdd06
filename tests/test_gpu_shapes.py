"""GPU parity at the edges of the kernels' dispatch rules: shapes where a tile, a chunk or a row group ends in the
middle, each in lockstep with the CPU oracle (unroll bit for bit in fp32, update per parameter region)."""
import numpy as np
import pytest

from paper_2104_06272_amd import workloads as W
import parity as PT

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4
TOL_BF16 = 2e-2


@pytest.fixture(scope="module")
def gpu():
    from paper_2104_06272_amd import binding
    binding.load()
    return binding


def variant(name, hidden, B, T, dtype="fp32", **env):
    cfg = W.get(name, B=B, T=T)
    cfg["net"]["hidden"] = list(hidden)
    cfg["net"]["dtype"] = dtype
    cfg["env"] = dict(cfg["env"], **env)
    return cfg


def lockstep(gpu, orc, cfg, seed, updates=2, tol=TOL_F32):
    kind = cfg["env"]["kind"]
    print(f"[{kind}] hidden={cfg['net']['hidden']} B={cfg['B']} T={cfg['T']}", flush=True)
    g = gpu.Anakin(cfg, seed=seed)
    o = orc.Oracle(cfg, seed=seed)
    PT.assert_same_init(g, o, kind)
    for _ in range(updates):
        PT.sync_oracle_from_gpu(g, o)
        g.rollout(); o.rollout()
        PT.assert_rollout_equal(g, o, kind)
        PT.assert_final_state_equal(g, o, kind)
        g.learn(); o.learn()
        PT.assert_learn_close(g, o, tol)
    g.close()


def forced_lockstep(gpu, orc, cfg, seed, updates=2):
    """bf16 nets on the matrix-core path: the oracle samples and steps from the GPU's head outputs, which are checked
    against its own forward pass"""
    kind = cfg["env"]["kind"]
    print(f"[bf16 {kind}] hidden={cfg['net']['hidden']} B={cfg['B']} T={cfg['T']}", flush=True)
    g = gpu.Anakin(cfg, seed=seed)
    o = orc.Oracle(cfg, seed=seed)
    assert g.plan()["bf16_matrix_path"] == 1
    for _ in range(updates):
        PT.sync_oracle_from_gpu(g, o)
        g.rollout()
        tr = g.trajectory()
        o.rollout(forced_head=tr["head"])
        PT.assert_rollout_equal(g, o, kind, forced=True)
        PT.assert_final_state_equal(g, o, kind)
        PT.assert_heads_close(g, o, tr, TOL_BF16)
        g.learn(); o.learn()
        PT.assert_learn_close(g, o, TOL_BF16)
    g.close()


# one hidden layer of 64 or 128 units with many samples: every chunk's head gradient is summed
@pytest.mark.parametrize("name,hidden,B,T", [("catch_262144", 64, 512, 8), ("catch_262144", 128, 256, 16), ("pendulum_8192", 64, 1024, 4)])
def test_one_layer_many_samples(gpu, orc, name, hidden, B, T):
    lockstep(gpu, orc, variant(name, [hidden], B, T), 3)


# 32 units on Catch, few environments (returns, loss and backward pass in launches of their own): boards of two cells and of the
# most that fit, one block of 256 environments and several; the bias gradient is the paddle's row added up
@pytest.mark.parametrize("rows,cols,B,T", [(2, 1, 256, 1), (17, 6, 512, 7), (2, 51, 256, 5), (6, 8, 768, 4)])
def test_one_layer_of_32_units(gpu, orc, rows, cols, B, T):
    lockstep(gpu, orc, variant("catch_262144", [32], B, T, rows=rows, cols=cols, max_steps=rows - 1), 3)


# as many environments as the single launch of that update takes them from, which depends on T: time steps that end inside a
# chunk of four, a block of 256 environments to a workgroup (one less than a power of two of them, too) and, from 514 blocks, two
@pytest.mark.parametrize("rows,cols,B,T", [(6, 8, 18432, 1), (6, 8, 20480, 2), (4, 3, 53248, 2), (2, 1, 53248, 5), (17, 6, 53504, 3), (2, 51, 53248, 1),
                                           (4, 3, 131584, 3), (3, 2, 131584, 5)])
def test_one_layer_update_in_one_launch(gpu, orc, rows, cols, B, T):
    cfg = variant("catch_262144", [32], B, T, rows=rows, cols=cols, max_steps=rows - 1)
    g = gpu.Anakin(cfg, seed=1)
    blocks, splits = B // 256, g.plan()["splits"]
    assert splits[0] == splits[1] == (blocks if blocks <= 512 else blocks // 2), splits   # the single launch's workgroups
    g.close()
    lockstep(gpu, orc, cfg, 2)


# one hidden layer on Catch, its backward pass by tiles of 32 cells: boards of 2 cells up to the most of every width, on and
# off whole tiles, one unit of 16 samples, units that do not divide by the wavefronts or chunks, more samples than chunks of one
# unit take; the pendulum's blocks of 64 samples, whole and not, wavefronts without any
@pytest.mark.parametrize("name,hidden,rows,cols,B,T", [
    ("catch_262144", 32, 2, 1, 64, 1), ("catch_262144", 32, 17, 6, 64, 5), ("catch_262144", 32, 8, 8, 2112, 17), ("catch_262144", 32, 13, 5, 512, 3),
    ("catch_262144", 64, 17, 5, 48, 11), ("catch_262144", 64, 2, 1, 16, 3), ("catch_262144", 64, 10, 5, 2064, 17),
    ("catch_262144", 128, 8, 8, 80, 7), ("catch_262144", 128, 11, 3, 16, 1), ("catch_262144", 128, 10, 5, 1040, 17),
    ("catch_262144", 256, 9, 7, 80, 7), ("catch_262144", 256, 4, 4, 16, 1), ("catch_262144", 256, 10, 5, 1040, 17), ("catch_262144", 256, 8, 8, 48, 5),
    ("pendulum_8192", 256, 0, 0, 16, 1), ("pendulum_8192", 256, 0, 0, 80, 7), ("pendulum_8192", 256, 0, 0, 1040, 17),
    ("pendulum_8192", 32, 0, 0, 64, 1), ("pendulum_8192", 32, 0, 0, 192, 7), ("pendulum_8192", 32, 0, 0, 4160, 33),
    ("pendulum_8192", 64, 0, 0, 16, 1), ("pendulum_8192", 64, 0, 0, 80, 7), ("pendulum_8192", 64, 0, 0, 2064, 33),
    ("pendulum_8192", 128, 0, 0, 16, 3), ("pendulum_8192", 128, 0, 0, 112, 9), ("pendulum_8192", 128, 0, 0, 1040, 67)])
def test_one_layer_backward_in_one_launch(gpu, orc, name, hidden, rows, cols, B, T):
    env = dict(rows=rows, cols=cols, max_steps=rows - 1) if rows else {}
    lockstep(gpu, orc, variant(name, [hidden], B, T, **env), 3)


# 64-64 on Catch, the whole update in one launch: 1 to 112 samples per workgroup, ends on and off its tiles of 16, time
# steps in every remainder of the scan's batches of eight, boards of 2 to 64 cells
@pytest.mark.parametrize("rows,cols,B,T", [(2, 1, 16, 1), (8, 8, 16, 16), (10, 5, 16, 17), (9, 7, 64, 28), (5, 3, 80, 7), (4, 16, 48, 37), (3, 11, 16, 111),
                                              (6, 7, 32, 10), (10, 5, 64, 27), (7, 3, 80, 22)])
def test_small_update_in_one_launch(gpu, orc, rows, cols, B, T):
    lockstep(gpu, orc, variant("catch_small", [64, 64], B, T, rows=rows, cols=cols, max_steps=rows - 1), 5)


# returns and loss in one launch, 16 environments to a workgroup and (T = 17, 31) 8: fewer samples than threads, more than a
# thread asks for ahead, the most a workgroup holds, time steps in whole batches of the recursion and off them
@pytest.mark.parametrize("name,B,T", [("catch_4096", 16, 3), ("pendulum_8192", 32, 33), ("maze_16384", 32, 40), ("pendulum_8192", 16, 64), ("catch_4096", 48, 63), ("pendulum_8192", 48, 17), ("maze_16384", 32, 31)])
def test_returns_and_loss_in_one_launch(gpu, orc, name, B, T):
    env = dict(rows=5, cols=7, max_steps=9) if name.startswith("maze") else {}
    lockstep(gpu, orc, variant(name, [128, 64], B, T, **env), 6)


# a first layer of 32 units below a wider one, with batches that fill tiles of 16 environments
@pytest.mark.parametrize("name,hidden,B", [("pendulum_8192", [32, 64], 320), ("catch_small", [32, 512], 64)])
def test_narrow_first_layer(gpu, orc, name, hidden, B):
    lockstep(gpu, orc, variant(name, hidden, B, 6), 4)


# sample counts with odd factors: the last chunk of every split reduction is shorter than the others
@pytest.mark.parametrize("name,hidden,B,T", [("catch_4096", [512, 256], 400, 15), ("catch_4096", [256, 256], 288, 19), ("pendulum_8192", [256, 256], 352, 13),
                                             ("pendulum_8192", [64, 128], 1808, 3), ("maze_16384", [64, 64], 208, 11)])
def test_ragged_chunks(gpu, orc, name, hidden, B, T):
    env = dict(rows=5, cols=7, max_steps=9) if name.startswith("maze") else {}
    lockstep(gpu, orc, variant(name, hidden, B, T, **env), 5)


@pytest.mark.parametrize("name,hidden,B,T", [("catch_4096", [256, 256], 192, 7), ("pendulum_8192", [256, 256, 256], 64, 1), ("maze_16384", [256, 256], 192, 3),
                                             ("pendulum_8192", [512, 256, 128], 320, 3)])
def test_ragged_chunks_bf16(gpu, orc, name, hidden, B, T):
    env = dict(max_steps=9) if not name.startswith("catch") else {}
    forced_lockstep(gpu, orc, variant(name, hidden, B, T, dtype="bf16", **env), 6)


# bf16 head pass of 128 columns, half of the wavefronts on each half of a step's samples: one step of 64 samples, two, many
@pytest.mark.parametrize("name,hidden,B,T", [("catch_4096", [256, 128], 64, 1), ("pendulum_8192", [128, 128], 64, 2), ("maze_16384", [512, 128], 192, 5)])
def test_bf16_head_pass_of_128_columns(gpu, orc, name, hidden, B, T):
    env = dict(max_steps=9) if not name.startswith("catch") else {}
    forced_lockstep(gpu, orc, variant(name, hidden, B, T, dtype="bf16", **env), 4)


# backward products on split operands, few samples (their small tiles): one row tile or less, ends in the middle of a tile,
# several tiles side by side, every pairing of their widths
@pytest.mark.parametrize("name,hidden,B,T", [("catch_4096", [256, 256], 16, 1), ("pendulum_8192", [256, 256], 48, 3), ("pendulum_8192", [256, 512], 80, 5),
                                             ("catch_4096", [512, 512], 112, 5), ("pendulum_8192", [512, 256, 256], 144, 2),
                                             ("pendulum_8192", [64, 64], 16, 1), ("catch_4096", [64, 256], 80, 5), ("pendulum_8192", [64, 128, 64], 336, 3),
                                             ("catch_4096", [128, 256, 64], 48, 7), ("pendulum_8192", [128, 128], 144, 9), ("catch_4096", [512, 128], 16, 3)])
def test_split_operand_products(gpu, orc, name, hidden, B, T):
    lockstep(gpu, orc, variant(name, hidden, B, T), 8)


# acting on the matrix cores with streamed weights: tiles of 32 and 64 environments that end in the middle, layers too narrow
# for every wavefront to have a tile, first-layer weights that do not fit LDS, three layers, the replay between updates
@pytest.mark.parametrize("name,hidden,B,T", [("catch_4096", [64, 512], 8208, 2), ("pendulum_8192", [64, 128, 64], 16400, 2), ("catch_small", [128, 64, 512], 16, 6),
                                             ("pendulum_8192", [1024, 512], 48, 4), ("maze_16384", [512, 64], 80, 6), ("catch_4096", [1024, 64], 32, 4)])
def test_streaming_acting(gpu, orc, name, hidden, B, T):
    env = dict(rows=5, cols=7, max_steps=9) if name.startswith("maze") else {}
    cfg = variant(name, hidden, B, T, **env)
    lockstep(gpu, orc, cfg, 9)
    g = gpu.Anakin(cfg, seed=1); o = orc.Oracle(cfg, seed=1)
    g.set_updates_per_unroll(2, sequential=True)
    PT.sync_oracle_from_gpu(g, o)
    g.rollout(); o.rollout()
    g.learn(); o.learn_n(2, sequential=True)
    PT.assert_learn_close(g, o, TOL_F32, n_updates=2)
    g.close()


# weights-resident acting with two groups of 16 environments per workgroup where the last workgroup has one: the rows without an
# environment go through the first layer too (its matrix in LDS or, boards of many cells, in memory; the maze's always)
@pytest.mark.parametrize("name,hidden,env", [("maze_16384", [128, 128], dict(rows=5, cols=7, max_steps=9)), ("maze_16384", [256, 256], dict(rows=5, cols=7, max_steps=9)),
                                             ("catch_4096", [256, 256], dict(rows=12, cols=8, max_steps=11)), ("catch_4096", [256, 256], {}),
                                             ("catch_4096", [128, 128], dict(rows=16, cols=15, max_steps=15)),
                                             ("pendulum_8192", [128, 128], {}), ("pendulum_8192", [256, 256], {})])
def test_resident_acting_last_group_missing(gpu, orc, name, hidden, env):
    lockstep(gpu, orc, variant(name, hidden, 4112, 2, **env), 10, updates=1)


# the wall sums of bf16 mazes in the LDS of the activation buffers: first layers as wide as, wider and narrower than the others,
# one and several tiles of environments; the decoupled step's replay is cut along time, every workgroup with its own sums
@pytest.mark.parametrize("hidden,B,T", [([128, 512], 64, 5), ([512, 128], 128, 3), ([256], 64, 4), ([512, 512], 192, 6), ([128, 128], 64, 1)])
def test_bf16_maze_wall_sums(gpu, orc, hidden, B, T):
    cfg = variant("maze_16384", hidden, B, T, dtype="bf16", rows=8, cols=6, max_steps=9)
    forced_lockstep(gpu, orc, cfg, 11, updates=1)
    g = gpu.Anakin(cfg, seed=12)
    o = orc.Oracle(cfg, seed=12)
    for k in range(3):
        PT.sync_oracle_from_gpu(g, o)
        learned_on = (o.tr_reward.copy(), o.tr_done.copy())
        g.step_decoupled()
        tr = g.trajectory()
        o.step_decoupled(forced_head=tr["head"])
        PT.assert_rollout_equal(g, o, "maze", forced=True)
        if k > 0:
            PT.assert_learn_close(g, o, TOL_BF16, tr_after=tr, learned_on=learned_on, target_tol=TOL_BF16)
    g.close()


# a weight row that an environment's maze does not select is not touched, whatever it holds (fp32 acting: streamed weights,
# resident weights, the small resident form, the reference kernel)
@pytest.mark.parametrize("hidden,canonical", [([128, 64], False), ([128, 128], False), ([64, 64], False), ([64, 64], True)])
def test_infinite_wall_weight(gpu, hidden, canonical):
    cfg = variant("maze_16384", hidden, 64, 4, rows=5, cols=7, max_steps=9)
    heads = []
    for w in (0.0, -np.inf):
        g = gpu.Anakin(cfg, seed=13)
        if canonical:
            g.set_mode(gpu.MODE_CANONICAL_ACTING)
        walls = g.get_walls()
        cell = 8
        theta = g.get_params()
        theta[cell * hidden[0]:(cell + 1) * hidden[0]:3] = w
        g.set_params(theta)
        g.rollout()
        heads.append(g.trajectory()["head"])
        g.close()
    free = ((walls[:, cell >> 5] >> (cell & 31)) & 1) == 0
    assert 0 < free.sum() < 64
    assert np.array_equal(heads[0][:, free], heads[1][:, free])
    assert np.isfinite(heads[1]).all() and not np.array_equal(heads[0][:, ~free], heads[1][:, ~free])


def split_products_against_binary64(gpu, name, hidden, B, T, dtype="fp32", orc=None, edit=None, env={}):
    """The backward products on split operands and, as the measure, those on the vector ALU against binary64 on the stored
    forward pass.  A bf16 net's weights and observations are rounded before they are used; its gradients stay in binary32."""
    cfg = variant(name, hidden, B, T, dtype, **env)
    M = B * T
    regions, _ = PT.param_regions(cfg)
    grads = {}
    for mode in ("split", "valu"):
        g = gpu.Anakin(cfg, seed=14)
        assert g.plan()["bf16_matrix_path"] == 0
        if mode == "valu":
            g.set_mode(gpu.MODE_VALU_GEMM)
        theta = g.get_params() + (0.05 * np.random.default_rng(14).standard_normal(g.P)).astype(np.float32)
        if edit:
            edit(cfg, theta)
        g.set_params(theta)
        g.rollout()
        g.learn()
        tr = g.trajectory()
        grads[mode] = g.get_grads()
        g.close()
    X = PT.np_observation(cfg, tr)
    if dtype == "bf16":
        if name.startswith("pendulum"):
            # rounded from the specification's binary32 sine and cosine: from binary64 a few of 35088 samples could fall to the
            # other side of a tie, 2^-8 of a sample each
            X[:, 0], X[:, 1] = (orc.f32fun(f)(tr["state_f0"][:T].ravel()) for f in ("orc_cos", "orc_sin"))
        theta, X = PT.bf16_round_np(theta), PT.bf16_round_np(X.astype(np.float32))
    d = PT.np_head_gradient(cfg, tr["head"][:T].reshape(M, -1), tr["action"].reshape(M), tr["eps"].reshape(M), tr["adv"].reshape(M), tr["ret"].reshape(M))
    ref = PT.np_backward_from_stored(cfg, theta, X, [a.reshape(M, -1) for a in tr["act"]], d)
    # The rounding of a sample's head gradient, a few 2^-24 of it, is that of every sample with the same board and action: over
    # fewer boards than the standard one's 9 * 5 * 5 (rows left to fall, two columns) as many samples' errors add up in fewer
    # groups, larger by the root of the ratio
    boards = (env["rows"] - 1) * env["cols"] ** 2 if env else 225
    bound = PT.SPLIT_BOUND * max(1.0, (225 / boards) ** 0.5)
    for mode, got in grads.items():
        errors = {rname: PT.rel(got[sl], ref[sl]) for rname, sl in regions}
        print(f"{name} {hidden} {dtype} {B} x {T} {mode}: " + ", ".join(f"{k} {e:.1e}" for k, e in errors.items()), flush=True)
        assert max(errors.values()) <= bound, errors


# every pairing of tile widths, with the head pass and the pendulum's first layer folded in and without.  The bound notices the
# loss of any one product of terms, which the CPU suite plants (test_parity_helpers.py).
@pytest.mark.parametrize("name,hidden", [("catch_4096", [256, 256]), ("pendulum_8192", [256, 256]), ("catch_4096", [512, 256, 256]), ("pendulum_8192", [128, 128]),
                                         ("catch_4096", [128, 256]), ("catch_4096", [256, 128, 64]), ("pendulum_8192", [64, 64, 128]), ("pendulum_8192", [64, 256, 64])])
def test_split_products_keep_binary32(gpu, name, hidden):
    split_products_against_binary64(gpu, name, hidden, 416, 5)


# Every form of the kernel: each pairing of tile widths as a lower layer and as the top one (three heads, four or five folded
# in), with the first layer of the pendulum or of a small board and, in the tests of larger boards and mazes, without; (416, 5)
# takes the small tiles, (2064, 17) the large ones, several of them per workgroup, the last one not full.  That these shapes
# reach every form is checked on the CPU (test_library_host.py).
SPLIT_LAYERS = [[256, 256, 128], [256, 128, 128], [256, 64, 64], [128, 128, 64], [128, 64, 128], [64, 256, 256], [64, 64, 256, 64]]
SPLIT_PAIRS = [[256, 256], [256, 128], [256, 64], [128, 128], [128, 64], [64, 128], [64, 64]]
SPLIT_FORMS = [(name, h) for h in SPLIT_LAYERS for name in ("catch_4096", "pendulum_8192")] + [("pendulum_8192", h) for h in SPLIT_PAIRS]
SPLIT_BATCHES = [(416, 5), (2064, 17)]


@pytest.mark.parametrize("B,T", SPLIT_BATCHES)
@pytest.mark.parametrize("name,hidden", SPLIT_FORMS)
def test_every_form_of_the_split_products(gpu, name, hidden, B, T):
    split_products_against_binary64(gpu, name, hidden, B, T)


# Catch boards in the products: every pairing of tile widths as the only layer above the first (the three-layer nets above have
# the standard board), boards that fill the two tiles of 32 cells, one or none of them; the last has a cell too many for them
BOARDS = [dict(rows=8, cols=8, max_steps=7), dict(rows=16, cols=4, max_steps=15), dict(rows=7, cols=9, max_steps=6),
          dict(rows=3, cols=2, max_steps=2), dict(rows=8, cols=4, max_steps=7), dict(rows=11, cols=3, max_steps=10), dict(rows=5, cols=13, max_steps=4)]


@pytest.mark.parametrize("B,T", SPLIT_BATCHES + [(16, 1), (1040, 27)])
@pytest.mark.parametrize("hidden,env", list(zip(SPLIT_PAIRS, BOARDS)))
def test_small_boards_in_the_split_products(gpu, hidden, B, T, env):
    split_products_against_binary64(gpu, "catch_4096", hidden, B, T, env=env)


# layers under neither the heads nor a first layer that is folded in: those above a board that is too large for it
@pytest.mark.parametrize("B,T", SPLIT_BATCHES)
@pytest.mark.parametrize("hidden", SPLIT_LAYERS)
def test_layers_above_a_large_board_in_the_split_products(gpu, hidden, B, T):
    split_products_against_binary64(gpu, "catch_4096", hidden, B, T, env=BOARDS[-1])


@pytest.mark.parametrize("env", BOARDS)
@pytest.mark.parametrize("hidden", [[64, 64], [256, 256]])
def test_every_small_board_in_the_split_products(gpu, hidden, env):
    split_products_against_binary64(gpu, "catch_4096", hidden, 208, 11, env=env)


@pytest.mark.parametrize("name,hidden,B,T", [("catch_4096", [256, 128, 64], 48, 3), ("catch_4096", [256, 256], 2064, 17), ("pendulum_8192", [128, 64], 416, 5)])
def test_split_products_with_weights_at_the_lowest_value(gpu, name, hidden, B, T):
    """A weight at the type's lowest value keeps its unit from firing wherever its input is positive; the gradient that meets
    it there is 0, and so is the product."""
    split_products_against_binary64(gpu, name, hidden, B, T, edit=PT.lowest_weights)


# five heads folded in (the maze's four actions and the value): every pairing of tile widths
@pytest.mark.parametrize("B,T", SPLIT_BATCHES)
@pytest.mark.parametrize("hidden", SPLIT_PAIRS)
def test_five_heads_in_the_split_products(gpu, hidden, B, T):
    """The update's gradient against binary64 on the stored forward pass, as in test_every_form_of_the_split_products."""
    cfg = variant("maze_16384", hidden, B, T, "fp32", rows=5, cols=7, max_steps=9)
    print(f"[five heads] {hidden} {B} x {T}", flush=True)
    g = gpu.Anakin(cfg, seed=23)
    theta = g.get_params() + (0.05 * np.random.default_rng(23).standard_normal(g.P)).astype(np.float32)
    g.set_params(theta)
    g.rollout()
    g.learn()
    tr, got = g.trajectory(), g.get_grads()
    walls = np.unpackbits(g.get_walls().view(np.uint8), axis=1, bitorder="little")[:, :35].astype(bool)
    g.close()
    _, ref = PT.np_maze_backward_from_stored(cfg, theta, walls, (tr["state_s0"][:T] & 0xffff).astype(np.int64), tr["act"], tr["head"][:-1], tr["action"], tr["adv"], tr["ret"])
    errors = {rname: PT.rel(got[sl], ref[sl]) for rname, sl in PT.param_regions(cfg)[0]}
    assert max(errors.values()) <= PT.SPLIT_BOUND, errors


# bf16 nets off the bf16 matrix path in the large tiles (few samples: test_bf16_products_off_the_bf16_matrix_path)
SPLIT_LARGE_BF16 = [("catch_4096", [256, 256]), ("pendulum_8192", [256, 256]), ("catch_4096", [256, 128]), ("pendulum_8192", [128, 256, 128]),
                    ("catch_4096", [128, 128]), ("catch_4096", [128, 64, 256])]


@pytest.mark.parametrize("name,hidden", SPLIT_LARGE_BF16)
def test_bf16_products_off_the_bf16_matrix_path_in_large_tiles(gpu, orc, name, hidden):
    split_products_against_binary64(gpu, name, hidden, 2064, 17, "bf16", orc)


# the observation is rounded for the first layer's gradient as it was for the forward pass, also where the kernel is not the
# split products' (unrounded: 4e-5 here)
@pytest.mark.parametrize("hidden", [[64], [256], [32, 64], [256, 32]])
def test_bf16_pendulum_gradient_takes_the_rounded_observation(gpu, orc, hidden):
    split_products_against_binary64(gpu, "pendulum_8192", hidden, 2080, 17, "bf16", orc)


@pytest.mark.parametrize("name,hidden,B,T,env", [
    ("catch_4096", [64, 128], 16, 3, {}),                    # half blocks of inputs, one pair of output tiles per wavefront
    ("catch_4096", [128, 64], 48, 4, {}),                    # one block per wavefront
    ("catch_4096", [64, 64, 64, 64], 32, 3, {}),             # as many layers as there can be
    ("catch_4096", [512, 64], 32, 2, {}),                    # four blocks in a row; first layer of 512
    ("catch_4096", [256, 128, 64], 16, 3, dict(rows=13, cols=7, max_steps=12)),   # pairs, then a single block: five of six places
    ("catch_4096", [64, 128, 128], 32, 3, {}),               # half-block pairs before whole ones
    ("catch_4096", [64, 256], 16, 2, dict(rows=16, cols=12, max_steps=15)),       # head matrix from LDS
    ("pendulum_8192", [256, 64], 48, 4, {}),
    ("pendulum_8192", [64, 64, 128], 16, 3, {}),             # a single block, then a pair at the next even place
    ("pendulum_8192", [128, 256], 32, 2, {}),
    ("maze_16384", [128, 64], 32, 4, dict(rows=9, cols=13, max_steps=128)),       # wall words that end inside a pair of words
    ("maze_16384", [256, 64], 16, 3, {}),                    # agent plane read from memory: it does not fit LDS
    ("maze_16384", [64, 128], 16, 3, dict(rows=2, cols=2, max_steps=8, p_wall=0.0)),
    ("maze_16384", [64, 64, 64], 16, 3, dict(rows=16, cols=16, max_steps=64, p_wall=0.3)),   # more walls than one round of loads takes
])
def test_acting_with_pinned_matrices(gpu, orc, name, hidden, B, T, env):
    lockstep(gpu, orc, variant(name, hidden, B, T, "fp32", **env), seed=5, updates=1)


@pytest.mark.parametrize("name,hidden,B", [("catch_4096", [256, 128, 64], 4096), ("catch_4096", [256, 128, 64], 4112), ("maze_16384", [128, 64], 4096)])
def test_pinned_and_streamed_matrices_give_the_same_unroll(gpu, name, hidden, B):
    """The largest batch with one tile per compute unit, and one tile more (which streams)."""
    cfg = variant(name, hidden, B, 6)
    runs = []
    for mode in (0, gpu.MODE_STREAM_WEIGHTS):
        g = gpu.Anakin(cfg, seed=9)
        g.set_mode(mode)
        g.rollout(); g.rollout()
        tr = g.trajectory()
        runs.append((tr, g.get_env_state()))
        g.close()
    (a, sa), (b, sb) = runs
    for key in ("state_s0", "action", "reward", "done", "value", "head", "act"):
        for x, y in zip(a[key], b[key]):                     # steps, or layers
            np.testing.assert_array_equal(x, y, err_msg=key)
    for x, y in zip(sa, sb):
        np.testing.assert_array_equal(x, y)


# two layers of 64: a wavefront per four environments up to 4096 of them, boards with the smallest and largest first layer
@pytest.mark.parametrize("name,B,env", [
    ("catch_4096", 16, dict(rows=2, cols=1, max_steps=1)), ("catch_4096", 4096, {}), ("catch_4096", 4112, {}),
    ("catch_4096", 48, dict(rows=32, cols=19, max_steps=31)), ("catch_4096", 48, dict(rows=32, cols=20, max_steps=31)),   # W1 fits LDS, and does not
    ("pendulum_8192", 16, dict(max_steps=3)), ("pendulum_8192", 4096, dict(max_steps=5)),
    ("maze_16384", 16, dict(rows=2, cols=2, max_steps=4)), ("maze_16384", 4096, dict(rows=16, cols=16, max_steps=5)), ("maze_16384", 80, dict(rows=5, cols=13, max_steps=7)),
])
def test_two_layers_of_64_give_the_same_bits_as_streamed(gpu, name, B, env):
    cfg = variant(name, [64, 64], B, 7, "fp32", **env)
    print(f"[64-64] {name} B={B} {env}", flush=True)
    runs = []
    for mode in (0, gpu.MODE_STREAM_WEIGHTS):
        g = gpu.Anakin(cfg, seed=21)
        g.set_mode(mode)
        g.rollout(); g.rollout()
        runs.append((g.trajectory(), g.get_env_state()))
        g.close()
    (a, sa), (b, sb) = runs
    for key in ("state_s0", "reward", "done", "value", "head", "act") + (("state_f0", "state_f1", "eps", "action_f") if name.startswith("pendulum") else ("action",)):
        for x, y in zip(a[key], b[key]):
            np.testing.assert_array_equal(x, y, err_msg=key)
    for x, y in zip(sa, sb):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("name,hidden,B,env", [
    ("catch_4096", [128, 128], 64, {}),
    ("pendulum_8192", [128], 64, {}),                        # no matrix between hidden layers
    ("catch_4096", [256, 512], 128, {}),                     # two tiles of outputs per wavefront and layer
    ("pendulum_8192", [512, 256], 64, {}),                   # four blocks in a row; ReLU masks of the first layer
    ("catch_4096", [128, 512, 128], 64, {}),
    ("maze_16384", [128, 128, 128], 64, dict(rows=8, cols=8, max_steps=64)),
    ("maze_16384", [512, 128], 64, {}),                      # agent plane read from memory: it does not fit LDS
    ("catch_4096", [256, 256, 256], 8256, {}),               # 64 environments per workgroup
    ("pendulum_8192", [512, 128], 8256, {}),
    ("maze_16384", [256, 256], 8256, dict(rows=8, cols=6, max_steps=64)),
])
def test_bf16_pinned_and_streamed_matrices_give_the_same_update(gpu, name, hidden, B, env):
    """Same bits: the unroll, and through the update the packed activations and ReLU masks that it reads."""
    cfg = variant(name, hidden, B, 3, "bf16", **env)
    print(f"[bf16 pinned] {name} {hidden} B={B}", flush=True)
    runs = []
    for mode in (0, gpu.MODE_STREAM_WEIGHTS):
        g = gpu.Anakin(cfg, seed=9)
        assert g.plan()["bf16_matrix_path"] == 1
        g.set_mode(mode)
        g.step(); g.step()
        runs.append((g.trajectory(), list(g.get_env_state()) + [g.get_params(), g.get_grads()]))
        g.close()
    (a, sa), (b, sb) = runs
    pendulum = cfg["env"]["kind"] == "pendulum"
    for key in ("state_s0", "reward", "done", "value", "head", "act", "adv", "ret") + (("state_f0", "state_f1", "eps", "action_f") if pendulum else ("action",)):
        for x, y in zip(a[key], b[key]):
            np.testing.assert_array_equal(x, y, err_msg=key)
    for x, y in zip(sa, sb):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("name,hidden,B,dtype,env", [
    # one hidden layer: a row of 16 lanes per environment; 256 has its head weights in LDS
    ("catch_4096", [32], 256, "fp32", {}),
    ("catch_4096", [64], 48, "fp32", {}),
    ("catch_4096", [128], 80, "bf16", {}),
    ("catch_4096", [256], 48, "fp32", dict(rows=16, cols=12, max_steps=15)),       # first-layer rows beyond LDS: read from memory
    ("catch_4096", [256], 4176, "bf16", dict(rows=16, cols=12, max_steps=15)),
    ("pendulum_8192", [32], 96, "fp32", {}),
    ("pendulum_8192", [128], 16, "fp32", {}),
    ("pendulum_8192", [256], 80, "bf16", {}),
    ("maze_16384", [32], 32, "fp32", dict(rows=5, cols=7, max_steps=16)),
    ("maze_16384", [64], 48, "bf16", {}),
    ("maze_16384", [128], 4112, "fp32", dict(rows=9, cols=13, max_steps=64)),
    ("maze_16384", [256], 16, "bf16", dict(rows=16, cols=16, max_steps=64, p_wall=0.3)),
    # from here a lane per environment: the smallest batch of each width, last workgroups and wavefronts part filled
    ("catch_4096", [32], 24576, "fp32", dict(rows=2, cols=1, max_steps=1)),
    ("catch_4096", [64], 32784, "fp32", dict(rows=16, cols=12, max_steps=15)),
    ("pendulum_8192", [32], 24608, "fp32", {}),
    ("pendulum_8192", [64], 32768, "fp32", {}),
    # bf16 nets that the bf16 matrix path does not take, on the fp32 matrix instruction
    ("catch_4096", [128, 128], 48, "bf16", {}),
    ("catch_4096", [256, 512], 80, "bf16", dict(rows=16, cols=12, max_steps=15)),  # streamed, first-layer rows from memory
    ("pendulum_8192", [128, 64, 128], 16, "bf16", {}),
    ("pendulum_8192", [512, 512], 48, "bf16", {}),
    ("maze_16384", [256, 128], 48, "bf16", dict(rows=12, cols=14, max_steps=64)),
    ("maze_16384", [512, 256], 64, "bf16", dict(rows=9, cols=13, max_steps=64)),   # a batch of 64, but cells no multiple of 16
    ("maze_16384", [128, 256], 8208, "bf16", {}),                                  # more than one tile of 16 per compute unit
])
def test_acting_kernels_give_the_canonical_update(gpu, name, hidden, B, dtype, env):
    """The unroll, the learner's replays and what the update makes of them, bit for bit as with the vector-ALU kernel."""
    cfg = variant(name, hidden, B, 9, dtype, **env)
    print(f"[canonical {dtype}] {name} {hidden} B={B}", flush=True)
    runs = []
    for mode in (gpu.MODE_CANONICAL_ACTING, 0, gpu.MODE_STREAM_WEIGHTS):
        g = gpu.Anakin(cfg, seed=4)
        if dtype == "bf16":
            assert g.plan()["bf16_matrix_path"] == 0
        g.set_mode(mode)
        g.step()
        tr, out = g.trajectory(), [g.get_params()]
        g.step_decoupled(); g.step_decoupled(); g.step_decoupled()
        out += [g.get_params(), g.get_grads()] + list(g.get_env_state())
        runs.append((tr, out))
        g.close()
    a, sa = runs[0]
    pendulum = cfg["env"]["kind"] == "pendulum"
    for b, sb in runs[1:]:
        for key in ("state_s0", "reward", "done", "value", "head", "act") + (("state_f0", "state_f1", "eps", "action_f") if pendulum else ("action",)):
            for x, y in zip(a[key], b[key]):
                np.testing.assert_array_equal(x, y, err_msg=key)
        for x, y in zip(sa, sb):
            np.testing.assert_array_equal(x, y)


# a top layer of 256 above narrower ones: groups of four environments up to 1024 (beside a learner 256), pairs of them above one
# layer of 128 up to 2048, and the pinned kernel from there on
@pytest.mark.parametrize("name,hidden,B,dtype,env", [
    ("catch_4096", [64, 256], 1024, "fp32", dict(rows=16, cols=12, max_steps=15)), ("catch_4096", [64, 256], 1040, "fp32", dict(rows=16, cols=12, max_steps=15)),
    ("pendulum_8192", [128, 256], 256, "fp32", {}), ("pendulum_8192", [128, 256], 272, "fp32", {}), ("catch_4096", [128, 256], 2048, "fp32", {}),
    ("catch_4096", [128, 256], 2064, "fp32", {}), ("maze_16384", [64, 128, 256], 1024, "fp32", dict(rows=16, cols=16, max_steps=64)),
    ("pendulum_8192", [128, 128, 256], 1040, "fp32", {}), ("catch_4096", [64, 64, 256], 48, "fp32", {}), ("maze_16384", [128, 256], 1008, "bf16", dict(rows=9, cols=13, max_steps=64)),
])
def test_acting_under_a_top_layer_of_256(gpu, name, hidden, B, dtype, env):
    test_acting_kernels_give_the_canonical_update(gpu, name, hidden, B, dtype, env)


@pytest.mark.parametrize("name,hidden,B,T,dtype,env", [
    # boards: edges of the 32-cell tiles and of the pairs of them a kernel is made for, one to 32 column tiles, chunks
    # that end inside a maze's time steps, one unit of 16 samples in all; a board beyond the kernel's 256 cells
    ("catch_4096", [64, 64], 16, 1, "fp32", dict(rows=2, cols=1, max_steps=1)),
    ("catch_4096", [32, 64], 96, 5, "fp32", dict(rows=8, cols=4, max_steps=7)),
    ("catch_4096", [128, 64], 272, 11, "fp32", dict(rows=13, cols=5, max_steps=12)),
    ("catch_4096", [1024, 64], 32, 3, "fp32", dict(rows=16, cols=8, max_steps=15)),
    ("catch_4096", [256, 64], 80, 7, "fp32", dict(rows=43, cols=3, max_steps=42)),
    ("catch_4096", [64, 32], 160, 9, "fp32", dict(rows=16, cols=12, max_steps=15)),
    ("catch_4096", [64, 64], 96, 6, "fp32", dict(rows=64, cols=4, max_steps=63)),
    ("catch_4096", [64, 64], 32, 6, "fp32", dict(rows=64, cols=5, max_steps=63)),
    ("maze_16384", [32], 32, 1, "fp32", dict(rows=2, cols=2, max_steps=8)),
    ("maze_16384", [64, 64], 1040, 23, "fp32", dict(rows=8, cols=8, max_steps=16)),
    ("maze_16384", [128, 32], 96, 7, "fp32", dict(rows=5, cols=13, max_steps=16)),
    ("maze_16384", [512, 64], 112, 5, "fp32", dict(rows=8, cols=16, max_steps=16)),
    ("maze_16384", [64, 64], 16, 33, "fp32", dict(rows=16, cols=12, max_steps=16)),
    ("maze_16384", [256, 64], 400, 12, "fp32", dict(rows=16, cols=16, max_steps=16)),
    ("catch_4096", [128, 128], 48, 3, "bf16", dict(rows=13, cols=5, max_steps=12)),
    ("maze_16384", [128, 256], 80, 9, "bf16", dict(rows=9, cols=13, max_steps=16)),
])
def test_first_layer_of_boards(gpu, orc, name, hidden, B, T, dtype, env):
    lockstep(gpu, orc, variant(name, hidden, B, T, dtype, **env), seed=23, tol=TOL_F32 if dtype == "fp32" else TOL_BF16)


@pytest.mark.parametrize("name,hidden,B,T,env", [
    ("catch_4096", [128, 64], 272, 11, dict(rows=13, cols=5, max_steps=12)),
    ("catch_4096", [512, 64], 400, 15, dict(rows=16, cols=12, max_steps=15)),
    ("catch_4096", [64, 64], 96, 6, dict(rows=64, cols=4, max_steps=63)),
    ("maze_16384", [64, 64], 1040, 23, dict(rows=8, cols=8, max_steps=16)),
    ("maze_16384", [128, 64], 1040, 23, dict(rows=9, cols=13, max_steps=128)),
    ("maze_16384", [128, 32], 96, 7, dict(rows=5, cols=13, max_steps=16)),
    ("maze_16384", [256, 64], 400, 12, dict(rows=16, cols=16, max_steps=16)),
])
def test_first_layer_of_boards_keeps_binary32(gpu, name, hidden, B, T, env):
    """The first layer's gradient against binary64 on the stored forward pass; the bound notices the loss of the third term of
    dZ_1, which the CPU suite plants (test_parity_helpers.py)."""
    cfg = variant(name, hidden, B, T, **env)
    M = B * T
    regions, _ = PT.param_regions(cfg)
    g = gpu.Anakin(cfg, seed=19)
    theta = g.get_params() + (0.05 * np.random.default_rng(19).standard_normal(g.P)).astype(np.float32)
    g.set_params(theta)
    g.rollout()
    g.learn()
    tr, got = g.trajectory(), g.get_grads()
    if name.startswith("maze"):
        cells = env["rows"] * env["cols"]
        walls = np.unpackbits(g.get_walls().view(np.uint8), axis=1, bitorder="little")[:, :cells].astype(bool)
        _, ref = PT.np_maze_backward_from_stored(cfg, theta, walls, (tr["state_s0"][:T] & 0xffff).astype(np.int64), tr["act"], tr["head"][:-1], tr["action"], tr["adv"], tr["ret"])
    else:
        d = PT.np_head_gradient(cfg, tr["head"][:T].reshape(M, -1), tr["action"].reshape(M), tr["eps"].reshape(M), tr["adv"].reshape(M), tr["ret"].reshape(M))
        ref = PT.np_backward_from_stored(cfg, theta, PT.np_observation(cfg, tr), [a.reshape(M, -1) for a in tr["act"]], d)
    g.close()
    errors = {rname: PT.rel(got[sl], ref[sl]) for rname, sl in regions}
    print(f"{name} {hidden}: " + ", ".join(f"{k} {e:.1e}" for k, e in errors.items()), flush=True)
    assert max(errors.values()) <= PT.SPLIT_BOUND, errors


@pytest.mark.parametrize("name,hidden,rows,cols,B,T", [
    ("catch_262144", 32, 17, 6, 320, 9), ("catch_262144", 64, 10, 5, 1040, 23), ("catch_262144", 128, 8, 8, 272, 11), ("catch_262144", 256, 9, 7, 512, 16),
    ("pendulum_8192", 256, 0, 0, 1040, 23)])
def test_one_layer_keeps_binary32(gpu, name, hidden, rows, cols, B, T):
    """The same for nets of one layer, whose activations the update rebuilds (256 units store them too)."""
    cfg = variant(name, [hidden], B, T, **(dict(rows=rows, cols=cols, max_steps=rows - 1) if rows else {}))
    M, D = B * T, rows * cols
    regions, _ = PT.param_regions(cfg)
    g = gpu.Anakin(cfg, seed=19)
    theta = g.get_params() + (0.05 * np.random.default_rng(19).standard_normal(g.P)).astype(np.float32)
    g.set_params(theta)
    g.rollout()
    g.learn()
    tr, got = g.trajectory(), g.get_grads()
    g.close()
    X = PT.np_observation(cfg, tr)
    if rows:
        W1, b1 = theta[:D * hidden].reshape(D, hidden), theta[D * hidden:D * hidden + hidden]
        cells = np.nonzero(X)[1].reshape(M, 2)                   # the ball's cell, then the paddle's: the order of the sum
        h = np.maximum((b1 + W1[cells[:, 0]]) + W1[cells[:, 1]], np.float32(0))
    else:
        h = tr["act"][0].reshape(M, -1)
    d = PT.np_head_gradient(cfg, tr["head"][:T].reshape(M, -1), tr["action"].reshape(M), tr["eps"].reshape(M), tr["adv"].reshape(M), tr["ret"].reshape(M))
    ref = PT.np_backward_from_stored(cfg, theta, X, [h], d)
    errors = {rname: PT.rel(got[sl], ref[sl]) for rname, sl in regions}
    print(f"{name} {hidden}: " + ", ".join(f"{k} {e:.1e}" for k, e in errors.items()), flush=True)
    assert max(errors.values()) <= PT.SPLIT_BOUND, errors


@pytest.mark.parametrize("hidden,rows,cols,B,T", [(32, 17, 6, 64, 5), (32, 10, 5, 64, 5), (64, 10, 5, 512, 9), (64, 17, 5, 64, 5), (128, 8, 8, 64, 5), (256, 9, 7, 64, 5)])
def test_one_layer_with_an_infinite_gradient(gpu, hidden, rows, cols, B, T):
    """A unit that fires where the ball is in one cell, by 2^-119, and whose weight to the value is 2^127: a value of 256 and a
    finite loss, but dZ_1 beyond binary32 for those samples.  dW_1 is infinite in the cells that they have set and nowhere else."""
    cfg = variant("catch_262144", [hidden], B, T, rows=rows, cols=cols, max_steps=rows - 1)
    cfg["net"] = dict(cfg["net"], value_coef=0.5 * B * T)        # (the loss is a mean: a gradient of about 256 per sample)
    M, D, NH, unit, cell = B * T, rows * cols, 4, hidden - 3, cols + 1
    g = gpu.Anakin(cfg, seed=23)
    theta = g.get_params()
    W1, b1 = theta[:D * hidden].reshape(D, hidden), theta[D * hidden:(D + 1) * hidden]
    Wh = theta[(D + 1) * hidden:(D + 1) * hidden + hidden * NH].reshape(hidden, NH)
    W1[:, unit], b1[unit], Wh[unit] = 0.0, 0.0, 0.0
    W1[cell, unit], Wh[unit, NH - 1] = 2.0 ** -119, 2.0 ** 127
    g.set_params(theta)
    g.rollout()
    g.learn()
    tr, got = g.trajectory(), g.get_grads()
    loss = g.metrics()["loss"]
    g.close()
    X = PT.np_observation(cfg, tr)
    cells = np.nonzero(X)[1].reshape(M, 2)
    d = PT.np_head_gradient(cfg, tr["head"][:T].reshape(M, -1), tr["action"].reshape(M), tr["eps"].reshape(M), tr["adv"].reshape(M), tr["ret"].reshape(M))
    hit = cells[:, 0] == cell
    assert np.isfinite(loss) and 0 < hit.sum() < M and (d[hit, NH - 1] > 4.0).all(), (loss, hit.sum())
    want = np.zeros(D)
    want[np.unique(cells[hit])] = np.inf
    np.testing.assert_array_equal(got[:D * hidden].reshape(D, hidden)[:, unit], want)
    assert got[D * hidden + unit] == np.inf
    # the other columns are what they are without that unit
    h = np.maximum((b1 + W1[cells[:, 0]]) + W1[cells[:, 1]], np.float32(0))
    others = np.arange(hidden) != unit
    dz = np.where(h[:, others] > 0, d @ Wh[others].astype(np.float64).T, 0.0)
    err = PT.rel(got[:D * hidden].reshape(D, hidden)[:, others], X.T.astype(np.float64) @ dz)
    print(f"[infinite gradient] {hidden} {rows} x {cols}: {err:.1e}", flush=True)
    assert err <= PT.SPLIT_BOUND


@pytest.mark.parametrize("name,hidden,B,T,env", [
    ("catch_4096", [128, 128], 64, 1, {}),
    ("catch_4096", [256, 128], 192, 5, dict(rows=16, cols=12, max_steps=15)),
    ("catch_4096", [128, 128], 320, 7, dict(rows=16, cols=8, max_steps=15)),
    ("maze_16384", [128, 128], 64, 1, dict(rows=8, cols=8, max_steps=16)),
    ("maze_16384", [512, 128], 192, 9, dict(rows=8, cols=8, max_steps=16)),
    ("maze_16384", [128, 128], 320, 11, dict(rows=12, cols=12, max_steps=16)),
    ("maze_16384", [128, 256], 128, 23, dict(rows=16, cols=16, max_steps=16)),
])
def test_first_layer_of_boards_bf16(gpu, orc, name, hidden, B, T, env):
    forced_lockstep(gpu, orc, variant(name, hidden, B, T, "bf16", **env), seed=29)


@pytest.mark.parametrize("name,hidden,B,T,env", [
    ("catch_4096", [128, 128], 48, 7, {}),                   # heads folded in, 128-wide tiles
    ("pendulum_8192", [256, 512], 80, 5, {}),                # and the pendulum's first layer
    ("maze_16384", [256, 64], 112, 5, dict(rows=9, cols=13, max_steps=16)),     # five heads folded in
    ("maze_16384", [32, 64], 96, 3, dict(rows=9, cols=13, max_steps=16)),       # five heads above a 32-wide side: a head pass of its own
    ("maze_16384", [128, 32], 64, 5, dict(rows=9, cols=13, max_steps=16)),      # and on the vector ALU, below 64 columns
    ("catch_4096", [32, 128, 32], 96, 4, {}),                # a 32-wide side: the tiled fp32 products with rounded weights
])
def test_bf16_products_off_the_bf16_matrix_path(gpu, name, hidden, B, T, env):
    """Matrix-core products of a bf16 net's fp32 activations and rounded weights against those on the vector ALU.  Both
    differ from binary64 by at most SPLIT_BOUND per region (test_split_products_keep_binary32), so from each other by twice it."""
    cfg = variant(name, hidden, B, T, "bf16", **env)
    regions, _ = PT.param_regions(cfg)
    grads = []
    for mode in (0, gpu.MODE_VALU_GEMM):
        g = gpu.Anakin(cfg, seed=17)
        assert g.plan()["bf16_matrix_path"] == 0
        g.set_mode(mode)
        g.rollout()
        g.learn()
        grads.append(g.get_grads())
        g.close()
    errors = {rname: PT.rel(grads[0][sl], grads[1][sl]) for rname, sl in regions}
    print(f"{name} {hidden}: " + ", ".join(f"{k} {e:.1e}" for k, e in errors.items()), flush=True)
    assert max(errors.values()) <= 2 * PT.SPLIT_BOUND, errors


@pytest.mark.parametrize("hidden,B,T", [([128, 128], 64, 1), ([256, 128], 192, 7), ([512, 128], 320, 13), ([128], 1024, 5), ([128, 256], 2112, 9)])
def test_first_layer_of_the_pendulum_bf16(gpu, orc, hidden, B, T):
    # blocks of 256 samples: one that is not full, chunks that end in one, one to four blocks of columns
    forced_lockstep(gpu, orc, variant("pendulum_8192", hidden, B, T, "bf16"), seed=31)


@pytest.mark.parametrize("name,hidden,B,T", [
    # the small tiles of the split-operand products and the last batch that takes them: samples x inputs = 2^21
    ("catch_4096", [256, 256], 512, 16), ("catch_4096", [256, 256], 528, 16), ("catch_4096", [512, 512], 256, 16), ("catch_4096", [512, 512], 272, 16),
    ("pendulum_8192", [64, 256], 16, 1), ("catch_4096", [64, 64], 48, 3), ("catch_4096", [128, 64], 112, 5), ("pendulum_8192", [512, 128], 208, 6),
    ("maze_16384", [256, 64, 128], 80, 7),
])
def test_split_products_of_few_samples(gpu, orc, name, hidden, B, T):
    lockstep(gpu, orc, variant(name, hidden, B, T), seed=37)


def test_optimiser_of_few_partials(gpu, orc):
    # 2^18 parameters and more with at most 16 partials, regions of different counts in a lane's four parameters
    lockstep(gpu, orc, variant("maze_16384", [256, 256], 16, 24), seed=41)


@pytest.mark.parametrize("name,hidden,B,dtype,env", [
    # groups of four environments, weights in registers, in LDS and streamed: one group or pairs of groups per workgroup (up
    # to 1024 and above), layers cut along their inputs, one to three layers per wavefront, two passes over a layer
    ("catch_4096", [256, 256], 16, "fp32", {}),
    ("catch_4096", [256, 256], 1040, "fp32", {}),
    ("catch_4096", [64, 512], 1024, "fp32", dict(rows=16, cols=12, max_steps=15)),
    ("catch_4096", [512, 512], 48, "fp32", dict(rows=16, cols=12, max_steps=15)),  # first-layer rows from memory
    ("catch_4096", [512, 64, 512], 80, "fp32", {}),
    ("catch_4096", [64, 1024, 64], 64, "fp32", {}),
    ("catch_4096", [128, 128, 256, 256], 48, "fp32", {}),
    ("pendulum_8192", [256, 512], 2032, "fp32", {}),
    ("pendulum_8192", [512, 128], 16, "fp32", {}),
    ("maze_16384", [512, 256], 32, "fp32", dict(rows=16, cols=16, max_steps=64)),
    ("maze_16384", [256, 256], 2048, "fp32", dict(rows=9, cols=13, max_steps=64)),
    ("maze_16384", [1024, 128], 1040, "fp32", dict(rows=12, cols=14, max_steps=64)),   # pairs: the streaming kernel does not fit LDS
    ("catch_4096", [256, 256, 256], 48, "bf16", {}),
    ("pendulum_8192", [512, 512], 1040, "bf16", {}),
    ("maze_16384", [128, 512], 80, "bf16", dict(rows=9, cols=13, max_steps=64)),
])
def test_acting_in_groups_of_four(gpu, name, hidden, B, dtype, env):
    test_acting_kernels_give_the_canonical_update(gpu, name, hidden, B, dtype, env)


@pytest.mark.parametrize("name,hidden,B,T,updates,env", [
    # the learner's replay with the matrix in registers: tiles of 32 to 64 samples, a last one that is not full, more than
    # one tile per workgroup, first-layer rows beyond LDS; the smallest number of samples that takes it
    ("catch_4096", [256, 256], 272, 16, 1, {}),
    ("catch_4096", [256, 256], 1040, 21, 1, dict(rows=16, cols=12, max_steps=15)),
    ("catch_4096", [256, 256], 2064, 7, 1, {}),
    ("catch_4096", [128, 128], 4112, 8, 1, {}),
    ("pendulum_8192", [256, 256], 256, 15, 1, {}),
    ("pendulum_8192", [128, 128], 2064, 11, 1, {}),
    ("pendulum_8192", [128, 128], 2048, 8, 4, {}),
    ("catch_4096", [256, 256], 4160, 4, 2, {}),
])
def test_replay_with_the_matrix_in_registers(gpu, name, hidden, B, T, updates, env):
    """Parameters after decoupled steps or sequential updates, bit for bit as with the streaming replay."""
    cfg = variant(name, hidden, B, T, **env)
    runs = []
    for mode in (0, gpu.MODE_STREAM_WEIGHTS):
        g = gpu.Anakin(cfg, seed=6)
        g.set_mode(mode)
        if updates > 1:
            g.set_updates_per_unroll(updates, sequential=True)
            g.step(); g.step()
        else:
            g.step_decoupled(); g.step_decoupled(); g.step_decoupled()
        runs.append([g.get_params(), g.get_grads()] + list(g.get_env_state()))
        g.close()
    for x, y in zip(*runs):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("hidden,dtype,tol", [([256], "fp32", TOL_F32), ([64], "bf16", TOL_BF16)])
def test_updates_of_one_layer_in_chunks_of_many_pieces(gpu, orc, hidden, dtype, tol):
    # half of the unroll would take more first-stage workgroups of the head gradient (193 x 2) than all of it (221 x 1)
    cfg = variant("catch_4096", hidden, 3088, 16, dtype)
    g = gpu.Anakin(cfg, seed=43); o = orc.Oracle(cfg, seed=43)
    g.set_updates_per_unroll(2)
    PT.sync_oracle_from_gpu(g, o)
    g.rollout(); o.rollout()
    g.learn(); o.learn_n(2)
    PT.assert_learn_close(g, o, tol, n_updates=2)
    g.close()


def test_updates_of_one_layer_in_chunks_of_many_pieces_bf16(gpu, orc):
    # the same on the bf16 matrix path: 195 x 2 against 223 x 1
    cfg = variant("pendulum_8192", [128], 3328, 30, "bf16")
    g = gpu.Anakin(cfg, seed=47); o = orc.Oracle(cfg, seed=47)
    assert g.plan()["bf16_matrix_path"] == 1
    g.set_updates_per_unroll(2)
    PT.sync_oracle_from_gpu(g, o)
    g.rollout()
    o.rollout(forced_head=g.trajectory()["head"])
    g.learn(); o.learn_n(2)
    PT.assert_learn_close(g, o, TOL_BF16, n_updates=2)
    g.close()


def bf16_products_against_binary64(gpu, name, hidden, B, T, whole, rows=1):
    """The update's gradient against binary64 on the stored forward pass.  What differs is the rounding of dZ to bfloat16,
    once per layer from the top down to the region's own: up to 2^-9 of an entry, 2^-9 / sqrt(3) in the root mean square, and
    independent from layer to layer, so that n of them leave sqrt(n) 2^-9 / sqrt(3) of a sum whose terms have either sign; the
    bound is sqrt(3) times that.  The head matrix meets its gradient in two terms, 2^-17 of an entry.  A stage less of 238
    would cost a part in fifteen (1 / sqrt(238)) of such a sum, of 1540 a part in 39."""
    cfg = variant(name, hidden, B, T, "bf16")
    M = B * T
    print(f"[bf16 products] {name} {hidden} {B} x {T}", flush=True)
    g = gpu.Anakin(cfg, seed=29)
    plan = g.plan()
    assert plan["bf16_matrix_path"] == 1 and (not whole or all(r >= rows for r in plan["dx_rows"][1:len(hidden)])), plan
    theta = g.get_params() + (0.05 * np.random.default_rng(29).standard_normal(g.P)).astype(np.float32)
    g.set_params(theta)
    g.rollout()
    g.learn()
    tr, got = g.trajectory(), g.get_grads()
    if name.startswith("maze"):
        walls = np.unpackbits(g.get_walls().view(np.uint8), axis=1, bitorder="little").astype(bool)
        _, ref = PT.np_maze_backward_from_stored(cfg, theta, walls, (tr["state_s0"][:T] & 0xffff).astype(np.int64), tr["act"], tr["head"][:-1], tr["action"], tr["adv"], tr["ret"])
    else:
        d = PT.np_head_gradient(cfg, tr["head"][:T].reshape(M, -1), tr["action"].reshape(M), tr["eps"].reshape(M), tr["adv"].reshape(M), tr["ret"].reshape(M))
        X = PT.bf16_round_np(PT.np_observation(cfg, tr).astype(np.float32))
        ref = PT.np_backward_from_stored(cfg, PT.bf16_round_np(theta), X, [a.reshape(M, -1) for a in tr["act"]], d)
    g.close()
    for rname, sl in PT.param_regions(cfg)[0]:
        err = PT.rel(got[sl], ref[sl])
        # (a maze's first step has every agent in one cell, samples too alike for their roundings to be independent: n 2^-9 there)
        alike = T == 1 and name.startswith("maze") and not whole
        bound = 2.0 ** -15 if rname in ("Wh", "bh") else 2.0 ** -9 * (len(hidden) + 1 - int(rname[1])) ** (1.0 if alike else 0.5)
        print(f"  {rname} {err:.1e} of {bound:.1e}", flush=True)
        assert err <= bound, (rname, err, bound)


# both products of bf16 layers in whole 256-wide tiles in one launch: every width of either side, with and without the mask
# words of the layer below (a first layer of 256 has none), three, four and five heads; 2, 6, 30, 74 and 238 stages of 32
# samples, so that chunks and row ranges have one, an even and an odd number of them, up to four
@pytest.mark.parametrize("B,T", [(64, 1), (64, 3), (192, 5), (64, 37), (448, 17)])
@pytest.mark.parametrize("name,hidden", [
    ("catch_4096", [256, 256]), ("pendulum_8192", [512, 256]), ("catch_4096", [256, 512]), ("pendulum_8192", [512, 512]),
    ("catch_4096", [256, 512, 256]), ("maze_16384", [256, 256]), ("maze_16384", [512, 512, 512]),
])
def test_bf16_products_of_256_wide_tiles(gpu, name, hidden, B, T):
    bf16_products_against_binary64(gpu, name, hidden, B, T, whole=True)


# the same with eight stages and more to a row range, more than the loads run ahead and the places that they go to: every width
# as the top layer and below it, with and without the mask words of the layer below
@pytest.mark.parametrize("name,hidden,B,T", [
    ("pendulum_8192", [256, 256], 704, 70), ("maze_16384", [256, 256], 704, 70), ("catch_4096", [512, 256], 448, 53), ("pendulum_8192", [256, 512], 704, 70),
    ("catch_4096", [512, 512], 448, 53), ("catch_4096", [256, 256, 256], 704, 70), ("pendulum_8192", [512, 256, 256], 704, 70),
    ("pendulum_8192", [256, 512, 256], 704, 70), ("maze_16384", [512, 512, 512], 448, 53),
])
def test_bf16_products_of_256_wide_tiles_in_long_ranges(gpu, name, hidden, B, T):
    bf16_products_against_binary64(gpu, name, hidden, B, T, whole=True, rows=256)


# the head pass, and of two layers the pendulum's first layer, folded into the products of a top layer in 128-wide tiles: every shape of it, three, four and five heads, alone and
# above another layer; half a stage of 128 samples, one and a half, a last one that is not full, chunks of two and a half
@pytest.mark.parametrize("B,T", [(64, 1), (64, 3), (448, 17), (2112, 17)])
@pytest.mark.parametrize("name,hidden", [
    ("pendulum_8192", [128, 128]), ("catch_4096", [256, 128]), ("pendulum_8192", [512, 128]), ("catch_4096", [128, 256]),
    ("maze_16384", [128, 512]), ("maze_16384", [128, 128]), ("catch_4096", [128, 128, 128]), ("pendulum_8192", [256, 256, 128]),
    ("pendulum_8192", [256, 128]), ("pendulum_8192", [128, 256]), ("pendulum_8192", [128, 512]), ("pendulum_8192", [128, 128, 128]),
])
def test_bf16_heads_in_the_products_of_128_wide_tiles(gpu, name, hidden, B, T):
    bf16_products_against_binary64(gpu, name, hidden, B, T, whole=False)


# many samples: a chunk per compute unit, the last ones shorter
@pytest.mark.parametrize("name,hidden,B,T", [("pendulum_8192", [128, 128], 4160, 17), ("catch_4096", [256, 128], 6464, 17)])
def test_bf16_products_of_128_wide_tiles_in_many_chunks(gpu, name, hidden, B, T):
    bf16_products_against_binary64(gpu, name, hidden, B, T, whole=False)
