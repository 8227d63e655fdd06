"""GPU parity at the edges of the kernels' dispatch rules: shapes where a tile, a chunk or a row group ends in the
middle, each in lockstep with the CPU oracle (unroll bit for bit in fp32, update per parameter region)."""
import pytest

from paper_2104_06272_amd import workloads as W
import parity as PT

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4


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


# one hidden layer of 64 or 128 units with many samples: every chunk's head gradient is summed
@pytest.mark.parametrize("name,hidden,B,T", [("catch_262144", 64, 512, 8), ("catch_262144", 128, 256, 16), ("pendulum_8192", 64, 1024, 4)])
def test_one_layer_many_samples(gpu, orc, name, hidden, B, T):
    lockstep(gpu, orc, variant(name, [hidden], B, T), 3)


# a first layer of 32 units below a wider one, with batches that fill tiles of 16 environments
@pytest.mark.parametrize("name,hidden,B", [("pendulum_8192", [32, 64], 320), ("catch_small", [32, 512], 64)])
def test_narrow_first_layer(gpu, orc, name, hidden, B):
    lockstep(gpu, orc, variant(name, hidden, B, 6), 4)
