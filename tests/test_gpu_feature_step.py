"""The feature dynamics' step kernel at the sizes where its tiling can go
wrong: one env, one less and one more than a 16- or 32-env tile, and both
sides of the batch sizes (16, 32, 48 and 64 envs per CU) where the tile or the
number of wavefronts changes, for every state width; given and kernel-sampled actions, 2 to 8 seats.  States, returns
and rewards are compared bit for bit with the oracle's sequential fused chain
(gpu_helpers.check_parity), also where products, sums and states are subnormal."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import check_parity, run_gpu, say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _edges(n, rng):
    """Envs around every tile boundary near both ends, and a few others."""
    at = {0, 15, 16, 31, 32, n // 2, n - 33, n - 32, n - 17, n - 16, n - 1}
    at |= set(rng.integers(0, n, size=6).tolist())
    return np.array(sorted(e for e in at if 0 <= e < n))


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("d", [64, 128, 256, 512])
def test_step_tile_edges(d, sampled):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for k, n in enumerate([1, 15, 16, 17, 33, 16 * cus, 16 * cus + 1, 32 * cus + 31,
                           48 * cus + 1, 48 * cus, 64 * cus, 64 * cus + 1]):
        seats = [2, 8, 3, 5][k % 4]
        # fp32 policies leave the sampling to the step kernel
        wl = W.team_variant(seats, d=d, P=3, n_envs=n, horizon=2)
        if sampled:
            wl = W.with_policies(wl, W.MLP_F32, [d, 32, 32, 18])
        say(f"[step] d={d} n={n} seats={seats} sampled={sampled}")
        sel = np.arange(n) if n < 64 else _edges(n, np.random.default_rng(n))
        check_parity(wl, run_gpu(wl, snaps=[0, 1]), sel)


@pytest.mark.parametrize("n", [33, 4200])
@pytest.mark.parametrize("d", [64, 256])
def test_step_subnormal_sums(d, n):
    """Dynamics scaled so that the chains' products and sums, the embeddings
    and from the second step on the states are subnormal."""
    wl = W.team_variant(2, d=d, P=3, n_envs=n, horizon=3)
    wl.W = (wl.W * np.float32(2.0 ** -128)).astype(np.float32)
    wl.emb = (wl.emb * np.float32(2.0 ** -130)).astype(np.float32)
    wl.u = (wl.u * np.float32(2.0 ** 20)).astype(np.float32)
    g = run_gpu(wl, snaps=[0, 1, 2])
    s1 = np.abs(g["states"][1])
    assert ((s1 > 0) & (s1 < np.finfo(np.float32).tiny)).mean() > 0.9
    check_parity(wl, g, np.arange(n) if n < 64 else _edges(n, np.random.default_rng(1)))


@pytest.mark.parametrize("d,n", [(256, 2 ** 24), (512, 2 ** 23)])
def test_observation_rows_past_2_32_elements(d, n):
    """The last envs of a batch whose states hold more than 2^32 values play as
    they do in a small batch at their offset (64-row and persistent forward)."""
    from paper_2106_07551_amd import workload_io as IO
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB")
    extra = 1500
    wl = W.team_variant(2, d=d, P=2, n_envs=extra, horizon=2)
    wl = W.with_policies(wl, W.MLP_BF16, [d, 64, 64, 18])
    env, pop = IO.make_env(wl), IO.make_population(wl)
    g = torch.Generator(device="cuda").manual_seed(d)
    pairs = torch.randint(0, 2, (n + extra, 2), generator=g, device="cuda", dtype=torch.int32)
    ref = torch.empty((2, extra), device="cuda")
    pop.rollout(env, extra, pairs[n:].contiguous(), wl.seed, 2, env_offset=n, returns=ref)
    ret = torch.empty((2, n + extra), device="cuda")
    say(f"[step] d={d} n={n + extra}")
    pop.rollout(env, n + extra, pairs, wl.seed, 2, returns=ret)
    torch.cuda.synchronize()
    pop.close()
    assert torch.unique(ref).numel() > extra
    assert torch.equal(ret[:, n:], ref)
