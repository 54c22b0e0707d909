"""GPU: the count families' cluster draw on the FP32 matrix cores against the
FP64 oracle under the rules of parity_util: vocabularies on both sides of every
16-word block, K on both sides of a group of 64 clusters and of the sub-cluster
tables' room in LDS, components close together (many clusters of a point within
the Gumbel range, so that the candidate list fills) and apart."""
import numpy as np
import pytest

from oracle import dirmult, sampler
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 65, 1.0), (2, 64, 300, 1.0), (16, 40, 513, 0.05), (17, 5, 64, 1.0), (33, 65, 511, 0.1),
         (48, 64, 257, 0.05), (64, 130, 300, 0.1), (65, 20, 63, 1.0), (100, 50, 700, 0.1), (113, 3, 1, 1.0),
         (127, 90, 300, 1.0), (128, 33, 513, 0.05)]


@pytest.mark.parametrize("V,K,n,close", CASES)
def test_draw_of_dense_counts(V, K, n, close):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    seed = 7 * V + K
    g = np.random.Generator(np.random.PCG64(seed))
    th = g.dirichlet(np.full(V, 0.5), size=(K, 3)) + 1e-4
    th = close * th + (1 - close) * th.mean((0, 1), keepdims=True)
    th /= th.sum(2, keepdims=True)
    params = sampler.Params(np.log(g.dirichlet(np.ones(K))), np.log(g.dirichlet(np.ones(2), size=K)),
                            log_theta=np.log(th))
    lab = g.integers(0, K, n)
    x = np.stack([g.multinomial(g.integers(5, 150), th[k, 0]) for k in lab]).astype(np.int32).reshape(n, V)
    S = Sampler("multinomial", V, K + 2, 2.0, seed, beta=np.ones(V))
    S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
    model = sampler.Model("multinomial", 2.0, dirmult.DirPrior(np.ones(V)), seed=seed)
    lc, ls = sampler.loglik(model, x, params)
    Mc, Ms = pu.mult_scale(x, params)
    xt = torch.from_numpy(x).cuda()
    for t in (1, 2):
        z, zs = S.sample_labels(xt, t)
        zn, zsn = z.cpu().numpy(), zs.cpu().numpy()
        bad_c, bad_s, tie_c, tie_s = pu.label_mismatches(seed, t, zn, zsn, lc, ls, Mc, Ms)
        assert bad_c.size == 0 and bad_s.size == 0, (bad_c[:10], bad_s[:10])
        assert tie_c <= max(2, n // 1000) and tie_s <= max(2, n // 1000)
        S.suffstats(xt, z, zs)
        ref = pu.stats_array(sampler.suffstats(model, x, zn.astype(np.int64), zsn.astype(np.int64), K), "multinomial")
        assert np.array_equal(S.get_stats(), ref)
    S.close()


def test_large_counts_do_not_overflow_a_partial_sum():
    # one cluster of 6e6 rows with 250 000 in every entry: a workgroup may take 17 179 of them at most
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    n, V = 6_000_000, 2
    x = torch.full((n, V), 250_000, dtype=torch.int32, device="cuda")
    S = Sampler("multinomial", V, 2, 2.0, 1, beta=np.ones(V))
    S.set_state(1)
    S.suffstats(x, torch.zeros(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda"))
    st = S.get_stats()
    assert np.array_equal(st[0, 0], np.concatenate([[n], np.full(V, n * 250_000)])) and not st[0, 1].any()
    S.close()


# workgroups of 256 and of 512 threads (n up to 65 536 and beyond), most clusters of a point in range, one and two groups
# of clusters: the candidates of a tile fill the list more than once
@pytest.mark.parametrize("V,K,n", [(3, 64, 65_536), (3, 65, 65_537), (30, 200, 511), (30, 701, 70_001)])
def test_draw_with_every_cluster_in_range(V, K, n):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    seed = 3 * V + K
    g = np.random.Generator(np.random.PCG64(seed))
    th = 1.0 + 0.2 * g.random((K, 3, V))
    th /= th.sum(2, keepdims=True)
    params = sampler.Params(np.log(g.dirichlet(np.full(K, 20.0))), np.log(g.dirichlet(np.ones(2), size=K)),
                            log_theta=np.log(th))
    x = g.poisson(0.7, (n, V)).astype(np.int32)
    S = Sampler("multinomial", V, K + 2, 2.0, seed, beta=np.ones(V))
    S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
    z, zs = S.sample_labels(torch.from_numpy(x).cuda(), 3)
    zn, zsn = z.cpu().numpy(), zs.cpu().numpy()
    S.close()
    rows = np.unique(np.concatenate([np.arange(0, n, 1 + n // 1500), np.arange(max(0, n - 130), n)]))
    model = sampler.Model("multinomial", 2.0, dirmult.DirPrior(np.ones(V)), seed=seed)
    lc, ls = sampler.loglik(model, x[rows], params)
    Mc, Ms = pu.mult_scale(x[rows], params)
    bad_c, bad_s, tie_c, tie_s = pu.label_mismatches(seed, 3, zn[rows], zsn[rows], lc, ls, Mc, Ms, points=rows)
    assert bad_c.size == 0 and bad_s.size == 0, (bad_c[:10], bad_s[:10])
    assert tie_c <= 4 and tie_s <= 4
    assert np.unique(zn).size > K // 2
