"""GPU: the FP32 cluster draw on the FP32 matrix cores, the log-likelihoods and
the vector-ALU draw of the dimensions around it, against the FP64 oracle under
the rules of parity_util.  Dimensions sit on both sides of every 16-row block
and of the switch between the two draws; row counts on both sides of a wave and
a workgroup step; K on both sides of one and several record groups in LDS."""
import numpy as np
import pytest

from oracle import niw, sampler
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

CASES = [  # d, K, n, spread: 4 well apart; 0.2 most clusters within the Gumbel range of every point
    (6, 5, 300, 4.0), (11, 30, 257, 0.2), (17, 9, 255, 4.0), (26, 40, 300, 0.2), (27, 40, 257, 0.2),
    (31, 3, 65, 4.0), (32, 33, 513, 0.2), (33, 1, 1, 4.0), (47, 12, 64, 0.2), (48, 13, 63, 4.0), (49, 20, 300, 0.2),
    (63, 9, 255, 4.0), (65, 10, 256, 0.2), (80, 6, 257, 4.0), (81, 6, 200, 0.2), (96, 5, 300, 4.0), (97, 4, 300, 0.2),
    (112, 3, 300, 4.0), (113, 2, 300, 0.2), (127, 5, 700, 0.2), (128, 7, 513, 0.2)]


@pytest.mark.parametrize("d,K,n,spread", CASES)
def test_fp32_draw_and_loglik(d, K, n, spread):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    seed = 50 + 3 * d + K
    params = pu.random_gauss_params(K, d, seed, spread=spread)
    x = pu.gauss_points(params, n, seed + 1)
    S = Sampler("gaussian", d, K + 2, 2.0, seed, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d))
    S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
    xt = torch.from_numpy(x).cuda()
    model = sampler.Model("gaussian", 2.0, niw.NIWPrior(1.0, np.zeros(d), d + 3, np.eye(d)), seed=seed)
    lc, ls = sampler.loglik(model, x.astype(np.float64), params)
    Mc, Ms = pu.gauss_scale(x, params)
    ll = S.loglik(xt).cpu().numpy().astype(np.float64)
    assert pu.check_loglik(ll, lc, ls, Mc, Ms) <= 1e-5
    for t in (1, 2):
        z, zs = S.sample_labels(xt, t)
        bad_c, bad_s, tie_c, tie_s = pu.label_mismatches(seed, t, z.cpu().numpy(), zs.cpu().numpy(), lc, ls, Mc, Ms)
        assert bad_c.size == 0 and bad_s.size == 0, (bad_c[:10], bad_s[:10])
        assert tie_c <= max(2, n // 1000) and tie_s <= max(2, n // 1000)
    S.close()


# one infinite coordinate, at the first, a middle and the last column of a 16-row block, the last block ragged or not:
# every whitened coordinate from it on is infinite and no other is touched, so every log-likelihood is -inf; a NaN
# stays one, and the rows beside have the bits that they have alone
@pytest.mark.parametrize("d", [3, 16, 17, 32, 45, 128])
def test_loglik_of_rows_with_an_infinity(d):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    K, n = 5, 300
    params = pu.random_gauss_params(K, d, 60 + d, spread=2.0)
    x = pu.gauss_points(params, n, 61 + d)
    S = Sampler("gaussian", d, K + 2, 2.0, 3, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d))
    S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
    ref = S.loglik(torch.from_numpy(x).cuda()).cpu().numpy()
    cols = sorted({c for c in (0, 1, 7, 15, 16, 23, 31, 32, 40, 44, 63, 64, 100, 127, d - 1) if c < d})
    inf_rows = np.arange(len(cols)) * 5 + 2
    y = x.copy()
    for i, c in zip(inf_rows, cols):
        y[i, c] = np.inf if c % 2 else -np.inf
    nan_rows = np.array([0, n - 1])
    y[nan_rows, d // 2] = np.nan
    out = S.loglik(torch.from_numpy(y).cuda()).cpu().numpy()
    S.close()
    assert np.all(out[inf_rows] == -np.inf), np.argwhere(out[inf_rows] != -np.inf)[:5]
    assert np.all(np.isnan(out[nan_rows]))
    same = np.setdiff1d(np.arange(n), np.concatenate([inf_rows, nan_rows]))
    assert np.all(np.isfinite(ref)) and np.array_equal(out[same], ref[same])


# the statistics over sorted rows by themselves: on both sides of the switch from one row per lane to padded
# tiles (32 | 33), of the padded widths (64 | 65), at the smallest and largest dimension of each, with empty
# sub-clusters; d < 5 with more clusters than the per-lane sums hold
@pytest.mark.parametrize("d,K,n", [(1, 900, 3000), (3, 300, 2001), (5, 4, 1), (7, 3, 65), (15, 2, 700), (17, 9, 1300),
                                   (31, 5, 4097), (33, 3, 513), (63, 2, 257), (65, 4, 130), (99, 2, 129), (127, 3, 700)])
def test_stats_of_any_dimension(d, K, n):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    from tests.test_gpu_parity import _check_stats
    g = np.random.Generator(np.random.PCG64(d * 31 + K))
    x = (g.standard_normal((n, d)) * 3 + 1).astype(np.float32)
    z = g.integers(0, K, n).astype(np.int32)
    zs = g.integers(0, 2, n).astype(np.uint8)
    zs[z == 0] = 1
    S = Sampler("gaussian", d, K, 2.0, 5, m=np.zeros(d), psi=np.eye(d))
    S.set_state(K)
    S.suffstats(torch.from_numpy(x).cuda(), torch.from_numpy(z).cuda(), torch.from_numpy(zs).cuda())
    _check_stats(S.get_stats(), x, z, zs, K, d)
    S.close()


# the draw over rows sorted by a guessed cluster (48 <= d, several clusters, n K >= 250 000), with ragged last
# steps, a word boundary of the clusters' bit sets (K = 33) and several groups of heads (K = 130); clusters apart
# (most ruled out by their first rows) and overlapping (none)
@pytest.mark.parametrize("d,K,n,spread", [(48, 64, 3907, 4.0), (49, 130, 2003, 0.2), (64, 20, 12545, 0.2),
                                          (100, 12, 20999, 4.0), (113, 33, 7600, 0.5), (128, 9, 27801, 4.0)])
def test_fp32_draw_by_guess(d, K, n, spread):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    seed = 70 + d + K
    params = pu.random_gauss_params(K, d, seed, spread=spread)
    x = pu.gauss_points(params, n, seed + 1)
    x[5] *= 100.0  # far from every cluster
    S = Sampler("gaussian", d, K + 2, 2.0, seed, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d))
    S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
    xt = torch.from_numpy(x).cuda()
    z, zs = S.sample_labels(xt, 3)
    st = S.get_stats()
    zn, zsn = z.cpu().numpy(), zs.cpu().numpy()
    assert st[..., 0].sum() == n and np.array_equal(st[..., 0], np.bincount(2 * zn + zsn, minlength=2 * K).reshape(K, 2))
    rows = np.unique(np.concatenate([np.arange(0, n, 7), np.arange(n - 70, n), [5]]))
    model = sampler.Model("gaussian", 2.0, niw.NIWPrior(1.0, np.zeros(d), d + 3, np.eye(d)), seed=seed)
    xs = x[rows]
    lc, ls = sampler.loglik(model, xs.astype(np.float64), params)
    Mc, Ms = pu.gauss_scale(xs, params)
    bad_c, bad_s, tie_c, tie_s = pu.label_mismatches(seed, 3, zn[rows], zsn[rows], lc, ls, Mc, Ms, points=rows)
    assert bad_c.size == 0 and bad_s.size == 0, (bad_c[:10], bad_s[:10])
    assert tie_c <= max(2, n // 1000) and tie_s <= max(2, n // 1000)
    S.close()


# rows with a NaN, an infinity or values whose squares overflow, the first row among them: every row is drawn, and
# as the FP32 context draws it
# (d = 32: one and two buffers of clusters, K = 16 | 17, ragged waves and steps)
@pytest.mark.parametrize("d,K,n", [(64, 4, 700), (64, 20, 12545), (128, 5, 513), (128, 9, 27801), (32, 1, 1), (32, 16, 513),
                                   (32, 17, 1025), (32, 25, 4223)])
def test_bf16_draw_of_rows_without_a_score(d, K, n):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    params = pu.random_gauss_params(K, d, 7 + d, spread=3.0)
    x = pu.gauss_points(params, n, 8 + d)
    x[::97, 3] = np.nan
    x[5::101, 7] = np.inf
    x[7::103] *= 1e30
    xt = torch.from_numpy(x).cuda()
    z = {}
    for prec in ("fp32", "bf16"):
        S = Sampler("gaussian", d, K + 2, 2.0, 11, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d), precision=prec)
        S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
        z[prec] = S.sample_labels(xt, 1)[0].cpu().numpy()
        S.close()
    assert z["bf16"].min() >= 0 and z["bf16"].max() < K
    assert np.array_equal(z["fp32"], z["bf16"])


# the BF16 draw by a guess (d = 64, 128, n >= 1e6, K >= 64, 32): all points by it, some left open by the guess's
# bound, and none (the sample decides against it); ragged last steps, rows without a score
@pytest.mark.parametrize("d,K,n,spread", [(64, 64, 1_000_000, 3.0), (64, 131, 1_000_003, 1.2), (64, 64, 1_000_100, 0.2),
                                          (128, 32, 1_000_001, 3.0), (128, 33, 1_000_447, 1.6)])
def test_bf16_draw_by_guess(d, K, n, spread):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    params = pu.random_gauss_params(K, d, 9 + d, spread=spread)
    g = torch.Generator(device="cuda").manual_seed(d + K)
    x = torch.randn((n, d), device="cuda", generator=g)
    mu = torch.from_numpy(params.mu[:, 0]).float().cuda()
    x += mu[torch.randint(0, K, (n,), device="cuda", generator=g)]
    x[5::4001, 3] = float("nan")
    x[::5003, 7] = float("inf")
    z = {}
    for prec in ("fp32", "bf16"):
        S = Sampler("gaussian", d, K + 2, 2.0, 11, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d), precision=prec)
        S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
        z[prec], zs = S.sample_labels(x, 1)
        got = S.get_stats()[:, :, 0]
        S.close()
    assert torch.equal(z["fp32"], z["bf16"])
    count = torch.bincount(z["bf16"].long() * 2 + zs.long(), minlength=2 * K).cpu().numpy()
    assert np.array_equal(got, count.reshape(K, 2))


# the buffers of the draw by a guess belong to the contexts that take it: with K too small for it a label step
# holds the permutation and the sorted labels, in BF16 beside the candidate lists and the sub-labels' lists
@pytest.mark.parametrize("d,prec,per_point", [(48, "fp32", 8), (64, "bf16", 8 + 32 + 9)])
def test_scratch_of_a_label_step_with_few_clusters(d, prec, per_point):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    K, sizes = 2, (1_000_000, 9_000_000)
    params = pu.random_gauss_params(K, d, 3)
    taken = []
    for n in sizes:
        x = torch.zeros((n, d), device="cuda")
        z = torch.empty(n, dtype=torch.int32, device="cuda")
        zs = torch.empty(n, dtype=torch.uint8, device="cuda")
        S = Sampler("gaussian", d, K, 2.0, 11, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d), precision=prec)
        S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        S.sample_labels(x, 1, z, zs)
        torch.cuda.synchronize()
        taken.append(free - torch.cuda.mem_get_info()[0])
        S.close()
        del x, z, zs
    # (allocations are rounded up to 2 MB)
    assert taken[1] - taken[0] <= per_point * (sizes[1] - sizes[0]) + (8 << 20), taken


# the draw by a guess against the draw that forms every score: as many of the first rows as stay below the guess's
# range (n K < 250 000, BF16 n < 1e6) have the labels that they have among all; covariances of condition 10 and 1e6,
# data about one centre, far from it, and in two groups
@pytest.mark.parametrize("d,K,prec", [(48, 12, "fp32"), (64, 40, "fp32"), (100, 130, "fp32"), (128, 9, "fp32"),
                                      (64, 70, "bf16"), (128, 34, "bf16")])
@pytest.mark.parametrize("cond,shift", [(10.0, 0.0), (1e6, 0.0), (1e6, 500.0), (10.0, 40.0)])
def test_draw_by_guess_equals_the_full_draw(d, K, prec, cond, shift):
    import torch

    from paper_2204_08988_amd.sampler import Sampler
    n = 1_000_100 if prec == "bf16" else 20_000 + 400_000 // K
    few = 249_999 // K if prec == "fp32" else 60_000
    params = pu.random_gauss_params(K, d, 21 + d + K, spread=1.5, cond=cond)
    params.mu[: K // 2] += shift
    params.mu[K // 2:] += -shift if shift == 40.0 else shift
    g = torch.Generator(device="cuda").manual_seed(d + K)
    x = torch.randn((n, d), device="cuda", generator=g)
    lab = torch.randint(0, K, (n,), device="cuda", generator=g)
    L = torch.from_numpy(np.linalg.cholesky(params.sigma[:, 0])).float().cuda()
    for k in range(K):
        x[lab == k] = x[lab == k] @ L[k].T.contiguous()
    x += torch.from_numpy(params.mu[:, 0]).float().cuda()[lab]
    S = Sampler("gaussian", d, K + 2, 2.0, 11, kappa=1.0, nu=d + 3.0, m=np.zeros(d), psi=np.eye(d), precision=prec)
    S.set_params(params.log_pi, params.log_pisub, pu.comp_array(params))
    z, zs = S.sample_labels(x, 3)
    zf, zsf = S.sample_labels(x[:few].contiguous(), 3)
    S.close()
    assert torch.equal(z[:few], zf) and torch.equal(zs[:few], zsf)
    assert torch.unique(zf).numel() > K // 2
