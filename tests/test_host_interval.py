"""The lower bound of a bf16x3 score against the FP32 score it stands for, on the
CPU: both forms rounded as the kernels round them (BF16 parts to nearest even, FP32
sums one after the other, in both directions of the sum for the matrix form), the
bound from the library's own header.  (A fixed share of the squared norm, q / 4096 +
0.05, misses by 0.2 and 0.6 at condition 1e10.)"""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
F = np.float32


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    exe = str(tmp_path_factory.mktemp("interval") / "interval_driver")
    subprocess.run([gxx, "-O2", "-ffp-contract=off", "-std=c++17", "-o", exe,
                    os.path.join(HERE, "host", "interval_driver.cpp")], check=True)
    return exe


def _bf16(x):
    u = np.ascontiguousarray(x, F).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & np.uint32(0xFFFF0000)).astype(np.uint32).view(F)


def _sum32(terms, axis_reversed):
    """FP32 sum over the last axis, one term after the other (products exact in float64)."""
    acc = np.zeros(terms.shape[:-1], F)
    order = range(terms.shape[-1])
    for i in (reversed(order) if axis_reversed else order):
        acc = (acc.astype(np.float64) + terms[..., i]).astype(F)
    return acc


def _scores(W, v, c, axis_reversed):
    """(FP32 score, bf16x3 norm) of the rows v under the lower-triangular W."""
    q32 = np.zeros(v.shape[0], F)
    q3 = np.zeros(v.shape[0], F)
    wh, vh = _bf16(W), _bf16(v)
    wl, vl = _bf16(W - wh), _bf16(v - vh)
    for r in range(W.shape[0]):
        k = r + 1
        y = _sum32(W[r, :k].astype(np.float64) * v[:, :k], False)
        q32 = (q32.astype(np.float64) + y.astype(np.float64) ** 2).astype(F)
        a, b, e = (W64[r, :k].astype(np.float64) * u[:, :k] for W64, u in ((wh, vh), (wh, vl), (wl, vh)))
        y3 = _sum32(np.concatenate([a, b, e], axis=1), axis_reversed)
        q3 = (q3.astype(np.float64) + y3.astype(np.float64) ** 2).astype(F)
    return (c - 0.5 * q32.astype(np.float64)).astype(F), np.sqrt(q3)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cond", [1e2, 1e6, 1e8, 1e10])
def test_x3_lower_bound(driver, d, cond):
    g = np.random.Generator(np.random.PCG64(int(np.log10(cond)) + d))
    n = 200
    for kind in range(3):
        q, _ = np.linalg.qr(g.standard_normal((d, d)))
        lam = np.exp(g.uniform(-0.5, 0.5, d) * np.log(cond))
        lam[0], lam[1] = cond ** 0.5, cond ** -0.5
        sigma = (q * lam) @ q.T
        L = np.linalg.cholesky(sigma + 1e-16 * np.eye(d))
        W = np.linalg.inv(L).astype(F)
        # rows of the cluster, rows far off, and rows along its widest axis
        e = g.standard_normal((n, d))
        v = (e @ L.T if kind == 0 else 30.0 * e if kind == 1 else np.outer(e[:, 0], q[:, 0]) * 3 * lam[0] ** 0.5).astype(F)
        c = F(np.log(np.abs(np.diag(W).astype(np.float64))).sum())
        wf = np.sqrt((W.astype(np.float64) ** 2).sum())
        for rev in (False, True):
            l32, s = _scores(W, v, c, rev)
            wv = (wf * np.sqrt((v.astype(np.float64) ** 2).sum(axis=1)) * 1.00001).astype(F)
            text = "\n".join(f"{c:.9g} {a:.9g} {b:.9g}" for a, b in zip(s, wv)) + "\n"
            out = subprocess.run([driver], input=text, capture_output=True, text=True, check=True).stdout.split()
            low = np.array(out, dtype=np.float64)
            assert low.shape == (n,)
            assert np.all(low <= l32), (kind, rev, np.max(low - l32))
