"""The routing of one token (csrc/routing.hpp), compiled for the host: its picks are those of a stable descending sort, and with
logits outside the contract (a NaN among them) they still lie in [0, E) and never name an expert twice, which the lists of the
projection have no room for."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_06938_amd", "csrc")

HOST = r"""
#include <math.h>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_exp2f exp2f
#include "routing.hpp"
extern "C" void route(const float *logits, long tokens, int E, int K, int32_t *idx, float *w)
{
    for (long t = 0; t < tokens; ++t)
        swimba::route_token([&](int e) { return logits[t * E + e]; }, E, K, idx + t * K, w + t * K);
}
"""


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    d = tmp_path_factory.mktemp("routing")
    (d / "route.cpp").write_text(HOST)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wno-unknown-pragmas", "-I" + CSRC, str(d / "route.cpp"),
                    "-o", str(d / "route.so")], check=True)
    lib = ctypes.CDLL(str(d / "route.so"))

    def call(g, k):
        g = np.ascontiguousarray(g, dtype=np.float32)
        idx = np.full((len(g), k), -1, dtype=np.int32)
        w = np.zeros((len(g), k), dtype=np.float32)
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        lib.route(p(g), ctypes.c_long(len(g)), g.shape[1], k, p(idx), p(w))
        return idx, w
    return call


# both sides of the register forms (8, 16 experts) and the largest
SIZES = [(1, 1), (2, 2), (4, 4), (8, 3), (8, 8), (9, 9), (16, 16), (17, 16), (32, 16), (256, 16)]


@pytest.mark.parametrize("E,k", SIZES)
def test_picks_are_a_stable_descending_sort(route, E, k):
    rng = np.random.default_rng(E)
    g = rng.integers(-2, 3, (400, E)).astype(np.float32)        # ties
    g[rng.random(g.shape) < 0.1] = -0.0
    g[rng.random(g.shape) < 0.1] = -np.inf
    g[:, 0] = np.where(np.isinf(g).all(axis=1), 0.0, g[:, 0])
    idx, w = route(g, k)
    np.testing.assert_array_equal(idx, np.argsort(-g, axis=1, kind="stable")[:, :k])
    e = np.exp(g - g.max(axis=1, keepdims=True), dtype=np.float64)
    np.testing.assert_allclose(w, np.take_along_axis(e / e.sum(axis=1, keepdims=True), idx.astype(np.int64), axis=1), rtol=1e-5)


@pytest.mark.parametrize("E,k", SIZES)
def test_no_expert_is_picked_twice_whatever_the_logits(route, E, k):
    rng = np.random.default_rng(100 + E)
    g = rng.integers(-2, 3, (4000, E)).astype(np.float32)
    for v, share in ((np.nan, 0.3), (np.inf, 0.05), (-np.inf, 0.2)):
        g[rng.random(g.shape) < share * rng.random((len(g), 1))] = v
    g[0], g[1] = np.nan, -np.inf
    if E == 8: g[2] = [3, 5] + [np.nan] * 6
    if E == 4: g[2] = [9, np.nan, 3, 5]
    idx, _ = route(g, k)
    assert idx.min() >= 0 and idx.max() < E
    assert (np.diff(np.sort(idx, axis=1), axis=1) > 0).all()
