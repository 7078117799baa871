"""The kernels' sampler (cce_sampler.hpp) compiled for the host: its ids against the reference sampler, and what one draw costs."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import sampler as S
from workloads import alias_table, popularity_weights

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = """
#pragma once
#include <stdint.h>
#define __device__
#define __forceinline__ inline
struct uint2 { unsigned x, y; };
static long products = 0;   // 64-bit products: twenty a generator call, one a column
static inline uint32_t __umulhi(uint32_t a, uint32_t b) { ++products; return (uint32_t)(((uint64_t)a * b) >> 32); }
"""
MAIN = """
#include <hip/hip_runtime.h>
#include "cce_sampler.hpp"
extern "C" long draw_one_by_one(int kind, uint64_t seed, uint32_t stream, uint32_t V, const uint32_t *thresh, const int32_t *alias,
                                const uint64_t *packed, int N, int K, int32_t *one, int32_t *four)
{
    cce::Sampler s{(uint32_t)kind, (uint32_t)seed, (uint32_t)(seed >> 32), stream, V, thresh, alias, reinterpret_cast<const uint2 *>(packed)};
    products = 0;
    for (int i = 0; i < N; ++i)
        for (int k = 0; k < K; ++k) one[(long)i * K + k] = cce::sample1(s, (uint64_t)i, (uint32_t)k + 1);
    const long cost = products;
    for (int i = 0; i < N; ++i)
        for (int q = 0; q <= K / 4; ++q) {
            cce::Draws d[1];
            int32_t id[4], looked_up[1][4];
            cce::sample4(s, (uint64_t)i, (uint32_t)q, id);
            cce::draw4(s, (uint64_t)i, (uint32_t)q, d[0]);
            cce::resolve4(s, d, looked_up);
            for (int t = 0; t < 4; ++t)
                if (4 * q + t >= 1 && 4 * q + t <= K) four[(long)i * K + 4 * q + t - 1] = id[t] == looked_up[0][t] ? id[t] : -1;
        }
    return cost;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_draws_on_the_host(tmp_path):
    """Draws one by one and in groups of four, from the caller's table and from its copy with both words side by side, give the
    reference ids; a draw on its own costs one generator call and one column of the table."""
    import ctypes

    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "draws.cpp").write_text(MAIN)
    lib = str(tmp_path / "draws.so")
    res = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-I", str(tmp_path), "-I",
                          os.path.join(ROOT, "paper_2509_09682_amd", "csrc"), str(tmp_path / "draws.cpp"), "-o", lib],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    f = ctypes.CDLL(lib).draw_one_by_one
    f.restype = ctypes.c_long
    N, K, V, seed, stream = 37, 30, 1009, 0x0123_4567_89AB_CDEF, 7
    thresh, alias = alias_table(popularity_weights(np.random.default_rng(3).permutation(V).astype(np.int32), 1.2, 0.75))
    packed = (thresh.astype(np.uint32).astype(np.uint64) | (alias.astype(np.uint64) << np.uint64(32)))
    ptr = lambda x: None if x is None else x.ctypes.data_as(ctypes.c_void_p)
    for kind, table in ((S.UNIFORM, (None, None, None)), (S.ALIAS, (thresh, alias, None)), (S.ALIAS, (thresh, alias, packed))):
        one, four = np.empty((N, K), np.int32), np.empty((N, K), np.int32)
        cost = f(kind, ctypes.c_uint64(seed), stream, V, ptr(table[0]), ptr(table[1]), ptr(table[2]), N, K, ptr(one), ptr(four))
        want = S.sample_negatives(kind, seed, stream, N, K, V, per_position=True, thresh=table[0], alias=table[1])
        assert np.array_equal(one, want) and np.array_equal(four, want)
        assert cost == 21 * N * K, (kind, cost / (N * K))
