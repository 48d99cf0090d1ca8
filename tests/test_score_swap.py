"""Which keys the single-sweep scoring kernel moves into its reference tiles
(csrc/kara_score_swap.h), checked on the host: the kernel's bound search and
pairing, written out here over the header's own rank and sizes, must never
list more keys than its arrays hold, whatever the keys' norms are -- among
them NaN of either sign, as pool memory that was never written can give."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_01237_amd", "csrc")

MODEL = r"""
#include "kara_score_swap.h"
using namespace kara;
// norm bits of 64 * nt keys, the first n of them real; the listed keys and
// positions (room for any number), their counts in cnt[0], cnt[1]
extern "C" uint32_t pair_keys(const uint32_t* norm, int nt, int n, int32_t* key, int32_t* pos, int32_t* cnt) {
  const int keys = 64 * nt;
  uint32_t bound = 0;
  for (int bit = kSwapRankBits - 1; bit >= 0; --bit) {
    const uint32_t cand = bound | (1u << bit);
    int all = 0;
    for (int j = 0; j < keys; ++j) all += swap_rank(norm[j]) >= cand;
    if (all >= kSwapMax) bound = cand;
  }
  cnt[0] = cnt[1] = 0;
  for (int j = 0; j < keys; ++j)
    if (swap_rank(norm[j]) > bound && j % (nt * 16) >= 16) key[cnt[0]++] = j;
  for (int i = 0; i < kSwapMax; ++i) {
    const int p = (i >> 4) * nt * 16 + (i & 15);
    if (p < n && swap_rank(norm[p]) <= bound) pos[cnt[1]++] = p;
  }
  return bound;
}
extern "C" int swap_max() { return kSwapMax; }
extern "C" int rank_bits() { return kSwapRankBits; }
extern "C" uint32_t rank(uint32_t b) { return swap_rank(b); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("swap")
    src, so = d / "model.cpp", d / "model.so"
    src.write_text(MODEL)
    subprocess.run([shutil.which("g++") or "c++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(so)],
                   check=True)
    return ctypes.CDLL(str(so))


def _norms(kind, keys, n, rng):
    x = (rng.standard_normal((keys, 128)).astype(np.float32) ** 2).sum(1).astype(np.float32)
    b = x.view(np.uint32).copy()
    if kind == "heavy":
        b = np.where(rng.random(keys) < 0.02, (x * 16).astype(np.float32), x).astype(np.float32).view(np.uint32)
    elif kind == "equal":
        b[:] = np.float32(128).view(np.uint32)
    elif kind == "zero":
        b[:] = 0
    elif kind == "nan":
        b[:] = 0x7FC00000
    elif kind == "nan_sign":                    # every key a NaN with its sign set
        b[:] = 0xFFC00000
    elif kind == "nan_all_ones":                # memory filled with 0xFF
        b[:] = 0xFFFFFFFF
    elif kind == "some_nan_sign":               # more of them than may change places
        b[rng.permutation(keys)[:100]] = 0xFFC00000
    elif kind == "mixed":
        b = rng.choice(np.array([0, 0x42FE0000, 0x7F800000, 0x7FC00000, 0xFF800001, 0xFFC00000, 0xFFFFFFFF], np.uint32), keys)
    b[n:] = 0
    return np.ascontiguousarray(b)


def test_ranks_are_below_the_search_range(lib):
    lib.rank.restype = ctypes.c_uint32
    top = 1 << lib.rank_bits()
    assert all(lib.rank(ctypes.c_uint32(hi << 16 | lo)) < top for hi in range(0, 65536, 5) for lo in (0, 0xFFFF))
    assert all(lib.rank(ctypes.c_uint32(b)) < top for b in (0xFFFFFFFF, 0xFFC00000, 0xFF800001, 0x7FFFFFFF))


@pytest.mark.parametrize("kind", ["random", "heavy", "equal", "zero", "nan", "nan_sign", "nan_all_ones", "some_nan_sign", "mixed"])
@pytest.mark.parametrize("nt,n", [(12, 513), (12, 768), (16, 1000), (28, 1792), (32, 2048)])
def test_no_more_keys_change_places_than_fit(lib, kind, nt, n):
    rng = np.random.default_rng(nt * 10000 + n)
    keys = 64 * nt
    norm = _norms(kind, keys, n, rng)
    key, pos, cnt = np.full(keys, -1, np.int32), np.full(64, -1, np.int32), np.zeros(2, np.int32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    lib.pair_keys(p(norm), nt, n, p(key), p(pos), p(cnt))
    assert cnt[0] < lib.swap_max() and cnt[1] <= lib.swap_max()
    k, s = key[:cnt[0]], pos[:cnt[1]]
    # real keys from outside the reference tiles change places with real ones
    # inside them, each at most once
    assert (k < n).all() and (s < n).all()
    assert (k % (nt * 16) >= 16).all() and (s % (nt * 16) < 16).all()
    assert len(set(k)) == len(k) and len(set(s)) == len(s)
    if kind == "heavy":
        assert cnt[0] > 0
