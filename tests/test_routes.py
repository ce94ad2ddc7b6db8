"""The size rules that choose a kernel variant (csrc/kf_route.h), compiled for
the host: each shape below goes to the kernel that measured faster there, and the
shapes of the GPU tests reach the kernels that they are written for."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "kf_route.h"
extern "C" int training(int dh, long long BH, int two, long long N, long long k, int *prow, int *blocks) {
  const long long nq = two ? 2 * N * k : N + N * k;
  const kf::TrainingRoute r = kf::training_route(dh, BH, two != 0, N, k, nq);
  *prow = r.prow;
  *blocks = r.blocks32;
  return r.rows32 ? 32 : 16;
}
extern "C" int attention(int dh, int B, int H, int R, int qoff, int T, int empty, int *ns) {
  const kf::AttentionRoute r = kf::attention_route(dh, B, H, R, qoff, T, 8192, empty != 0);
  *ns = r.ns;
  return r.tiled ? 2 : r.wide ? 1 : 0;
}
extern "C" int plain_rows(int t128, int t160, int K) { return kf::plain_tile_rows(t128, t160, K); }
extern "C" int columns(int fp32, int M, int R) { return kf::value_columns(fp32 != 0, M, R); }
extern "C" int two_groups(int fp32, int tiles, int nk) { return kf::two_groups(fp32 != 0, tiles, nk); }
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "r.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2606_10820_amd", "csrc"),
                    str(d / "r.cpp"), "-o", str(d / "r.so")], check=True)
    L = ctypes.CDLL(str(d / "r.so"))
    L.training.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong,
                           ctypes.POINTER(ctypes.c_int), ctypes.POINTER(ctypes.c_int)]

    def training(dh, BH, mask, N, k):
        prow, blocks = ctypes.c_int(), ctypes.c_int()
        rows = L.training(dh, BH, mask, N, k, ctypes.byref(prow), ctypes.byref(blocks))
        return rows, prow.value, blocks.value
    L.training_route = training

    def attention(dh, B, H, R, T, empty=False, qoff=0):
        ns = ctypes.c_int()
        return ("split", "wide", "tiled")[L.attention(dh, B, H, R, qoff, T, int(empty), ctypes.byref(ns))], ns.value
    L.attention_route = attention
    return L


# (d_head, heads, mask, N, k, rows per wavefront), time of 32 rows over 16 rows
@pytest.mark.parametrize("dh,BH,mask,N,k,want", [
    (64, 192, 0, 1024, 4, 32),   # OWT-shaped training batch: 0.92
    (64, 384, 0, 123, 2, 32),    # self-forcing rollout, round 1: 0.94
    (64, 384, 1, 123, 2, 32),    # and round 2: 0.86
    (64, 1024, 1, 16, 1, 16),    # a quarter of a workgroup's rows: 1.34
    (64, 2048, 0, 8, 8, 32),     # one block of 72 rows: 0.76
    (64, 128, 0, 1000, 1, 16),   # 2048 workgroups of long rows: 1.06
    (64, 128, 1, 1000, 1, 32),   # the same under M_D: 0.81
    (64, 384, 0, 100, 1, 32),    # 200 rows, one round: 0.83
    (64, 512, 1, 64, 2, 16),     # 256 rows, a round and a third: 1.08
    (64, 128, 0, 160, 1, 16),    # 384 workgroups: 1.11
    (64, 1024, 0, 86, 4, 16),    # last block of 46 rows: 1.19
    (64, 512, 0, 16, 8, 16),     # 144 rows, the second workgroup nearly empty: 1.20
    (64, 512, 0, 86, 4, 16),     # 430 rows: 1.17
    (64, 256, 1, 100, 4, 16),    # 800 rows: 1.18
    (64, 512, 0, 300, 2, 16),    # 900 rows: 1.16
    (64, 108, 0, 1000, 0, 16),   # causal, few workgroups: 1.10
    (128, 8, 0, 160, 1, 16),     # 24 workgroups: 1.21
    (128, 8, 1, 300, 4, 16),     # 160 workgroups: 1.99 (blocks across the halves)
    (128, 512, 0, 215, 4, 32),   # 0.79
    (128, 384, 0, 16, 2, 16),    # 48 rows: 1.14
    (128, 4096, 0, 32, 4, 16),   # 160 rows: 1.10
    (128, 256, 1, 86, 1, 32),    # 172 rows: 0.80
    (128, 96, 0, 123, 2, 32),    # 288 workgroups, last block of 113 rows: 0.86
    (32, 96, 1, 250, 2, 32),     # 0.83
    (32, 1024, 0, 160, 4, 32),   # last block of 32 rows among seven: 0.85
    (32, 32, 1, 1000, 1, 16),    # 512 workgroups: 16 rows as before
    (32, 1024, 0, 300, 2, 16),   # 900 rows: 1.13
    (32, 512, 0, 250, 4, 32),    # 0.80
])
def test_training_rows(routes, dh, BH, mask, N, k, want):
    assert routes.training_route(dh, BH, mask, N, k)[0] == want


def test_training_blocks_cover_the_rows_once(routes):
    """Blocks of 128 rows cut from row 0 on, or from each half of M_D by itself
    (512 rows a half on): every row in exactly one block."""
    for mask in (0, 1):
        for N in (1, 2, 63, 64, 65, 127, 255, 256, 257, 511, 512, 513, 1000):
            for k in (1, 2, 3, 7):
                nq = N + N * k if mask == 0 else 2 * N * k
                _, prow, blocks = routes.training_route(64, 1, mask, N, k)
                cut = mask == 1 and N * k >= 512
                assert prow == (N * k if cut else nq)
                per = -(-prow // 128)
                assert blocks == per * (nq // prow)


def test_gpu_shapes_reach_the_32_row_kernel(routes):
    from tests import test_gpu_training_attention_grids as G
    for mask, N, k, dh, BH in G.LARGE + G.HALVES:
        assert routes.training_route(dh, BH, mask, N, k)[0] == 32, (mask, N, k, dh, BH)


# (d_head, sequences, heads, rows, capacity, starts empty, kernel), time of the tiled
# kernel over the one of key splits or of one workgroup per 16 rows
@pytest.mark.parametrize("dh,B,H,R,T,empty,want", [
    (64, 1, 12, 32, 1024, False, "split"),    # one sequence, k = 16, 880 keys: 1.61
    (128, 1, 12, 32, 1024, False, "split"),   # 1.98
    (32, 1, 12, 34, 1024, False, "split"),    # 1.44
    (128, 4, 12, 32, 1024, False, "split"),   # 1.22
    (32, 8, 12, 34, 1024, False, "split"),    # 288 blocks without splits: 1.20
    (64, 2, 12, 34, 1024, False, "wide"),
    (64, 16, 12, 34, 1024, False, "tiled"),   # 0.68
    (128, 8, 12, 32, 1024, False, "tiled"),   # two splits: 0.90
    (32, 64, 12, 32, 1024, False, "tiled"),   # 0.65
    (64, 1, 12, 65, 1024, True, "tiled"),     # a prompt of 61: 0.82
    (64, 1, 12, 65, 128, True, "split"),      # no splits at 128 keys: 1.14
    (128, 1, 12, 65, 128, True, "split"),     # 1.37
    (32, 1, 12, 384, 1024, True, "split"),    # 288 blocks: 1.20
    (64, 4, 12, 96, 1024, True, "split"),     # 288 blocks: 1.14
    (64, 8, 12, 511, 1024, True, "tiled"),
    (64, 24, 16, 704, 1024, True, "tiled"),
    (64, 64, 12, 20, 128, True, "split"),     # fewer than 32 rows
])
def test_attention_kernel(routes, dh, B, H, R, T, empty, want):
    assert routes.attention_route(dh, B, H, R, T, empty)[0] == want


def test_attention_of_a_part_of_the_rows_is_never_tiled(routes):
    """The tiled kernel starts at row 0 of a step: the last layer's noise rows go elsewhere."""
    for B in (1, 8, 64, 512):
        for R in (33, 64, 200):
            assert routes.attention_route(64, B, 12, R, 1024, True, qoff=1)[0] != "tiled"


def test_gpu_shapes_reach_their_kernels(routes):
    from tests import test_gpu_attention_routes as G
    for kernel, d, H, B, n_ctx, N in G.DECODE:
        for R in (32, 33):
            assert routes.attention_route(d // H, B, H, R, n_ctx)[0] == kernel, (kernel, d, H, B, R)
    for d, H, B, rows in G.PREFILL:
        assert routes.attention_route(d // H, B, H, rows, 384, True) == ("tiled", 1), (d, H, B, rows)


# (fp32, tiles, K steps), time of two K groups over splits of K
@pytest.mark.parametrize("fp32,tiles,nk,want", [
    (1, 48, 24, True),     # out-projection at K = 768: 0.92
    (1, 64, 32, False),    # K = 1024: 1.17
    (1, 96, 128, False),   # MLP-down at K = 4096: 1.34
    (1, 72, 96, False),    # K = 3072: 1.19
    (1, 64, 10, True), (0, 64, 10, True),   # too short to split
    (0, 96, 48, False), (0, 96, 24, False),
    (1, 128, 96, True), (0, 256, 48, True), (0, 257, 48, False),
])
def test_k_groups_of_small_grids(routes, fp32, tiles, nk, want):
    assert bool(routes.two_groups(fp32, tiles, nk)) == want


def test_qkv_runs_no_tile_of_four_wavefronts(tmp_path):
    """The built library holds 128 x 128 tiles of four wavefronts for MLP-up and the heads,
    none for QKV (K = 1024: up to 1.32 times as long as eight)."""
    from tests.test_kernel_registers import LIB, READELF, _kernels
    if not (os.path.exists(LIB) and os.path.exists(READELF)):
        pytest.skip("needs the built library and llvm-readelf")
    four = [n for n, _ in _kernels(tmp_path) if "gemm_kernelIDF16bLi128ELi128ELi2ELi2E" in n]
    assert any("EpBias" in n for n in four) and any("EpHead" in n for n in four)
    assert [n for n in four if "EpQKV" in n] == []


# (M, N, K, rows of the four-wavefront tile or 0), its time over eight wavefronts of 128 rows
@pytest.mark.parametrize("M,N,K,want", [
    (11808, 768, 3072, 160),    # 0.73
    (16896, 1024, 4096, 160),   # 0.84
    (8192, 768, 3072, 128),     # 0.94
    (12288, 1024, 4096, 128),   # 0.96
    (19200, 768, 768, 0),       # 900 tiles of 128 rows, 720 of 160: 1.04 and more in either
    (18432, 768, 3072, 128),    # 160 rows against 128: 1.07
    (13312, 1024, 1024, 0),     # 160 rows: 1.04
    (4000, 768, 3072, 0),       # fewer than 256 tiles
    (8192, 768, 832, 0),        # an odd number of K steps
])
def test_plain_tiles(routes, M, N, K, want):
    tiles = lambda rows: -(-M // rows) * -(-N // 128)  # noqa: E731
    assert routes.plain_rows(tiles(128), tiles(160), K) == want


# (fp32, rows, rows per sequence, by column)
@pytest.mark.parametrize("fp32,M,R,want", [
    (0, 48, 8, False),     # k = 4, 6 sequences, a context off the 4-slot blocks: 8.8 us by column, 7.1 by row
    (0, 192, 8, False), (0, 224, 4, False),
    (0, 256, 8, True),     # whole blocks through a page table: 9.3 us by column, 9.7 by row
    (0, 256, 6, False),
    (0, 512, 8, True),     # whole blocks: 11.0 us by column, 11.6 by row
    (0, 512, 6, False), (0, 96, 1, False), (0, 513, 1, True), (1, 512, 8, False), (1, 513, 8, True),
])
def test_value_tiles(routes, fp32, M, R, want):
    assert bool(routes.columns(fp32, M, R)) == want
