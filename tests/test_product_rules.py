"""The rules that choose the kernel of an expert product, on the host: what each range of sizes is served by, and that long
contraction indices reach only kernels whose offsets hold them."""
import ctypes as C

import pytest

import paper_2205_10034_amd as M

from gpu_util import product_kernel


def second_product(N, K, A, E=1, k=1):
    return product_kernel(M.MoEConfig(T=A // k, d_model=N, d_ff=K, E=E, k=k), 1)


LONG = 3355456          # first multiple of 64 whose 320 rows of bf16 reach 2 GiB
L22, L23, L24, L25 = (1 << n for n in (22, 23, 24, 25))


@pytest.mark.parametrize("N", [64, 320, 512])
def test_few_assignments_take_any_contraction_length(N):
    """Up to 16 assignments the matrix-vector kernels (64-bit offsets) serve what the weight-streaming ones cannot."""
    for K in (64, 4096, LONG - 64, LONG, L22, L24, L25, 1 << 27):
        for A in (1, 8):
            assert second_product(N, K, A) == "gemv 8"
        for A in (9, 12, 16):
            assert second_product(N, K, A) == ("stream 64x32" if K < LONG else "gemv 16")
            assert second_product(N, K, A, E=8, k=2 if A % 2 == 0 else 1) == ("stream 64x32" if K < LONG else "gemv 16")


@pytest.mark.parametrize("A", [17, 30, 200, 700, 3000])
def test_long_contractions_beyond_sixteen_assignments(A):
    """256-row tiles hold up to 2^22 values of the contraction index, narrow ones (feature counts that are no multiple of
    256, or below) up to 2^23; beyond, the call is refused."""
    for K in (LONG, L22 - 64, L22, L22 + 64, L23 - 64, L23, L24, L25):
        assert second_product(64, K, A) == ("grouped 128" if K < L23 else "refused")
        assert second_product(320, K, A) == ("grouped 256" if K < L22 else "grouped 128" if K < L23 else "refused")
        assert second_product(512, K, A) in (("grouped 256", "refused") if K < L22 else ("refused",))


def test_no_kernel_is_chosen_beyond_its_offsets():
    rows = {"stream 64x32": 64, "stream 64x64": 64, "stream 128x64": 128, "stream 128x128": 128, "stream 128x192": 192,
            "stream 256x64": 256, "stream 256x128": 256, "grouped 128": 128, "grouped 256": 256, "grouped 320": 320}
    seen = set()
    for act in ("gelu", "swiglu"):
        for E, k in ((1, 1), (3, 1), (8, 2), (64, 2), (128, 6)):
            for per in (1, 7, 12, 20, 33, 41, 60, 90, 120, 150, 400, 1100):
                T = max(1, per * E // k)
                for N in (64, 128, 448, 1024, 4096):
                    for K in (64, 1024, 4096, 8192, LONG - 64, LONG, L22, L23 - 64, L23, L25):
                        for second, cfg in ((0, M.MoEConfig(T=T, d_model=K, d_ff=N, E=E, k=k, act=act)), (1, M.MoEConfig(T=T, d_model=N, d_ff=K, E=E, k=k, act=act))):
                            name = product_kernel(cfg, second)
                            seen.add(name)
                            if name in rows:
                                assert rows[name] * K * 2 < 1 << 31, (name, cfg)
    assert seen >= set(rows) | {"gemv 8", "gemv 16", "refused"}, seen


def test_tuning_keys_keep_the_streaming_kernels_out():
    for key, value in ((M.MOE_TUNE_GEMM_TILE_ROWS, 256), (M.MOE_TUNE_GEMM_MFMA, 16)):
        M.moe_set_tuning(key, value)
        try:
            assert second_product(512, 1024, 12) == "gemv 16" and second_product(512, 1024, 200) == "grouped 256"
        finally:
            M.moe_set_tuning(key, 0)
    M.moe_set_tuning(M.MOE_TUNE_FEW_TOKEN_KERNELS, 0)
    try:
        assert second_product(512, 1024, 4).startswith("grouped") and second_product(512, 1024, 12).startswith("grouped")
    finally:
        M.moe_set_tuning(M.MOE_TUNE_FEW_TOKEN_KERNELS, 1)


def test_tiles_beyond_one_round_need_long_rows_of_weights():
    """Shapes that measured slower than the grouped GEMM: several rounds of tiles over few values of the contraction index,
    row counts just below a tile edge that uneven routing crosses, two rounds of 128 x 192."""
    first = lambda rows, E, N, K, act="gelu": product_kernel(M.MoEConfig(T=rows * E, d_model=K, d_ff=N, E=E, k=1, act=act), 0)
    for rows, E, N, K in ((36, 16, 10752, 512), (28, 64, 1792, 512), (27, 16, 9984, 576), (34, 32, 3136, 896),   # 128 x 64
                          (62, 128, 7296, 512), (85, 32, 7168, 512), (46, 16, 2560, 512), (66, 64, 576, 1024),   # 256 x 128, 128 x 128
                          (105, 96, 512, 1088), (128, 32, 1536, 2560), (124, 64, 768, 3584),               # over 96 rows
                          (381, 16, 1216, 1408), (384, 32, 640, 768), (209, 16, 1408, 704), (206, 24, 768, 640)):
        assert first(rows, E, N, K) == "grouped 256", (rows, E, N, K)
    # beside them: one round, longer rows, a row count clear of the edge
    for rows, E, N, K, want in ((30, 64, 1280, 1280, "128x64"), (35, 64, 1152, 832, "128x64"), (30, 8, 4096, 512, "128x64"), (60, 8, 3520, 512, "128x128"), (62, 32, 1664, 2560, "128x128"),
                                (38, 128, 1600, 832, "256x128"), (64, 64, 8192, 2048, "256x128"), (330, 16, 1216, 1408, "128x128"),
                                (170, 16, 1408, 704, "128x192"), (209, 16, 1408, 4096, "128x192")):
        assert first(rows, E, N, K) == "stream " + want, (rows, E, N, K)
    # two products per tile: shorter rows still pay
    for rows, E, N, K, want in ((28, 128, 1600, 768, "stream 128x64"), (34, 16, 5952, 512, "grouped 256"), (80, 128, 896, 768, "stream 256x128"), (80, 128, 896, 704, "grouped 256")):
        assert first(rows, E, N, K, "swiglu") == want, (rows, E, N, K)


def test_the_rule_follows_the_products_place_and_not_its_sizes():
    """d_ff == d_model: each product keeps its own lines (one round of 256 x 192 tiles: not with an activation in the end)."""
    for rows, E, d, first, second in ((112, 16, 2112, "grouped 256", "stream 256x192"), (112, 16, 2176, "grouped 256", "stream 256x192"),
                                      (120, 128, 4096, "stream 256x192", "stream 256x192"), (120, 128, 1920, "stream 256x192", "stream 256x192"),
                                      (120, 128, 1216, "stream 256x192", "stream 256x192"), (130, 128, 4096, "stream 256x192", "stream 256x192")):
        for k in (2, 4):
            cfg = M.MoEConfig(T=rows * E // k, d_model=d, d_ff=d, E=E, k=k)
            assert product_kernel(cfg, 0) == first and product_kernel(cfg, 1) == second, (rows, E, d)
        beside = M.MoEConfig(T=rows * E // 2, d_model=d, d_ff=d + 64, E=E, k=2)
        assert product_kernel(beside, 1) == second


def test_products_of_97_to_160_rows_that_stay_with_the_grouped_kernel():
    """Shapes that measured slower on the streaming kernel: tiles that fill their rounds where an expert's rows are likely to spill
    into a second tile, and combines (one choice per token) of short rows.  A capacity that rules a second tile out lifts the first."""
    kernel = lambda rows, E, N, K, k, cf=0.0: product_kernel(M.MoEConfig(T=rows * E // k, d_model=N, d_ff=K, E=E, k=k, capacity_factor=cf), 1)
    for rows, E, N, K, k in ((155, 64, 896, 5056, 2), (142, 64, 896, 2752, 2), (148, 128, 896, 1792, 2), (135, 16, 4096, 4096, 2),
                             (134, 32, 4032, 1984, 1), (121, 64, 3584, 1152, 1), (123, 96, 1280, 2496, 1)):
        assert kernel(rows, E, N, K, k) == "grouped 256", (rows, E, N, K, k)
    for rows, E, N, K, k, cf in ((142, 64, 1088, 2752, 2, 0.0), (134, 64, 896, 2752, 2, 0.0), (142, 64, 896, 2752, 2, 1.25), (123, 96, 1280, 2560, 1, 0.0),
                                 (155, 64, 896, 5056, 2, 1.0), (148, 128, 1088, 1792, 2, 0.0)):
        assert kernel(rows, E, N, K, k, cf) == "stream 256x192", (rows, E, N, K, k, cf)


def test_one_round_of_256_weight_rows():
    """Up to 96 rows, long rows of weights: 256 x 128 only where 128 x 128 makes more than one round (with 16 experts and more only with
    room for a hot expert's further row tiles).  Shapes on both sides, either product."""
    for rows, E, N, K, act, want in ((43, 12, 1344, 3584, "swiglu", "128x128"), (86, 12, 1344, 4032, "swiglu", "128x128"), (82, 12, 2624, 1216, "gelu", "128x128"),  # 252 tiles
                                     (90, 12, 1472, 3584, "swiglu", "256x128"), (82, 12, 2752, 2048, "gelu", "256x128"),
                                     (60, 16, 2816, 2304, "gelu", "256x128"), (60, 16, 2880, 2304, "gelu", "128x128"),   # 176 and 192 tiles of 256
                                     (60, 8, 8192, 2304, "gelu", "256x128"), (72, 24, 1088, 4416, "swiglu", "128x128"),
                                     (60, 176, 192, 4096, "gelu", "128x128")):                                          # fewer features than a tile
        assert product_kernel(M.MoEConfig(T=rows * E // 2, d_model=K, d_ff=N, E=E, k=2, act=act), 0) == "stream " + want, (rows, E, N, K, act)
    for rows, E, N, K, k, want in ((96, 12, 2688, 2624, 1, "128x128"), (54, 48, 576, 4288, 1, "128x128"), (78, 12, 2688, 2560, 2, "128x128"),
                                   (66, 48, 576, 3776, 2, "128x128"), (60, 24, 1536, 2304, 2, "256x128"), (54, 12, 2752, 3584, 1, "256x128")):
        assert product_kernel(M.MoEConfig(T=rows * E // k, d_model=N, d_ff=K, E=E, k=k), 1) == "stream " + want, (rows, E, N, K, k)


def test_short_rows_of_weights_on_256_weight_rows():
    """Up to 96 rows, several rounds of tiles: the line of each end, lowest for the plain one, highest for the combine."""
    second = lambda rows, E, N, K, k: product_kernel(M.MoEConfig(T=rows * E // k, d_model=N, d_ff=K, E=E, k=k), 1)
    for rows, E, N, K, k, want in ((64, 64, 2048, 512, 2, "stream 256x128"), (64, 64, 2048, 448, 2, "grouped 256"), (64, 64, 2048, 512, 1, "grouped 256"),
                                   (64, 64, 2048, 768, 1, "grouped 256"), (70, 32, 2176, 768, 1, "grouped 256"), (64, 64, 2048, 832, 1, "stream 256x128")):
        assert second(rows, E, N, K, k) == want, (rows, E, N, K, k)


def f32_rows(rows, E, N, K, cf=0.0, act="gelu", layout="output_major", second=1):
    """Tile rows of a float32 product [rows E, K] -> N."""
    f = M.lib().moe_test_f32_tile_rows
    f.restype = C.c_int32
    d, h = (N, K) if second else (K, N)
    cfg = M.MoEConfig(T=rows * E, d_model=d, d_ff=h, E=E, k=1, act=act, dtype="f32", capacity_factor=cf)
    return f(C.byref(cfg.c()), second + 2 * (layout == "input_major"))


def test_float32_tiles_of_160_rows():
    """Not where an expert is likely to overflow them and open a further round, where features or rows leave them half empty, or
    where tiles of 64 rows are as full; a capacity rules the overflow out."""
    for rows, E, N, K, cf in ((256, 64, 256, 4096, 0.0), (271, 32, 512, 7040, 0.0), (241, 64, 192, 11136, 1.25), (339, 7, 1472, 5696, 1.25),
                              (172, 32, 512, 3648, 0.0), (170, 16, 1024, 2048, 0.0), (491, 64, 128, 2432, 1.25)):
        assert f32_rows(rows, E, N, K, cf) != 160, (rows, E, N, K, cf)
    for rows, E, N, K, cf in ((256, 16, 1024, 4096, 0.0), (256, 16, 4096, 1024, 1.25), (256, 64, 256, 4096, 1.25), (64, 32, 1024, 2048, 0.0),
                              (512, 16, 2048, 2048, 1.25), (17, 64, 512, 2048, 0.0)):
        assert f32_rows(rows, E, N, K, cf) == 160, (rows, E, N, K, cf)


def test_float32_tiles_of_80_rows():
    """Not where random routing opens a further round of the first four, nor in the fifth and sixth, nor for two to three rounds of
    SwiGLU on input-major weights."""
    for rows, E, N, K, cf in ((140, 16, 512, 1088, 1.25), (1016, 8, 704, 1024, 1.25), (453, 16, 512, 1536, 1.25), (260, 16, 1344, 1280, 0.0)):
        assert f32_rows(rows, E, N, K, cf) == 64, (rows, E, N, K, cf)
    for rows, E, N, K in ((787, 8, 192, 2944), (599, 8, 960, 3264), (66, 16, 896, 1792)):
        assert f32_rows(rows, E, N, K) == 80, (rows, E, N, K)
    for rows, N, first in ((375, 1024, 64), (66, 1792, 80)):
        E = 8 if rows == 375 else 16
        assert f32_rows(rows, E, N, 512, 1.25, "swiglu", "output_major", 0) == 80
        assert f32_rows(rows, E, N, 512, 1.25, "swiglu", "input_major", 0) == first


def test_float32_copy_in_the_first_product():
    """16 MB of dispatched rows and more are copied by a kernel of their own where the product has fewer than 768 features."""
    copies = M.lib().moe_test_first_product_copies
    copies.restype = C.c_int32
    for T, d, f, E, k, cf, dtype, want in ((4096, 1024, 704, 8, 1, 0.0, "f32", 0), (4095, 1024, 704, 8, 1, 0.0, "f32", 1), (4096, 1024, 768, 8, 1, 0.0, "f32", 1),
                                           (2048, 1024, 64, 8, 2, 0.0, "f32", 0), (2048, 1024, 64, 8, 2, 0.5, "f32", 1), (8192, 1024, 128, 8, 2, 0.0, "bf16", 0)):
        assert copies(C.byref(M.MoEConfig(T=T, d_model=d, d_ff=f, E=E, k=k, capacity_factor=cf, dtype=dtype).c())) == want, (T, d, f, E, k, cf, dtype)
