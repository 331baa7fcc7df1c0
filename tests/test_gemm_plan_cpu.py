"""The tile plan of the GEMM (plan_gemm, a host function): what it picks where
several tiles were timed, and that every plan is one the launcher can run."""

import random

import pytest

from tests._plan import BF16, DOWN, F32, FEW, FUSES, SPLIT, TILES, plan_gemm

SPLIT_WS_MAX, MAX_SPLIT = 64 << 20, 16


def _dims(tile):
    return tuple(int(v) for v in TILES[tile].rstrip("ak").split("x"))


# (tokens, k, outputs, rank, a plain product): measured us of the plans near
# the fastest and of one that another cost model had chosen, all timed in turn
# on one gfx950 with weights read from memory
@pytest.mark.parametrize("T,K,N,rank,plain,us", [
    (32, 2560, 2560, 0, True, {"32x64a/4": 10.3, "64x64/4": 10.3, "32x128a/4": 10.6, "32x64a/6": 11.2}),
    (9, 4096, 4096, 0, True, {"gemv": 11.2, "32x128a/4": 12.4, "64x64/4": 12.4}),
    (16, 3584, 4416, 0, True, {"64x64/3": 12.4, "32x64a/3": 12.5, "gemv": 17.6}),
    (11, 9792, 2112, 0, True, {"32x64a/6": 15.7, "64x64/6": 16.1, "gemv": 28.7}),
    (17, 9728, 2560, 0, True, {"64x64/6": 16.2, "32x64a/6": 16.9}),
    (65, 2560, 2560, 0, True, {"64x64/3": 11.4, "128x128/8": 15.2}),
    (129, 2560, 2560, 0, True, {"64x64/2": 13.0, "128x128/6": 17.3}),
    (80, 4096, 2560, 0, True, {"64x64/3": 13.8, "128x64a/4": 14.4, "128x128/11": 17.2}),
    (160, 4096, 2560, 0, True, {"64x64/2": 15.5, "128x64a/3": 16.1, "128x128/6": 18.2}),
    (448, 4096, 2560, 0, True, {"128x128a/3": 22.5, "128x64a/1": 25.2}),
    (768, 9728, 2560, 0, True, {"128x256a/4": 54.3, "128x128a/2": 56.8, "128x64a/1": 65.8}),
    (256, 12288, 4096, 0, True, {"128x128a/4": 42.0, "128x256a/8": 43.0, "128x64a/2": 49.7}),
    (512, 12288, 4096, 0, True, {"128x256a/4": 63.7, "128x64a/1": 80.1}),
    (1152, 2560, 2560, 0, True, {"128x128a/1": 25.8, "128x128/1": 30.1}),
    (65, 4096, 24576, 0, True, {"128x96k/1": 44.4, "128x128a/1": 46.1, "128x192k/2": 49.0}),
    (4160, 12288, 4096, 0, True, {"128x256a/1": 466, "128x256/1": 556}),
    (8256, 12288, 4096, 0, True, {"128x256a/1": 851, "256x256a/1": 913}),
    (13120, 9728, 2560, 0, True, {"128x256a/1": 672, "256x256a/1": 734}),
    (7168, 2560, 6144, 0, False, {"256x256a/1": 206.9, "256x192a/1": 214.9, "128x192k/1": 233.7}),
    (5120, 2560, 6144, 16, False, {"256x256a/1": 160.6, "128x192k/1": 192.6}),
    (8192, 2560, 6144, 32, False, {"256x256a/1": 259.0, "256x192a/1": 274.4, "128x192k/1": 319.6}),
    (5120, 4096, 6144, 16, False, {"256x256a/1": 238.1, "128x192k/1": 287.7}),
    (1152, 2560, 6144, 16, False, {"128x256/1": 52.7, "128x256a/1": 57.2}),
    (5384, 704, 4096, 16, False, {"128x256/1": 57.9, "128x256a/1": 62.6, "128x128/1": 74.8}),
    (316, 256, 18432, 24, False, {"128x256/1": 14.3, "128x256a/1": 18.8, "128x128/1": 18.9}),
    (6144, 4096, 6144, 16, False, {"256x192a/1": 286.2, "128x192k/1": 353.5}),
])
def test_plan_is_near_the_fastest_measured(T, K, N, rank, plain, us):
    tile, n_split, _ = plan_gemm(T, N, K, (rank + 15) // 16 * 16, SPLIT | FEW if plain else DOWN)
    name = f"{TILES[tile]}/{n_split}" if tile >= 0 else "gemv"
    assert name in us and us[name] <= 1.04 * min(us.values()), (name, us)


def test_every_plan_can_be_launched():
    rng = random.Random(36722)
    for _ in range(50000):
        T, K, N = int(2 ** rng.uniform(0, 13.5)), 64 * int(2 ** rng.uniform(0, 7.6)), 64 * int(2 ** rng.uniform(0, 9))
        rank = rng.choice([0, 0, 0, 8, 16, 32, 33, 64])
        r_pad = (rank + 15) // 16 * 16
        may = rng.choice([DOWN, DOWN if rank > 32 else 0]) if rank else rng.choice([0, SPLIT, FEW, SPLIT | FEW])
        mode = BF16 if rank else rng.choice([BF16, F32])
        tile, n_split, kt_split = plan_gemm(T, N, K, r_pad, may, mode)
        case = (T, K, N, rank, may, mode, tile, n_split, kt_split)
        if tile < 0:  # the GEMV
            assert T <= 16 and n_split == 1, case
            continue
        bm, bn = _dims(tile)
        assert N % bn == 0, case
        assert bm != 32 or (may & FEW and T <= 32), case   # these sum no low-rank term
        assert not rank or may & DOWN or TILES[tile] in FUSES, case
        assert bm == 32 or mode != F32 or T > 16, case     # logits in place of the GEMV's: summed in parts
        if n_split == 1:
            assert kt_split == 0, case
            continue
        n_kt = K // 64
        assert may & SPLIT and n_split <= MAX_SPLIT and (n_split - 1) * kt_split < n_kt <= n_split * kt_split, case
        assert n_split * T * N * 4 <= SPLIT_WS_MAX, case
