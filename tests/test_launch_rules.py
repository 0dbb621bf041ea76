"""Rules that choose between launches of the tiled kernels, at sizes where the choice was timed.  Needs no GPU."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def L():
    from paper_2506_02024_amd import binding, build

    if build.is_stale():
        build.build_library()
    return binding.lib()


def through_lds(L, bm, bn, M, K, split):
    f = L._ZN3nfp16rows_through_ldsEiillli                    # nfp::rows_through_lds
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 2 + [ctypes.c_int64] * 3 + [ctypes.c_int]
    return f(bm, bn, M, K, K, split)


@pytest.mark.parametrize("bm,bn,M,K,split,lds", [
    # odd slices of rows on lines, microseconds through LDS and straight into registers: 170.7 / 158.7, 165.7 / 152.4, 339.7 / 318.7
    (256, 256, 1024, 14336, 3, False), (256, 256, 900, 14336, 3, False), (256, 256, 900, 32768, 3, False),
    # even ones and whole rows: 181.0 / more, 171.8 / 169.1 (2048 tokens: one of the few that lose 2 %); smaller tiles: 184.2 / 192.8
    (256, 256, 1024, 14336, 2, True), (256, 256, 2048, 6400, 1, True), (256, 128, 1024, 14336, 3, True),
])
def test_how_row_major_planes_reach_a_tile(L, bm, bn, M, K, split, lds):
    assert through_lds(L, bm, bn, M, K, split) == lds


def partial_bytes(L, kind, M, N, K, which="24large_gemm_partial_bytes"):
    f = getattr(L, "_ZN3nfp%sEilll" % which)
    f.restype, f.argtypes = ctypes.c_size_t, [ctypes.c_int] + 3 * [ctypes.c_int64]
    return f(kind, M, N, K)


@pytest.mark.parametrize("M,N,K,split", [
    # E4M3 weights, 45 to 46 weight tiles of 128 rows (a tail past a multiple of eight), 31 Mi and more, three and four token tiles: two
    # slices of 128 x 128 20.6, 19.9 and 22.4 us, 64-token tiles unsplit 29.6, 27.1 and 29.7
    (144, 5840, 5840, True), (160, 5696, 5696, True), (176, 5840, 5840, True),
    # no tail, or a plane that stays in the L2s: unsplit
    (160, 6144, 4096, False), (208, 4480, 4480, False),
])
def test_e4m3_weights_on_64_token_tiles_with_a_tail(L, M, N, K, split):
    assert (partial_bytes(L, 2, M, N, K) > 0) == split


@pytest.mark.parametrize("M,N,K", [(160, 17616, 5872), (200, 17616, 5872), (256, 17616, 5872)])
def test_fp16_splits_beyond_the_fixed_scratch(L, M, N, K):
    # three slices of 256 x 256: 61, 72 and 81 us on packed planes, unsplit 78, 86 and 103; the entry point without a workspace takes
    # a split that fits
    for kind in (1, 4, 6):
        assert partial_bytes(L, kind, M, N, K) == 3 * M * N * 4 > 32 << 20
        assert 16384 + partial_bytes(L, kind, M, N, K, "24large_gemm_bounded_bytes") <= 32 << 20
    # FP8 mode: what fits
    assert partial_bytes(L, 2, 256, 5120, 32768) + 256 * 32768 + 16384 + 2048 <= 32 << 20


def test_fp16_splits_beyond_the_fixed_scratch_are_never_chosen_without_a_workspace(L):
    import random

    rng = random.Random(3)
    for _ in range(3000):
        M, N, K = rng.randrange(65, 257), rng.randrange(1, 70000), 16 * rng.randrange(1, 2000)
        for kind in (1, 4):
            free, bounded = (partial_bytes(L, kind, M, N, K, w) for w in ("24large_gemm_partial_bytes", "24large_gemm_bounded_bytes"))
            assert bounded <= free and (bounded == free or free > (32 << 20) - 16384)


@pytest.mark.parametrize("M,N,K,fused", [
    # up to 8 tokens: several weight tiles per workgroup, or rows of up to 3072 columns (microseconds fused / not: 10.0 / 10.9,
    # 11.1 / 11.9, 18.6 / 19.5, 4.1 / 5.5; 8.9 / 8.6, 11.3 / 10.8)
    (8, 11008, 3072, True), (8, 7680, 5120, True), (8, 10240, 8192, True), (8, 1024, 1024, True), (8, 1024, 3072, True),
    (8, 4096, 4096, False), (8, 3072, 7168, False), (8, 1024, 3088, False),
    # 9 to 16 tokens: up to 1280 columns (5.2 / 5.8; 7.3 / 6.8, 11.5 / 9.2)
    (16, 1024, 1024, True), (9, 1024, 1280, True), (9, 1024, 1296, False), (16, 2048, 2048, False), (16, 4096, 4096, False),
])
def test_which_batches_are_quantised_in_the_streaming_kernel(L, M, N, K, fused):
    f = L._ZN3nfp22small_gemm_fuses_quantElll                 # nfp::small_gemm_fuses_quant
    f.restype, f.argtypes = ctypes.c_bool, 3 * [ctypes.c_int64]
    assert f(M, N, K) == fused


def test_splits_of_more_than_256_tokens_and_the_fixed_scratch(L):
    # what fits the scratch unsplit gets a split that fits where there is no workspace, and the same one with a workspace unless
    # that outgrows the scratch
    import random

    size = L.nestedfp_gemm_workspace_size
    size.restype, size.argtypes = ctypes.c_size_t, 3 * [ctypes.c_int64] + [ctypes.c_int]
    rng = random.Random(4)
    for _ in range(3000):
        M, N, K = int(257 * 40 ** rng.random()), rng.randrange(1, 40000), 16 * rng.randrange(1, 2000)
        for kind in (1, 2, 4, 5):
            fp8 = kind in (2, 5)
            room = (32 << 20) - 16384 - (M * K + 4 * M + 512 if fp8 else 0)
            free, bounded = (partial_bytes(L, kind, M, N, K, w) for w in ("24large_gemm_partial_bytes", "24large_gemm_bounded_bytes"))
            if room >= 0:
                assert bounded <= room and (bounded == free or free > room - 512)
            else:
                assert bounded == free
            # where the query is within the scratch, both entry points sum in the same order
            if kind in (4, 5) and size(M, N, K, 1 if fp8 else 0) <= 32 << 20:
                assert bounded == free


@pytest.mark.parametrize("M,N,K,fused", [
    # 9 to 16 tokens, three weight tiles per workgroup and up to 3584 columns (us with a launch of its own and fused: 9.6 / 9.0, 14.2 / 13.7,
    # 8.3 / 8.7 with two tiles, 15.0 / 15.0)
    (16, 12288, 2048, True), (9, 16384, 3584, True), (9, 6144, 3072, False), (12, 16384, 4096, False),
])
def test_which_wide_layers_are_quantised_in_the_streaming_kernel(L, M, N, K, fused):
    f = L._ZN3nfp22small_gemm_fuses_quantElll                 # nfp::small_gemm_fuses_quant
    f.restype, f.argtypes = ctypes.c_bool, 3 * [ctypes.c_int64]
    assert f(M, N, K) == fused


def test_room_for_padded_codes_stays_inside_the_fixed_scratch(L):
    # The query of FP8 mode asks for rows of codes on 128-byte lines, decode batches included, but never takes a problem past the
    # scratch of the entry point without a workspace that would fit it with dense rows.
    import random

    rng = random.Random(5)
    size, scratch = L.nestedfp_gemm_workspace_size, 32 << 20
    size.restype, size.argtypes = ctypes.c_size_t, 3 * [ctypes.c_int64] + [ctypes.c_int]
    route = L._ZN3nfp11route_smallEillll                        # nfp::route_small
    route.restype, route.argtypes = ctypes.c_bool, [ctypes.c_int] + 4 * [ctypes.c_int64]

    def round256(n):
        return (n + 255) // 256 * 256

    padded = held_back = decode = 0
    for _ in range(6000):
        M, K = int(9000 ** rng.random()), 16 * rng.randrange(1, 2500)
        N = int(40000 ** rng.random())
        if rng.random() < 0.2:                                  # near the limit
            M, N = max(1, (scratch - rng.randrange(1 << 16)) // (K + 4)), rng.randrange(1, 64)
        sums = max(partial_bytes(L, kind, M, N, K, "24small_gemm_partial_bytes" if route(kind, M, N, K, K) else "24large_gemm_partial_bytes")
                   for kind in (2, 5))
        rest = 16384 + round256(4 * M) + round256(sums)
        dense, lines = rest + round256(M * K), rest + round256(M * ((K + 127) // 128 * 128))
        got = size(M, N, K, 1)
        assert got >= dense
        if dense <= scratch:
            assert got <= scratch
        if lines <= scratch or dense > scratch:
            assert got >= lines
            padded += lines > dense
            decode += lines > dense and M <= 64
        else:
            held_back += 1
        assert got in (dense, lines)                            # and for no other room
    assert padded > 1000 and decode > 500 and held_back > 5, (padded, decode, held_back)


@pytest.mark.parametrize("kind,cls", [(4, 1), (5, 2), (0, 3)])
def test_prices_above_256_tokens_can_be_fitted_again(L, kind, cls):
    # the model that fit_costs.py fits picks the launches that the library does, so its constants are the library's
    import random

    from paper_2506_02024_amd import fit_costs

    height = L._ZN3nfp17large_gemm_heightEilll                  # nfp::large_gemm_height
    height.restype, height.argtypes = ctypes.c_int, [ctypes.c_int] + 3 * [ctypes.c_int64]
    rng = random.Random(cls)
    heights, splits = set(), set()
    for _ in range(800):
        M, N, K = int(257 * 30 ** rng.random()), int(100 * 300 ** rng.random()), 16 * rng.randrange(20, 1500)
        launches, geo = zip(*fit_costs.tall_launches(cls, N, K, M))
        if max(g["slices"] for g in geo) * M * N * 4 + M * K > 30 << 20:
            geo, launches = zip(*((g, l) for g, l in zip(geo, launches) if g["slices"] == 1))
            if partial_bytes(L, kind, M, N, K) > 0:
                continue                                        # (rules of the fixed scratch decide as well)
        prices = fit_costs.price_tall(cls, fit_costs.columns(geo))
        (tm, tn, split, deep, tall), lowest = launches[prices.argmin()], prices.min()
        if sorted(prices)[1:2] and sorted(prices)[1] < lowest * (1 + 1e-9):
            continue
        assert height(kind, M, N, K) == tall, (M, N, K)
        assert partial_bytes(L, kind, M, N, K) == (split * M * ((N + 3) // 4 * 4) * 4 if split > 1 else 0), (M, N, K)
        heights.add(tall)
        splits.add(split)
    assert len(heights) >= 4 and len(splits) >= 4, (heights, splits)


@pytest.mark.parametrize("M,N,K", [
    # plain FP16, microseconds on 256 x 128 tiles and on 128 x 128 ones, which the floor of the memory bus prices alike: 80.7 / 96.0,
    # 91.0 / 102.9, 46.6 / 52.3, 76.2 / 96.1, 54.0 / 64.2, 56.2 / 65.3
    (125, 16142, 8128), (97, 15874, 9968), (97, 8118, 9456), (88, 10549, 15936), (113, 5328, 20160), (66, 16197, 6384),
])
def test_plain_fp16_layers_that_the_memory_bus_bounds(L, M, N, K):
    height = L._ZN3nfp17large_gemm_heightEilll                  # nfp::large_gemm_height
    height.restype, height.argtypes = ctypes.c_int, [ctypes.c_int] + 3 * [ctypes.c_int64]
    assert height(0, M, N, K) == 256


@pytest.mark.parametrize("kind,M,N,K", [
    # microseconds unsplit and in slices: plain FP16 28.5 / 20.2, 28.9 / 24.3, 29.5 / 23.7, FP16 mode 22.9 / 18.5, 19.2 / 14.9,
    # E4M3 40.1 / 32.9, 31.0 / 27.3
    (0, 504, 2560, 2560), (0, 767, 2560, 2560), (0, 377, 4224, 2816), (4, 470, 2432, 2432), (4, 310, 1456, 1456),
    (5, 995, 2016, 5872), (5, 379, 4864, 4864),
])
def test_workgroups_that_would_wait_for_memory_together_are_split(L, kind, M, N, K):
    assert partial_bytes(L, kind, M, N, K) > 0


@pytest.mark.parametrize("M", [649, 776])
def test_a_last_token_tile_of_few_rows_keeps_a_launch_unsplit(L, M):
    # the same layer with 9 and 8 rows in it: 21.5 us unsplit, 21.7 in two slices
    assert partial_bytes(L, 0, M, 2560, 2560) == 0
