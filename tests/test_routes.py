"""Which form a call takes (host decisions only, so this runs without a GPU): the lines of the dispatch rules, and that no rule asks for
more scratch than the call has."""
import ctypes as C

import pytest

from paper_2408_04275_amd import binding as mm
from test_gpu_f32_gradients import LONGER
from test_gpu_gemm_tiles import CUTS, SHAPES, WGRAD_SHAPES
from util import gemm_route


# the memory-side cache holds 256 MB; a shard whose arrays may still lie there from the pass before is not streamed
def test_optimizer_streams_only_what_cannot_be_cached():
    route = mm.load_library().mmtrain_route_adam
    route.argtypes = [C.c_int64, C.c_int32]
    for n, param_bytes, streamed in [(4 << 20, 2, 0), (12 << 20, 2, 0), (16 << 20, 2, 0), ((20 << 20) - 1, 2, 0), (20 << 20, 2, 1),
                                     (18 << 20, 4, 1), (17 << 20, 4, 0), (20 << 20, 0, 0), (24 << 20, 0, 1), (1 << 30, 2, 1)]:
        assert route(n, param_bytes) == streamed, (n, param_bytes)


# the sizes of the GPU parity tests take the forms that those tests name
@pytest.mark.parametrize("layout", [mm.GEMM_NT, mm.GEMM_NN])
@pytest.mark.parametrize("M,N,K,tile", SHAPES)
def test_tile_shapes(layout, M, N, K, tile):
    assert gemm_route(layout, M, N, K) == (*map(int, tile.split("x")), 0, 1)


@pytest.mark.parametrize("M,N,K,tile", WGRAD_SHAPES)
def test_weight_gradient_tile_shapes(M, N, K, tile):
    assert gemm_route(mm.GEMM_TN, M, N, K) == (*map(int, tile.split("x")), 0, 1)


def test_every_tile_shape_is_covered():
    assert {s[3] for s in SHAPES} == {"64x64", "64x128", "128x128", "192x128", "256x128", "160x256", "192x256", "224x256"}
    assert {s[3] for s in WGRAD_SHAPES} == {"64x64", "64x128", "128x128", "256x128"}


@pytest.mark.parametrize("M,N,K,room,chunks", CUTS)
def test_cuts_along_k(M, N, K, room, chunks):
    size = room * M * N * 4 if room else mm.mmtrain_gemm_workspace_bytes(mm.GEMM_NN, M, N)
    assert gemm_route(mm.GEMM_NN, M, N, K, size)[2:] == (0, chunks)
    assert gemm_route(mm.GEMM_NN, M, N, K)[2:] == (0, 1)               # no scratch, no cut


@pytest.mark.parametrize("layout", [mm.GEMM_NN, mm.GEMM_TN])
def test_last_round_cut_along_k(layout):
    # 288 tiles on 256 compute units: 32 of them in the last round, in 8 chunks (test_gpu_ops.py runs this product)
    assert gemm_route(layout, 4360, 4040, 4872, mm.mmtrain_gemm_workspace_bytes(layout, 4360, 4040)) == (256, 256, 32, 8)


@pytest.mark.parametrize("layout", [mm.GEMM_NT, mm.GEMM_NN, mm.GEMM_TN])
def test_cuts_stay_within_their_scratch(layout):
    for M in (8, 264, 520, 1032, 3000, 4360, 8192):
        for N in (64, 1024, 1032, 4096, 11008):
            for K in (8, 4096, 12288, 22016, 25608):
                for room in (0, 256, M * N * 4, 3 * M * N * 4, 1 << 24, 1 << 40):
                    tm, tn, tail, chunks = gemm_route(layout, M, N, K, room)
                    assert chunks == 1 or chunks * (tail * 65536 if tail else M * N) * 4 <= room
                    assert layout != mm.GEMM_NT or chunks == 1


@pytest.mark.parametrize("layout", [mm.GEMM_NN, mm.GEMM_TN])
def test_the_size_query_restricts_no_cut(layout):
    for M in (8, 264, 368, 520, 1032, 2304, 3000, 4360, 8192):
        for N in (64, 1024, 1032, 4096, 11008):
            for K in (8, 4096, 12288, 22016, 25608):
                size = mm.mmtrain_gemm_workspace_bytes(layout, M, N)
                assert gemm_route(layout, M, N, K, size) == gemm_route(layout, M, N, K, 1 << 40)


# a K of up to four steps of 64: 256 x 256 where its rounds are well filled; the smaller tiles where they are not, and from K = 257 on
def test_short_contractions():
    for M, N, K in [(28672, 4096, 64), (4096, 4096, 16), (4096, 11008, 128), (22016, 4096, 256), (6144, 2048, 160)]:
        assert gemm_route(mm.GEMM_TN, M, N, K) == (256, 256, 0, 1), (M, N, K)
    for layout in (mm.GEMM_NT, mm.GEMM_NN):
        for M, N, K in [(28360, 7384, 16), (9504, 4344, 16), (1000, 28672, 192), (1000, 28672, 256)]:
            assert gemm_route(layout, M, N, K) == (256, 256, 0, 1), (M, N, K)
        assert gemm_route(layout, 6000, 4096, 128)[:2] == (64, 128)     # 1.5 rounds of 256 x 256
    assert gemm_route(mm.GEMM_TN, 1024, 4096, 64)[:2] == (64, 128)
    assert gemm_route(mm.GEMM_NT, 1000, 28672, 264)[:2] != (256, 256)


def test_operands_from_hbm_need_a_larger_gain():
    assert gemm_route(mm.GEMM_NN, 1397, 28672, 5120)[:2] == (256, 256)  # 293 MB of weights, 4 % by the model; 13 % slower when measured
    assert gemm_route(mm.GEMM_NN, 795, 28672, 4096)[:2] == (224, 256)   # 10 % by the model


# fp32: short contractions over many tiles stay on the vector ALUs
def test_fp32_short_contractions():
    route = mm.load_library().mmtrain_route_gemm_f32
    for layout, K, matrix in [(mm.GEMM_TN, 80, 0), (mm.GEMM_TN, 96, 1), (mm.GEMM_NN, 64, 0), (mm.GEMM_NN, 72, 1), (mm.GEMM_NT, 8, 1)]:
        assert route(layout, 1352, 3288, K) == matrix, (layout, K)      # 1144 tiles of 64 x 64
        assert route(layout, 640, 640, K) == 1                          # 100


# Weight gradients added to fp32 contents: every second workgroup starts later only where the launch has two rounds of tiles and more and few
# enough tokens to gain by it.  (M, N, tokens): whether
@pytest.mark.parametrize("M,N,K,late", [(8192, 4096, 300, True), (12288, 4096, 1031, True), (28672, 4096, 2048, True), (8192, 4096, 4096, True), (22016, 4096, 4096, True),
                                        (6144, 4096, 1031, True), (6144, 4096, 2048, False), (4096, 4096, 1031, False), (8192, 4096, 4097, False),
                                        (22016, 4096, 8192, False), (8192, 12288, 6144, False), (8192, 8192, 200000, False)])
def test_late_start_of_fp32_gradients(M, N, K, late):
    route = mm.load_library().mmtrain_route_late_start
    route.argtypes = [C.c_int32] * 5
    units = route(M, N, K, 1, 256)
    assert (0 < units <= 30000 // 512) if late else units == 0
    assert route(M, N, K, 0, 256) == 0                                 # nothing is read: nothing to hide


# fp32 gradients of any width that the operands can have (the feed-forward width of test_gpu_f32_gradients.py's widest layer among them)
@pytest.mark.parametrize("N", [(1 << 21) + 16, (1 << 22) + 8, (1 << 23) - 65536])
def test_wide_fp32_gradients_stay_on_the_matrix_cores(N):
    route = mm.load_library().mmtrain_route_late_start
    route.argtypes = [C.c_int32] * 5
    assert route(272, N, 1, 1, 256) >= 0


@pytest.mark.parametrize("H,nh,d,F,T,tile1,tile2", LONGER)
def test_tiles_of_fp32_gradients(H, nh, d, F, T, tile1, tile2):
    for (M, N), tile in (((2 * F, H), tile1), ((H, F), tile2)):
        assert gemm_route(mm.GEMM_TN, M, N, T) == (*map(int, tile.split("x")), 0, 1)
        assert ((M + 255) // 256) * ((N + 255) // 256) > 128                 # a launch of its own, not one of a group


# parts of an input gradient are added up by the normalisation's backward kernel where that is faster than a kernel of their own
def test_widths_whose_normalisation_adds_parts():
    for dtype in (mm.F32, mm.BF16):
        for layernorm in (0, 1):
            for H in (256, 1024, 1040, 2048, 4096, 4112, 5120, 8192):
                adds = mm.load_library().mmtrain_route_norm_parts(dtype, layernorm, H)
                assert adds == (dtype == mm.BF16 and not layernorm and 1024 < H <= 4096), (dtype, layernorm, H)


# dQ and dK/dV of fp32 attention run together only where dK/dV of 64-wide heads leaves the chip part empty; a grid holds 65535 rows
def test_launches_of_f32_attention_backward():
    route = mm.load_library().mmtrain_route_attn_f32_bwd
    for T, nh, nkv, d, launches in [(512, 4, 4, 64, 1), (1792, 4, 4, 64, 1), (1793, 4, 4, 64, 2), (224, 32, 32, 64, 1), (225, 32, 32, 64, 2),
                                    (8192, 4, 1, 64, 2), (8192, 32, 32, 128, 1), (9, 40000, 40000, 64, 2), (2, 40000, 40000, 128, 2)]:
        assert route(T, nh, nkv, d) == launches, (T, nh, nkv, d)


def _encoder_sums(H, heads, d, F, T):
    """Weight gradients of a bf16 encoder layer that are computed together, and the partial sums at the end of its backward pass."""
    ceil = lambda a, b: -(-a // b)  # noqa: E731
    nq = heads * d
    products = [(m, n) for m, n in ((H, F), (F, H), (H, nq), (3 * nq, H)) if ceil(m, 256) * ceil(n, 256) <= 128]
    norm = min(ceil(T, 4), 512) if H <= 1024 else min(T, 1024)
    jobs = [(norm, H)] * 6 + [(ceil(T, 4 if T <= 3072 else 8 if T <= 6144 else 16), F), (ceil(T, 32), 3 * nq)]
    return products, jobs


# sums ride along only where they are done about when the products are: either side, as measured (us alone and along at the rule)
@pytest.mark.parametrize("H,heads,d,F,T,along", [
    (512, 8, 64, 2048, 300, 1), (512, 8, 64, 2048, 9536, 1), (768, 12, 64, 3072, 900, 0), (1024, 16, 64, 4096, 64, 1), (1024, 16, 64, 4096, 256, 1),
    (1024, 16, 64, 4096, 300, 1), (1024, 16, 64, 4096, 9536, 1), (1280, 16, 80, 5120, 900, 0), (1280, 16, 80, 5120, 2304, 0), (1280, 16, 80, 5120, 4111, 1),
    (1408, 16, 96, 6144, 300, 0), (1408, 16, 96, 6144, 900, 0), (1408, 16, 96, 6144, 2304, 1), (1536, 24, 64, 6144, 300, 0),
    (1536, 24, 64, 6144, 1500, 0), (1536, 24, 64, 6144, 4111, 1)])
def test_sums_ride_along_where_there_is_time(H, heads, d, F, T, along):
    products, jobs = _encoder_sums(H, heads, d, F, T)
    flat = lambda pairs: (C.c_int32 * (2 * len(pairs)))(*[v for p in pairs for v in p])  # noqa: E731
    assert mm.load_library().mmtrain_route_sums_along(len(products), flat(products), T, len(jobs), flat(jobs), 256) == along


# long input gradients: cut in three and more, which beats the tiles of 96 and 160 rows where they would fit too, but not in two, which does not
@pytest.mark.parametrize("M,N,K,route", [
    (1031, 2048, 11008, (256, 256, 0, 6)), (1984, 1280, 14336, (256, 256, 0, 6)), (576, 5120, 11264, (256, 256, 0, 4)), (1088, 4096, 9728, (256, 256, 0, 3)),
    (768, 3072, 12800, (256, 256, 0, 7)), (640, 8192, 13824, (160, 128, 0, 1)), (576, 8192, 27648, (160, 128, 0, 1)), (2304, 1024, 4096, (96, 128, 0, 1))])
def test_cuts_against_the_tiles_between(M, N, K, route):
    assert gemm_route(mm.GEMM_NN, M, N, K, 1 << 40) == route


# operands beyond 96 MB: these tiles need 15 % more of them than the older shapes, 22 % up to 1024 rows, or a full round
@pytest.mark.parametrize("layout", [mm.GEMM_NT, mm.GEMM_NN])
@pytest.mark.parametrize("M,N,K,tile", [
    (284, 7368, 10048, "128x128"), (442, 8248, 7616, "192x128"), (300, 12288, 4096, "192x128"), (600, 8192, 8192, "160x128"), (520, 4096, 11008, "128x128"), (640, 4096, 11008, "96x128"), (2048, 2176, 12032, "160x128"),
    (1031, 4096, 11008, "160x128"), (300, 11008, 4096, "160x128")])
def test_tiles_between_from_hbm(layout, M, N, K, tile):
    assert "%dx%d" % gemm_route(layout, M, N, K)[:2] == tile
