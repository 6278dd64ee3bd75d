"""Host logic of the GEMM launcher (no GPU): which kernel variant and how many K chunks a shard GEMM gets.
Checks properties that must hold for any tuning of the cost table, plus the choices the benchmark
configurations rely on."""
import itertools

import pytest

import paper_2504_06095_amd as N
from paper_2504_06095_amd import binding as Bd

TILES = {(256, 256), (256, 224), (224, 256), (256, 192), (192, 256), (256, 128), (128, 256), (128, 128)}
FAKE_WS = 0x10000000  # an aligned address: registering touches no memory


@pytest.fixture
def workspace_1gib():
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS, 1 << 30) == 0
    yield 1 << 30
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0


def _tiles(c, M, N):
    return -(-M // c["tile_m"]) * -(-N // c["tile_n"])


def test_choice_is_well_formed_over_a_grid_of_shapes():
    for layout, M, Nn, K in itertools.product((0, 1, 2), (1, 100, 586, 2048, 7022), (8, 640, 1792, 12288), (0, 8, 750, 2048, 16384)):
        c = N.ntp_gemm_choice(layout, M, Nn, K)
        assert (c["tile_m"], c["tile_n"]) in TILES and c["wavefronts"] in (4, 8)
        assert c["k_splits"] == 1, "nothing is split without a workspace"
        if not c["ring"]:
            assert (c["tile_m"], c["tile_n"], c["wavefronts"], c["persistent"]) == (128, 128, 4, 0)
        if K < 128 or M * Nn < 2 * 128 * 128:
            assert not c["ring"], (layout, M, Nn, K)


def test_benchmark_configuration_choices():
    # config 2 (GPT-3 shape, TP 7 rank 0): one round of 256 x 224 tiles for fc1, two of 256 x 192 for fc2
    assert _tiles(N.ntp_gemm_choice(0, 2048, 7022, 12288), 2048, 7022) == 256
    c = N.ntp_gemm_choice(1, 2048, 12288, 7022)
    assert (c["tile_m"], c["tile_n"], c["persistent"]) == (256, 192, 1) and _tiles(c, 2048, 12288) == 512
    # the weight gradient of QKV on 256 x 256 tiles
    c = N.ntp_gemm_choice(2, 5376, 12288, 2048)
    assert (c["tile_m"], c["tile_n"], c["persistent"]) == (256, 256, 1)
    # a lone small tile set runs on 8 wavefronts per workgroup
    c = N.ntp_gemm_choice(0, 512, 586, 1024)
    assert (c["tile_m"], c["tile_n"], c["wavefronts"], c["ring"]) == (128, 128, 8, 1)


def test_split_k_only_for_skinny_long_k(workspace_1gib):
    # config 3 QKV projection (48 tiles of 256 x 256 over K = 8192), config 4 fc1, config 2 dC: split
    for (M, Nn, K) in [(4096, 640, 8192), (8192, 750, 16384), (2048, 1792, 12288)]:
        c = N.ntp_gemm_choice(0, M, Nn, K)
        assert 2 <= c["k_splits"] <= 8 and c["persistent"] == 0, (M, Nn, K, c)
        assert _tiles(c, M, Nn) * c["k_splits"] <= 2 * 256
        assert c["k_splits"] * M * (-(-Nn // 16) * 16) * 4 <= workspace_1gib
        assert -(-K // 64) // c["k_splits"] >= 8, "chunks of at least 8 K tiles"
    # enough tiles, or short K: never
    for (layout, M, Nn, K) in [(0, 2048, 7022, 12288), (1, 2048, 12288, 7022), (2, 7022, 12288, 2048), (1, 4096, 8192, 384), (0, 4096, 640, 512)]:
        assert N.ntp_gemm_choice(layout, M, Nn, K)["k_splits"] == 1, (layout, M, Nn, K)


def test_split_k_respects_the_workspace_size():
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS, 8 << 20) == 0  # 8 MiB: two slices of 4096 x 640 fp32 would need 21 MB
    try:
        assert N.ntp_gemm_choice(0, 4096, 640, 8192)["k_splits"] == 1
    finally:
        assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0


def test_small_tiles_where_two_workgroups_per_unit_hold_them(workspace_1gib):
    """64 x 64 tiles, uncut, on either side of two per compute unit, and of 1.3 where K-contiguous rows do not start on cache lines."""
    tile = lambda *s: (lambda c: (c["tile_m"], c["tile_n"], c["k_splits"]))(N.ntp_gemm_choice(*s))  # noqa: E731
    assert tile(0, 2048, 1024, 1024) == tile(1, 2048, 1024, 1024) == (64, 64, 1)      # 2.0 per unit
    assert tile(0, 576, 3776, 1024) == tile(1, 576, 3776, 1024) == (128, 128, 1)      # 2.07
    assert tile(0, 640, 2304, 1280) == tile(1, 640, 2304, 1264) == (64, 64, 1)        # 1.41
    assert tile(0, 640, 2304, 1264) == (128, 128, 1)
    assert tile(0, 1664, 640, 1904) == (64, 64, 1)                                    # 1.02
    assert tile(2, 640, 2304, 1280)[:2] != (64, 64)
    assert N.ntp_gemm_choice(0, 2048, 1024, 1024)["wavefronts"] == 4


def test_chunks_fit_the_units_of_an_xcd(workspace_1gib):
    """A tile and its K chunks are on one of the eight XCDs: 128 x 128 tiles are cut into no more chunks than the 32 units of the busiest one take at once."""
    cut = 0
    for layout, M, Nn, K in itertools.product((0, 1, 2), (130, 637, 1028, 2066, 3300), (136, 536, 1200, 2600), (2056, 3992, 9472, 13520)):
        c = N.ntp_gemm_choice(layout, M, Nn, K)
        if (c["tile_m"], c["tile_n"], c["wavefronts"]) == (128, 128, 8) and c["k_splits"] > 1:
            cut += 1
            assert -(-_tiles(c, M, Nn) // 8) * c["k_splits"] <= 32, (layout, M, Nn, K, c)
    assert cut > 30
    assert N.ntp_gemm_choice(0, 2066, 536, 3992)["k_splits"] == 2  # 85 tiles: three chunks would be 33 workgroups on five of the XCDs


def test_choice_rejects_bad_arguments():
    for args in [(3, 8, 8, 8), (-1, 8, 8, 8), (0, 0, 8, 8), (0, 8, 0, 8), (0, 8, 8, -1), (0, 1 << 31, 8, 8)]:
        with pytest.raises(N.NtpError):
            N.ntp_gemm_choice(*args)


def test_schedule_choice_and_override():
    """Every layout gets the ping-pong kernel on the 8-wavefront tiles other than 128 x 128; the option forces either."""
    h = Bd.ntp_create()
    c = Bd.ntp_gemm_choice(0, 2048, 7022, 12288, handle=h)
    assert c["persistent"] == 1 and c["pingpong"] == 1
    assert Bd.ntp_gemm_choice(1, 2048, 12288, 7022, handle=h)["pingpong"] == 1  # row-parallel layout
    assert Bd.ntp_gemm_choice(1, 8192, 16384, 750, handle=h)["pingpong"] == 1  # ... at short K
    c = Bd.ntp_gemm_choice(2, 7022, 12288, 2048, handle=h)  # weight gradients on the 224 x 256 tile
    assert (c["tile_m"], c["tile_n"], c["pingpong"]) == (224, 256, 1)
    c = Bd.ntp_gemm_choice(2, 1792, 12288, 2048, handle=h)  # ... on the 192 x 256 tile
    assert (c["tile_m"], c["tile_n"], c["pingpong"]) == (192, 256, 1)
    assert Bd.ntp_gemm_choice(0, 512, 586, 1024, handle=h)["pingpong"] == 0  # the small 128 x 128 tile is the deep-pipelined kernel's
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_SCHEDULE, 1, handle=h)
    assert Bd.ntp_gemm_choice(0, 2048, 7022, 12288, handle=h)["pingpong"] == 0
    assert Bd.ntp_gemm_choice(2, 5376, 12288, 2048, handle=h)["pingpong"] == 1  # the ring kernel has no 256 x 256 weight-gradient tile
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_SCHEDULE, 2, handle=h)
    assert Bd.ntp_gemm_choice(1, 2048, 12288, 7022, handle=h)["pingpong"] == 1
    assert Bd.ntp_gemm_choice(2, 5376, 12288, 2048, handle=h)["pingpong"] == 1  # 256 x 256 weight-gradient tile
    assert Bd.lib().ntp_set_option(h.ptr, Bd.NTP_OPT_GEMM_SCHEDULE, 3) == Bd.NTP_ERR_INVALID_ARG
    Bd.ntp_destroy(h)


def test_choice_says_where_the_pingpong_kernel_runs(workspace_1gib):
    pp = lambda *s: (lambda c: (c["k_splits"], c["persistent"], c["pingpong"]))(N.ntp_gemm_choice(*s))  # noqa: E731
    assert pp(0, 4096, 640, 8192) == (3, 0, 1)      # cut, on 256 x 128 tiles
    assert pp(2, 384, 512, 4096)[2] == 0            # few tiles: the deep-pipelined kernel
    assert pp(0, 8192, 8192, 128) == (1, 1, 0) and pp(0, 8192, 8192, 136) == (1, 1, 1)  # two K tiles: the ring kernel
    assert pp(0, 100, 100, 4096)[2] == 0            # the generic kernel
    h = Bd.default_handle()
    try:
        Bd.ntp_set_option(Bd.NTP_OPT_GEMM_NO_RING_TAIL, 1, handle=h)
        assert pp(1, 8192, 16384, 750) == (1, 1, 0) and pp(1, 8192, 16384, 768) == (1, 1, 1) and pp(0, 8192, 16384, 752) == (1, 1, 1)
    finally:
        Bd.ntp_set_option(Bd.NTP_OPT_GEMM_NO_RING_TAIL, 0, handle=h)


def test_weight_gradient_tile_that_the_ring_kernel_does_not_have():
    """256 x 256: persistent where workgroups have several tiles of three to 64 K tiles; otherwise, and under the ring schedule, one workgroup per output tile."""
    h = Bd.ntp_create()
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_TILE, "256x256", handle=h)
    one = lambda M, K: Bd.ntp_gemm_choice(2, M, 4096, K, handle=h)  # noqa: E731
    assert [one(4097, K)["persistent"] for K in (8, 64, 128, 129, 192, 4096, 4097)] == [0, 0, 0, 1, 1, 1, 0]  # 272 tiles
    assert one(4096, 2048)["persistent"] == 0  # 256
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_WORKGROUPS, 8, handle=h)
    assert one(4096, 2048)["persistent"] == one(257, 2048)["persistent"] == 1
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_SCHEDULE, 1, handle=h)
    assert one(4097, 2048)["persistent"] == 0 and one(4097, 2048)["tile_m"] == one(4097, 2048)["tile_n"] == 256
    Bd.ntp_destroy(h)


def test_options_of_the_ring_kernels_reach_them_at_few_tiles():
    """A cap on the persistent grid and a K tail through registers are about the ring kernels: problems with few tiles run on those then."""
    h = Bd.ntp_create()
    small, tail, whole = (0, 512, 586, 1024), (1, 777, 1096, 1001), (1, 777, 1096, 1024)
    assert not any(Bd.ntp_gemm_choice(*s, handle=h)["persistent"] for s in (small, tail, whole))
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_WORKGROUPS, 8, handle=h)
    assert all(Bd.ntp_gemm_choice(*s, handle=h)["persistent"] for s in (small, tail, whole))
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_WORKGROUPS, 0, handle=h)
    Bd.ntp_set_option(Bd.NTP_OPT_GEMM_NO_RING_TAIL, 1, handle=h)
    assert [Bd.ntp_gemm_choice(*s, handle=h)["persistent"] for s in (small, tail, whole)] == [0, 1, 0]
    Bd.ntp_destroy(h)
