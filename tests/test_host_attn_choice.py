"""Host logic of the attention core launcher (no GPU): rows per wavefront and how many parts the walks are cut into."""
import math
import random

import pytest

import paper_2504_06095_amd as N
from paper_2504_06095_amd import binding as Bd

FAKE_WS = 0x10000000  # an aligned address: registering touches no memory


def _shape(n_q, n_kv, tp, rank, n_seq, S, causal, d=128):
    plan = N.ntp_attn_shard_plan(n_q, n_kv, d, tp, rank)
    return N.attn_core_shape(n_seq, S, plan, n_q // n_kv, causal)


@pytest.fixture
def workspace_1gib():
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS, 1 << 30) == 0
    yield
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0


def test_nothing_is_cut_without_a_workspace():
    for args in [(64, 8, 30, 0, 1, 4096, True), (96, 8, 7, 0, 1, 2048, False), (16, 16, 1, 0, 2, 8192, True)]:
        c = N.ntp_attn_core_choice(_shape(*args))
        assert (c["fwd_parts"], c["dq_parts"], c["dkv_parts"]) == (1, 1, 1)
        assert c["fwd_rows_per_wavefront"] in (16, 32)


def test_few_heads_get_cut_walks(workspace_1gib):
    # config 3, rank 0: 3 query heads on 1 KV head, one causal sequence of 4096 tokens (64 tiles, taken in 32 pairs):
    # 96 forward / dQ workgroups with walks of 65 tiles and 32 dK/dV workgroups with walks of 195.  The forward launch is
    # cut towards two workgroups per compute unit, the two backward kernels (one launch) towards one each
    c = N.ntp_attn_core_choice(_shape(64, 8, 30, 0, 1, 4096, True))
    assert c == dict(fwd_rows_per_wavefront=16, fwd_parts=4, dq_parts=2, dkv_parts=8)
    # the same heads without the mask: 192 and 64 workgroups with walks of 64 and 192 tiles
    c = N.ntp_attn_core_choice(_shape(64, 8, 30, 0, 1, 4096, False))
    assert c == dict(fwd_rows_per_wavefront=16, fwd_parts=2, dq_parts=1, dkv_parts=4)
    # ... and at 8192 tokens (384 and 128 workgroups)
    c = N.ntp_attn_core_choice(_shape(64, 8, 30, 0, 1, 8192, False))
    assert (c["fwd_parts"], c["dq_parts"], c["dkv_parts"]) == (1, 1, 2)
    # many heads and tokens: nothing to gain, and the forward kernel takes 32 rows per wavefront
    c = N.ntp_attn_core_choice(_shape(16, 16, 1, 0, 2, 8192, False))
    assert c == dict(fwd_rows_per_wavefront=32, fwd_parts=1, dq_parts=1, dkv_parts=1)


def test_launches_that_fill_the_device_stay_whole(workspace_1gib):
    # 14 heads x 2048 tokens: 448 forward workgroups of 32 tiles each, or 224 of 33 with the causal pairs: parts of 16
    # tiles would not pay; grouped KV heads leave 64 (32) dK/dV workgroups with walks of 7 heads' tiles
    causal = N.ntp_attn_core_choice(_shape(96, 8, 7, 0, 1, 2048, True))
    full = N.ntp_attn_core_choice(_shape(96, 8, 7, 0, 1, 2048, False))
    assert (causal["fwd_parts"], causal["dq_parts"]) == (1, 1)
    assert (full["fwd_parts"], full["dq_parts"]) == (1, 1)
    assert (causal["dkv_parts"], full["dkv_parts"]) == (8, 4)


def test_step_shape_keeps_whole_walks_with_the_dma_kernels(workspace_1gib):
    # 14 query and 14 KV heads x 2048 tokens, causal: 224 workgroups of 33 tiles in all three launches
    c = N.ntp_attn_core_choice(_shape(96, 96, 7, 0, 1, 2048, True))
    assert c == dict(fwd_rows_per_wavefront=16, fwd_parts=1, dq_parts=1, dkv_parts=1)


def test_register_copy_kernels_keep_their_own_rule(workspace_1gib):
    N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, 1)
    try:
        c = N.ntp_attn_core_choice(_shape(96, 96, 7, 0, 1, 2048, True))
        assert c == dict(fwd_rows_per_wavefront=16, fwd_parts=2, dq_parts=2, dkv_parts=2)
        c = N.ntp_attn_core_choice(_shape(64, 8, 30, 0, 1, 4096, True))
        assert c == dict(fwd_rows_per_wavefront=16, fwd_parts=5, dq_parts=5, dkv_parts=16)
    finally:
        N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, 0)


def test_short_walks_are_not_cut(workspace_1gib):
    c = N.ntp_attn_core_choice(_shape(8, 2, 3, 0, 1, 200, True))  # 4 key tiles
    assert (c["fwd_parts"], c["dq_parts"]) == (1, 1)


def test_small_launches_share_out_walks_inside_workgroups(workspace_1gib):
    """Walks that would be cut into parts where the launch is small enough for 16 rows per workgroup, and the sizes from which they are."""
    parts = lambda *a, **k: (lambda c: (c["fwd_parts"], c["dq_parts"], c["dkv_parts"]))(N.ntp_attn_core_choice(_shape(*a, **k)))  # noqa: E731
    assert parts(4, 1, 1, 0, 1, 512, True, d=64) == parts(3, 3, 1, 0, 1, 1432, False, d=64) == (1, 1, 1)
    assert parts(1, 1, 1, 0, 1, 1432, True) == (1, 1, 1)
    N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, 2)
    try:
        assert max(parts(4, 1, 1, 0, 1, 512, True, d=64)) > 1 and max(parts(1, 1, 1, 0, 1, 1432, True)) > 1
    finally:
        N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, 0)
    assert max(parts(4, 4, 1, 0, 1, 8192, True, d=64)) > 1 and max(parts(2, 1, 1, 0, 1, 4096, False)) > 1


@pytest.mark.parametrize("d,S", [(64, 1432), (128, 1432)])
def test_backward_launch_option_leaves_the_forward_call_alone(workspace_1gib, d, S):
    s, got = _shape(2, 1, 1, 0, 1, S, True, d=d), []
    for launches in (0, 1, 2):
        N.ntp_set_option(Bd.NTP_OPT_ATTN_BWD_LAUNCHES, launches)
        try:
            c = N.ntp_attn_core_choice(s)
        finally:
            N.ntp_set_option(Bd.NTP_OPT_ATTN_BWD_LAUNCHES, 0)
        got.append((c["fwd_rows_per_wavefront"], c["fwd_parts"]))
    assert got == [(16, 1)] * 3  # (two heads' walks would be cut on the other kernels)


# heads, KV heads, sequences, tokens, causal, rows of the backward kernels without and with a workspace (256 compute units): either side of
# each line of the rule, at shapes that were measured with both kernels
BWD_ROWS = [
    # (128 x 64) tile pairs per unit, whole walks and cut ones
    (16, 16, 1, 1024, 0, 32, 32), (16, 16, 1, 1024, 1, 16, 16), (12, 3, 1, 1700, 0, 32, 32), (12, 3, 1, 1700, 1, 32, 16),
    (16, 2, 1, 2048, 1, 32, 16), (56, 7, 2, 831, 1, 32, 32), (8, 1, 1, 4096, 1, 32, 32), (32, 1, 1, 2048, 0, 32, 32), (3, 1, 1, 4096, 1, 16, 16),
    # length of the walks: short sequences, many of them
    (14, 14, 150, 33, 0, 16, 16), (14, 14, 439, 64, 1, 16, 16), (14, 14, 75, 128, 0, 16, 16), (14, 14, 55, 256, 0, 16, 16), (14, 14, 25, 384, 0, 16, 16),
    (14, 14, 5, 512, 0, 32, 32), (14, 14, 22, 512, 1, 16, 16), (14, 14, 4, 768, 1, 32, 32), (7, 7, 16, 774, 1, 16, 16), (14, 14, 7, 768, 0, 32, 32), (18, 18, 2, 1024, 1, 32, 32),
    (16, 8, 16, 743, 1, 16, 16), (16, 16, 16, 462, 0, 16, 16), (16, 16, 8, 1267, 1, 32, 32), (64, 8, 8, 256, 1, 32, 16), (16, 2, 96, 128, 0, 16, 16),
    # workgroups per unit
    (4, 4, 1, 2048, 0, 16, 16), (2, 2, 1, 4096, 0, 16, 32), (1, 1, 1, 8192, 0, 16, 32), (4, 4, 1, 4096, 0, 32, 32), (3, 1, 1, 4096, 0, 16, 32),
    # full rounds of the 16-row kernels under the mask
    (10, 10, 1, 2048, 1, 32, 32), (14, 14, 1, 2048, 1, 16, 16), (16, 16, 1, 1999, 1, 16, 16), (2, 2, 8, 2113, 1, 32, 32), (8, 8, 4, 2023, 1, 16, 16),
    (14, 14, 1, 4096, 1, 32, 32), (14, 14, 1, 8192, 0, 32, 32), (14, 14, 1, 8192, 1, 32, 32)]


@pytest.mark.parametrize("ws", [False, True], ids=["no_workspace", "workspace"])
def test_rows_of_the_backward_kernels(ws):
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS if ws else None, 1 << 30 if ws else 0) == 0
    try:
        got = [(*c[:5], N.ntp_attn_core_bwd_rows(_shape(c[0], c[1], 1, 0, *c[2:5]))) for c in BWD_ROWS]
    finally:
        assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0
    assert got == [(*c[:5], c[6 if ws else 5]) for c in BWD_ROWS]


# the same at head dimension 64 (no workspace): causal and not, one and several query heads per KV head, sequences that 128 divides and others
@pytest.mark.parametrize("n_q,n_kv,n_seq,S,causal,rows", [
    (5, 5, 2, 3702, 1, 32), (3, 3, 8, 1294, 1, 16), (9, 9, 1, 4095, 1, 32), (12, 12, 4, 2048, 1, 32), (5, 5, 8, 2350, 1, 16), (8, 8, 8, 1371, 1, 16), (14, 14, 4, 1747, 1, 32),
    (11, 11, 4, 1600, 1, 16), (24, 3, 8, 1609, 1, 16), (14, 7, 4, 1536, 1, 16), (24, 3, 8, 1900, 1, 32), (56, 7, 4, 4096, 1, 32),
    (4, 4, 2, 2816, 0, 32), (5, 5, 1, 4244, 0, 16), (8, 8, 2, 1660, 0, 32), (4, 4, 2, 5823, 0, 16), (4, 4, 4, 3580, 0, 32),
    (16, 4, 4, 2048, 0, 32), (16, 4, 4, 2047, 0, 16), (8, 4, 1, 8028, 0, 16), (16, 4, 4, 3300, 0, 32), (16, 4, 4, 3072, 0, 16)])
def test_rows_of_the_backward_kernels_at_head_dimension_64(n_q, n_kv, n_seq, S, causal, rows):
    assert N.ntp_attn_core_bwd_rows(_shape(n_q, n_kv, 1, 0, n_seq, S, causal, d=64)) == rows


def test_rows_of_the_backward_kernels_by_option_and_head_dimension():
    long, short = _shape(14, 14, 1, 0, 1, 8192, False), _shape(14, 14, 1, 0, 1, 64, False)
    for copy, want in ((0, (32, 16)), (1, (16, 16)), (2, (16, 16)), (3, (32, 32))):
        N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, copy)
        try:
            assert (N.ntp_attn_core_bwd_rows(long), N.ntp_attn_core_bwd_rows(short)) == want
        finally:
            N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, 0)
    for copy, want in ((0, (32, 16)), (1, (16, 16)), (2, (16, 16)), (3, (32, 32))):  # (head dimension 64: where the launch is shared)
        N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, copy)
        try:
            assert tuple(N.ntp_attn_core_bwd_rows(_shape(14, 14, 1, 0, 1, S, False, d=64)) for S in (8192, 64)) == want
            N.ntp_set_option(Bd.NTP_OPT_ATTN_BWD_LAUNCHES, 1)
            assert N.ntp_attn_core_bwd_rows(_shape(14, 14, 1, 0, 1, 8192, False, d=64)) == 16
        finally:
            N.ntp_set_option(Bd.NTP_OPT_ATTN_COPY, 0)
            N.ntp_set_option(Bd.NTP_OPT_ATTN_BWD_LAUNCHES, 0)
    assert N.ntp_attn_core_bwd_rows(_shape(14, 14, 1, 0, 0, 8192, False)) == 16


def test_a_workspace_of_the_size_asked_for_gives_the_choice_of_an_unlimited_one():
    for c in BWD_ROWS:
        s = _shape(c[0], c[1], 1, 0, *c[2:5])
        n, got = N.ntp_workspace_bytes(Bd.NTP_CALL_ATTN_CORE_SHARD, s), []
        for size in (n, 1 << 40):
            assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS if size else None, size) == 0
            got.append((N.ntp_attn_core_bwd_rows(s), N.ntp_attn_core_choice(s)))
        assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0
        assert got[0] == got[1], c


def test_a_workspace_of_the_size_asked_for_gives_the_choice_of_an_unlimited_one_over_sizes():
    rng = random.Random(1)
    for _ in range(4000):
        kv = rng.randint(1, 14)
        c = (kv * rng.choice((1, 1, 2, 4, 8)), kv, rng.choice((1, 1, 2, 4, 8)), round(math.exp(rng.uniform(math.log(16), math.log(9000)))), rng.random() < 0.5, rng.choice((64, 128)))
        s = _shape(c[0], c[1], 1, 0, *c[2:5], d=c[5])
        n, got = N.ntp_workspace_bytes(Bd.NTP_CALL_ATTN_CORE_SHARD, s), []
        for size in (n, 1 << 40):
            assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS if size else None, size) == 0
            got.append((N.ntp_attn_core_bwd_rows(s), N.ntp_attn_core_choice(s)))
        assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0
        assert got[0] == got[1], c


def test_parts_respect_the_workspace_size():
    assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, FAKE_WS, 16 << 20) == 0  # 16 MiB
    try:
        c = N.ntp_attn_core_choice(_shape(64, 8, 30, 0, 1, 4096, True))
        # per part: forward 192 workgroups x 64 rows x 132 floats = 6.5 MB, dQ 192 x 64 x 128 floats = 6.3 MB,
        # dK/dV 64 workgroups x 64 rows x 256 floats = 4 MiB
        assert (c["fwd_parts"], c["dq_parts"], c["dkv_parts"]) == (2, 2, 4)
    finally:
        assert Bd.lib().ntp_set_workspace(Bd.default_handle().ptr, None, 0) == 0


@pytest.mark.parametrize("n_q,n_kv,n_seq,S,cut", [(8, 8, 1, 6720, False), (5, 5, 2, 3702, False),  # 128-row workgroups for 0.84 and 0.59 of the units
                                                  (7, 7, 1, 4194, True), (16, 4, 1, 3444, True)])  # 0.46; grouped, 0.22
def test_head_dimension_64_walks_in_one_piece(workspace_1gib, n_q, n_kv, n_seq, S, cut):
    c = N.ntp_attn_core_choice(_shape(n_q, n_kv, 1, 0, n_seq, S, True, d=64))
    assert (c["dq_parts"] > 1, c["dkv_parts"] > 1) == (cut, cut)


def test_choice_rejects_bad_shapes():
    s = _shape(8, 2, 3, 0, 1, 200, True, d=128)
    s.head_dim = 96
    with pytest.raises(N.NtpError):
        N.ntp_attn_core_choice(s)
