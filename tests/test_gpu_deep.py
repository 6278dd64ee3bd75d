"""The deep-pipelined GEMM kernel (problems with few output tiles), whole and with a cut K axis, against the oracle: sizes at the edges of
tiles, of K tiles and of the ring's five stages, in the three operand layouts and with every epilogue."""
import sys

import numpy as np
import pytest

from tests.helpers import TOL, AttnCase, MlpCase, rel_err

pytestmark = pytest.mark.gpu
MLP_NAMES = ("P", "Y", "Z", "dP", "dX", "dA_t", "dB")


@pytest.fixture(params=[False, True], ids=["whole", "workspace"])
def names(request):
    import torch
    import paper_2504_06095_amd as N
    ws = torch.full((8 << 20,), float("nan"), dtype=torch.float32, device="cuda") if request.param else None
    N.ntp_set_workspace(ws)
    N.ntp_kernel_timing_enable(1)
    N.ntp_kernel_timing_read()
    yield lambda: [r["name"].split("_")[-1] for r in N.ntp_kernel_timing_read()]
    N.ntp_kernel_timing_enable(0)
    N.ntp_kernel_timing_read()
    N.ntp_set_workspace(None)


# every GEMM's K once below, at and above the five stages (320) and off the K tile; M and N around multiples of 128
@pytest.mark.parametrize("M,H,n_r", [(256, 256, 256), (257, 264, 129), (513, 328, 320), (320, 384, 255), (130, 1288, 383), (1025, 520, 641), (129, 2056, 513),
                                     (2048, 136, 257), (300, 4096, 131)])
@pytest.mark.parametrize("mode", [0, 1], ids=["erf", "tanh"])
def test_mlp_deep(names, M, H, n_r, mode):
    print(f"[gpu-case] deep GEMM MLP M={M} H={H} n_r={n_r} mode={mode}", file=sys.stderr, flush=True)
    case = MlpCase(M, H, n_r, 1, 0)
    got, raw = case.run_gpu(mode=mode, accumulate_twice=True)
    picked = names()
    assert any("128x128w8d" in n for n in picked), picked
    want = case.oracle(mode)
    want["dA_t"], want["dB"] = 2 * want["dA_t"], 2 * want["dB"]
    for k in MLP_NAMES:
        assert np.isfinite(got[k]).all(), k
        e = rel_err(got[k], want[k])
        assert e <= TOL, f"{k}: rel err {e:.3e}"
    pad = -(-n_r // 8) * 8
    for k in ("P", "Y", "dP"):
        assert (raw[k][:, n_r:pad].float().cpu().numpy() == 0).all(), k


# 16 chunks whose last one is shorter than the ring: one ragged K tile, two and three
@pytest.mark.parametrize("M,H,n_r,layout", [(257, 9640, 520, "nt"), (257, 520, 9640, "nn"), (257, 10648, 520, "nt"), (257, 520, 10705, "nn")])
def test_mlp_deep_short_last_chunk(M, H, n_r, layout):
    import torch
    import paper_2504_06095_amd as N
    print(f"[gpu-case] deep GEMM MLP, short last chunk M={M} H={H} n_r={n_r}", file=sys.stderr, flush=True)
    N.ntp_set_workspace(torch.full((8 << 20,), float("nan"), dtype=torch.float32, device="cuda"))
    N.ntp_kernel_timing_enable(1)
    N.ntp_kernel_timing_read()
    try:
        case = MlpCase(M, H, n_r, 1, 0)
        got, _ = case.run_gpu()
        picked = [r["name"] for r in N.ntp_kernel_timing_read()]
    finally:
        N.ntp_kernel_timing_enable(0)
        N.ntp_set_workspace(None)
    assert any(n.startswith(f"gemm_{layout}") and n.endswith("128x128w8dk16") for n in picked), picked
    want = case.oracle()
    for k in MLP_NAMES:
        e = rel_err(got[k], want[k])
        assert np.isfinite(got[k]).all() and e <= TOL, f"{k}: rel err {e:.3e}"


@pytest.mark.parametrize("M,H,n_q,n_kv,d,tp,rank", [(385, 520, 6, 2, 64, 2, 1), (129, 1544, 8, 4, 64, 3, 1), (700, 264, 4, 4, 128, 2, 0)])
def test_attn_proj_deep(names, M, H, n_q, n_kv, d, tp, rank):
    print(f"[gpu-case] deep GEMM attention projections M={M} H={H}", file=sys.stderr, flush=True)
    case = AttnCase(M, H, n_q, n_kv, d, tp, rank)
    got, want = case.run_gpu(), case.oracle()
    picked = names()
    assert any("128x128w8d" in n for n in picked), picked
    for k in got:
        e = rel_err(got[k], want[k])
        assert e <= TOL, f"{k}: rel err {e:.3e}"


# 64 x 64 tiles (where a workspace is set): M and N around multiples of 64, K at six K tiles and off them, cut and whole; the last two:
# gradients over more than 24 K tiles, in the shared launch
@pytest.mark.parametrize("M,H,n_r,group", [(65, 448, 513, False), (193, 1288, 450, False), (450, 1000, 385, False), (127, 4104, 383, False), (1601, 520, 193, True),
                                           (1999, 264, 449, True)])
def test_mlp_deep_small_tiles(M, H, n_r, group):
    import torch
    import paper_2504_06095_amd as N
    print(f"[gpu-case] deep GEMM MLP, 64 x 64 tiles M={M} H={H} n_r={n_r}", file=sys.stderr, flush=True)
    ws = torch.full((8 << 20,), float("nan"), dtype=torch.float32, device="cuda")
    N.ntp_set_workspace(ws)
    N.ntp_kernel_timing_enable(1)
    N.ntp_kernel_timing_read()
    try:
        case = MlpCase(M, H, n_r, 1, 0)
        got, raw = case.run_gpu(accumulate_twice=True)
        picked = [r["name"] for r in N.ntp_kernel_timing_read()]
    finally:
        N.ntp_kernel_timing_enable(0)
        N.ntp_set_workspace(None)
    assert any("64x64d" in n for n in picked if "group" not in n) and ("gemm_group_64x64d" in picked) == group, picked
    want = case.oracle()
    want["dA_t"], want["dB"] = 2 * want["dA_t"], 2 * want["dB"]
    for k in MLP_NAMES:
        e = rel_err(got[k], want[k])
        assert np.isfinite(got[k]).all() and e <= TOL, f"{k}: rel err {e:.3e}"
    pad = -(-n_r // 8) * 8
    for k in ("P", "Y", "dP"):
        assert (raw[k][:, n_r:pad].float().cpu().numpy() == 0).all(), k


# the two gradient groups of the projections (dC and dWo, dX and dWqkv): 64 x 64 tiles shared where all workgroups are on the device at once, and
# not where they make the longest walks wait or rows of a K-contiguous operand do not start on cache lines
@pytest.mark.parametrize("M,H,n_q,n_kv,d,groups", [(2168, 584, 3, 1, 64, 2), (3792, 568, 6, 1, 128, 1), (4667, 1640, 4, 2, 128, 0)])
def test_attn_gradient_groups_small_tiles(M, H, n_q, n_kv, d, groups):
    import torch
    import paper_2504_06095_amd as N
    print(f"[gpu-case] deep GEMM gradient groups M={M} H={H}", file=sys.stderr, flush=True)
    N.ntp_set_workspace(torch.full((16 << 20,), float("nan"), dtype=torch.float32, device="cuda"))
    N.ntp_kernel_timing_enable(1)
    N.ntp_kernel_timing_read()
    try:
        case = AttnCase(M, H, n_q, n_kv, d, 1, 0)
        got = case.run_gpu()
        picked = [r["name"] for r in N.ntp_kernel_timing_read()]
    finally:
        N.ntp_kernel_timing_enable(0)
        N.ntp_set_workspace(None)
    assert picked.count("gemm_group_64x64d") == groups, picked
    want = case.oracle()
    for k in got:
        e = rel_err(got[k], want[k])
        assert np.isfinite(got[k]).all() and e <= TOL, f"{k}: rel err {e:.3e}"


# the forms above one tile per compute unit: two K tiles in LDS ("d2"), and 128 x 256 tiles with three
@pytest.mark.parametrize("M,H,n_r,form", [(129, 8200, 1090, "128x128w8d2"), (130, 4104, 2000, "128x128w8d2"), (2900, 1032, 1501, "128x128w8d2"),
                                          (1290, 1288, 3300, "128x256d"), (577, 1000, 9001, "128x128w8d2")])
def test_mlp_deep_more_tiles(M, H, n_r, form):
    import paper_2504_06095_amd as N
    print(f"[gpu-case] deep GEMM MLP, more tiles M={M} H={H} n_r={n_r}", file=sys.stderr, flush=True)
    N.ntp_kernel_timing_enable(1)
    N.ntp_kernel_timing_read()
    case = MlpCase(M, H, n_r, 1, 0)
    got, _ = case.run_gpu(accumulate_twice=True)
    picked = [r["name"].split("_")[-1] for r in N.ntp_kernel_timing_read()]
    N.ntp_kernel_timing_enable(0)
    assert form in picked, picked
    want = case.oracle()
    want["dA_t"], want["dB"] = 2 * want["dA_t"], 2 * want["dB"]
    for k in MLP_NAMES:
        e = rel_err(got[k], want[k])
        assert np.isfinite(got[k]).all() and e <= TOL, f"{k}: rel err {e:.3e}"


def test_deep_matches_the_other_kernels_bit_for_bit(opts):
    """Without a cut K axis both kernels add in the same order; the three gradient GEMMs of the backward call share a launch."""
    import paper_2504_06095_amd as N
    from paper_2504_06095_amd import binding as K
    print("[gpu-case] deep GEMM against the ring kernel", file=sys.stderr, flush=True)
    for M, H, n_r in ((512, 1024, 586), (640, 776, 1000), (258, 264, 257), (640, 1288, 1320)):
        case = MlpCase(M, H, n_r, 1, 0)
        N.ntp_kernel_timing_enable(1)
        N.ntp_kernel_timing_read()
        a, _ = case.run_gpu(pad_to=64)
        picked = [r["name"] for r in N.ntp_kernel_timing_read()]
        N.ntp_kernel_timing_enable(0)
        assert "gemm_group_128x128w8d" in picked and len(picked) == 4, picked
        opts(K.NTP_OPT_GEMM_SCHEDULE, 1)
        b, _ = case.run_gpu(pad_to=64)
        opts(K.NTP_OPT_GEMM_SCHEDULE, 0)
        for k in MLP_NAMES:
            assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("M,H,n_r", [(1000, 1288, 4000), (1040, 2056, 1300), (200, 4104, 3000), (4096, 3080, 1800)])
def test_accumulating_epilogue_adds_exactly_once(M, H, n_r):
    """Accumulating into a buffer gives, bit for bit, the buffer plus the overwriting call's result: same products, one fp32 addition."""
    import torch
    import paper_2504_06095_amd as N
    print(f"[gpu-case] accumulating epilogue M={M} H={H} n_r={n_r}", file=sys.stderr, flush=True)
    g = torch.Generator("cuda").manual_seed(1)
    mk = lambda r, c: torch.empty(r, c, device="cuda").normal_(generator=g).bfloat16()  # noqa: E731
    ld = -(-n_r // 8) * 8
    dZ, X, At, B, P, Y = mk(M, H), mk(M, H), mk(n_r, H), mk(n_r, H), mk(M, ld)[:, :n_r], mk(M, ld)[:, :n_r]
    dP, dX = torch.empty(M, ld, dtype=torch.bfloat16, device="cuda")[:, :n_r], torch.empty_like(X)
    plain = [torch.full((n_r, H + 4), 7.0, device="cuda")[:, :H] for _ in range(2)]
    start = [torch.empty(n_r, H + 4, device="cuda").normal_(generator=g) for _ in range(2)]
    acc = [t.clone() for t in start]
    N.ntp_mlp_shard_bwd(dZ, X, At, B, P, Y, dP, dX, *plain, n_r)
    N.ntp_mlp_shard_bwd(dZ, X, At, B, P, Y, dP, dX, *[t[:, :H] for t in acc], n_r, accumulate=True)
    torch.cuda.synchronize()
    for s, p, a in zip(start, plain, acc):
        assert torch.equal(a[:, :H], s[:, :H] + p) and torch.equal(a[:, H:], s[:, H:])
