"""Ragged K in the ping-pong GEMM kernel, whose ring runs on from one output tile into the next: K tails as a K tile of their own with several output tiles
per workgroup, and K chunks of one and two K tiles in its non-persistent form, for tile shapes whose long operand is A or B.  On a real MI355X."""
import sys

import numpy as np
import pytest

from paper_2504_06095_amd import binding as K
from tests.helpers import TOL, MlpCase, rel_err
from tests.test_gpu_split_k import workspace  # noqa: F401  (poisoned workspace, kernel names recorded)

pytestmark = pytest.mark.gpu
TILES = ["256x256", "224x256", "256x192", "192x256", "128x256"]


def _check(case, pad_to, tag):
    print(f"[gpu-case] {tag}", file=sys.stderr, flush=True)
    got, _ = case.run_gpu(pad_to=pad_to)
    want = case.oracle()
    for k in ("P", "Y", "Z", "dP", "dX", "dA_t", "dB"):
        assert np.isfinite(got[k]).all(), f"{tag}: {k} not finite"
        assert rel_err(got[k], want[k]) <= TOL, f"{tag}: {k} {rel_err(got[k], want[k]):.3e}"


@pytest.mark.parametrize("k", [131, 200, 321])  # 3, 4 and 6 K tiles: as short as the persistent form takes, one more, and past the ring's length
@pytest.mark.parametrize("tile", TILES)
def test_k_tail_with_many_output_tiles_per_workgroup(workspace, opts, tile, k):  # noqa: F811
    import paper_2504_06095_amd as N
    opts(K.NTP_OPT_GEMM_SCHEDULE, 2)
    opts(K.NTP_OPT_GEMM_TILE, tile)
    opts(K.NTP_OPT_GEMM_WORKGROUPS, 8)
    opts(K.NTP_OPT_GEMM_SPLIT, 1)

    def check(case, pad_to, tag):
        N.ntp_kernel_timing_read()
        _check(case, pad_to, f"{tile}, {tag}")
        names = [r["name"] for r in N.ntp_kernel_timing_read()]
        assert len(names) == 6 and all(n.endswith(f"{tile}pp") for n in names), names

    for pad_to in (8, 64):  # K = n_r, whose rows end right behind it or at the next K tile
        check(MlpCase(1300, 1400, k, 1, 0, tag=f"ppt.n.{k}"), pad_to, f"K = n_r = {k}, rows padded to {pad_to}")
    h = (k + 7) // 8 * 8
    check(MlpCase(1300, h, 1403, 1, 0, tag=f"ppt.h.{k}"), 8, f"K = H = {h}")
    check(MlpCase(k, 1400, 1403, 1, 0, tag=f"ppt.m.{k}"), 8, f"K = tokens = {k}")


@pytest.mark.parametrize("k,splits", [(488, 8), (987, 8), (1272, 7)])  # chunks of 1, 2 and 3 K tiles, the last one ragged
@pytest.mark.parametrize("tile", ["256x256", "192x256", "256x128"])
def test_short_ragged_k_chunks(workspace, opts, tile, k, splits):  # noqa: F811
    import paper_2504_06095_amd as N
    opts(K.NTP_OPT_GEMM_TILE, tile)
    opts(K.NTP_OPT_GEMM_SPLIT, splits)
    h = (k + 7) // 8 * 8
    for case, tag in ((MlpCase(700, 704, k, 1, 0, tag=f"pps.n.{k}"), "n_r"), (MlpCase(700, h, 705, 1, 0, tag=f"pps.h.{k}"), "H"),
                      (MlpCase(k, 704, 705, 1, 0, tag=f"pps.m.{k}"), "tokens")):
        N.ntp_kernel_timing_read()
        _check(case, 8, f"{tile}, {splits} chunks of K = {tag} = {k}")
        assert any(r["name"].endswith(f"{tile}k{splits}") for r in N.ntp_kernel_timing_read()), tag


def _projections(M, H, w, X, Cc, W, handle=None):
    """QKV = X W^T, Z = C W and dW = C^T dZ of one shard, and the names of the kernels."""
    import torch
    import paper_2504_06095_amd as N
    QKV, Z = torch.zeros(M, w, dtype=torch.bfloat16, device="cuda"), torch.zeros(M, H, dtype=torch.bfloat16, device="cuda")
    dC, dW = torch.zeros_like(QKV), torch.zeros(w, H, device="cuda")
    N.ntp_kernel_timing_read()
    N.ntp_attn_proj_shard_fwd(M, H, w, w, X=X, Wqkv=W, QKV=QKV, C_=Cc, Wo=W, Zpart=Z)
    N.ntp_attn_proj_shard_bwd(M, H, w, w, dZ=X, C_=Cc, Wo=W, dC=dC, dWo=dW)
    return (QKV, Z, dC, dW), [r["name"] for r in N.ntp_kernel_timing_read()]


def test_ragged_k_of_operands_past_2_gib_is_cut(workspace, opts):  # noqa: F811
    """A K-contiguous operand of more than 2 GiB (by its row length) and a ragged K, in three chunks: the bits of the same call on compact operands."""
    import torch
    print("[gpu-case] three ragged K chunks, operands past 2 GiB", file=sys.stderr, flush=True)
    M, H, w, ld = 700, 1000, 712, 1600000
    opts(K.NTP_OPT_GEMM_SPLIT, 3)
    g = torch.Generator("cuda").manual_seed(3)
    X, Cc, W = (torch.empty(r, c, device="cuda").normal_(generator=g).bfloat16() for r, c in ((M, H), (M, w), (w, H)))
    far = torch.full((M, ld), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert M * ld * 2 > 2 << 30
    far[:, :H], far[:, H:H + w] = X, Cc
    want, names = _projections(M, H, w, X, Cc, W)
    assert len(names) == 4 and all(n.split("_")[-1].split("x")[1].endswith("k3") for n in names), names
    got, names = _projections(M, H, w, far[:, :H], far[:, H:H + w], W)
    assert len(names) == 4 and all(n.split("_")[-1].split("x")[1].endswith("k3") for n in names), names
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_k_tail_option_leaves_cut_axes_alone(workspace, opts):  # noqa: F811
    """NTP_OPT_GEMM_NO_RING_TAIL is about persistent launches: a ragged row-parallel K is cut under it as without it."""
    opts(K.NTP_OPT_GEMM_SPLIT, 3)
    opts(K.NTP_OPT_GEMM_NO_RING_TAIL, 1)
    import paper_2504_06095_amd as N
    N.ntp_kernel_timing_read()
    _check(MlpCase(700, 704, 987, 1, 0, tag="ppo"), 64, "three chunks, K tails through registers asked for")
    names = [r["name"] for r in N.ntp_kernel_timing_read()]
    assert len(names) == 6 and all(n.endswith("k3") for n in names), names
