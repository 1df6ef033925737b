"""The expert GEMMs at the edges of their launches, in every weight format, against the float64
oracle: reductions with a partial last step (and shorter than one step), under one- and
two-tile gate/up launches and narrow and wide down launches, and the launches of large batches
at every count of token tiles, with experts in several slots, shared experts and GPU groups."""
import pytest
import torch

import test_gpu_ffn
import test_gpu_fp8
import test_gpu_mxfp4

pytestmark = pytest.mark.gpu
RUN = {"bf16": test_gpu_ffn._run, "fp8": test_gpu_fp8._run, "mxfp4": test_gpu_mxfp4._run}
FORMATS = pytest.mark.parametrize("fmt", list(RUN))


def _case(fmt, T, N, k, d, f, M, label):
    RUN[fmt](dict(N=N, k=k, d=d, f=f, T=T, logits="domains", Q=3), 5, 1, M,
             label=f"{label} {fmt} T{T} N{N} d{d} f{f} M{M}")


# the steps are 64, 128 or 256 elements: every count of 32-element groups in a partial step,
# alone (d or f below one step) and after whole ones
@FORMATS
@pytest.mark.parametrize("d,f", [(32, 32), (64, 96), (96, 224), (160, 192), (224, 288),
                                 (288, 320), (352, 480), (544, 160), (480, 416)])
def test_partial_steps(fmt, d, f):
    for T, N, k, M in [(5, 6, 2, 3), (41, 5, 2, 3)]:      # 1-8 rows an expert; up to 41
        _case(fmt, T, N, k, d, f, M, "partial step")


# grids of at least 768 blocks: two column tiles per gate/up wave, wide down waves
@FORMATS
def test_partial_steps_wide_launches(fmt):
    _case(fmt, 40, 120, 16, 288, 928, 110, "two tiles")
    _case(fmt, 40, 120, 16, 1760, 160, 110, "wide down")


# few small experts with a few rows each: the waves of a gate/up block split d (in 64 to 576
# elements a wave, whole steps and partial ones)
@FORMATS
@pytest.mark.parametrize("T,N,k,d,f,M", [(1, 16, 4, 256, 96, 4), (6, 24, 2, 512, 32, 12),
                                         (16, 40, 2, 1280, 160, 16), (2, 12, 8, 768, 224, 12),
                                         (9, 20, 1, 2304, 64, 9)])
def test_waves_split_d(fmt, T, N, k, d, f, M):
    _case(fmt, T, N, k, d, f, M, "waves split d")


# two experts hold every token: T rows each (past 128 in slots of nearly equal size), for each
# count of token tiles; d and f around the large-batch launches' steps and pairs of steps
@FORMATS
@pytest.mark.parametrize("T,d,f", [(33, 32, 96), (48, 64, 160), (64, 96, 32), (65, 160, 288),
                                   (96, 128, 128), (97, 224, 416), (128, 256, 544),
                                   (129, 288, 192), (300, 544, 352), (1000, 160, 96)])
def test_large_batch_tiles(fmt, T, d, f):
    _case(fmt, T, 2, 2, d, f, 2, "tiles")


# experts of 1 to 128 rows side by side; 256 weight rows a gate/up block (2048 blocks and more)
@FORMATS
def test_large_batch_uneven_experts(fmt):
    _case(fmt, 130, 64, 16, 160, 4128, 60, "uneven")
    _case(fmt, 400, 12, 2, 608, 224, 12, "uneven")


@pytest.mark.parametrize("T", [40, 129, 260])
def test_large_batch_shared_experts(T):
    import workloads as W
    from helpers import DEV, OracleOutputs, assert_ffn_close, bf16_weights_of, make_layer, say
    from oracle import ffn as OF
    from paper_2602_07265_amd import xshare as X
    c = dict(N=6, k=3, d=224, f=160, T=T, logits="domains", Q=2)
    h, _, x, w1, w3, w2 = make_layer(c, 1)
    sh = W.expert_weights(2, c["d"], c["f"], 9, DEV)
    say(f"large batch shared experts T={T}")
    res = X.moe_forward(x, torch.from_numpy(h).to(DEV), w1, w3, w2, 3, 1, 6, shared=sh)
    torch.cuda.synchronize()
    bits = [tuple(W.bf16_bits(m[s]) for m in sh) for s in range(2)]
    ref = OracleOutputs(x, bf16_weights_of(w1, w3, w2), bits).y(res["ids"].cpu().numpy(),
                                                               res["w"].cpu().numpy())
    assert_ffn_close(OF.bf16_to_f64(W.bf16_bits(res["y"])), ref, f"shared T{T}")


@pytest.mark.parametrize("fmt", ["fp8", "mxfp4"])
def test_large_batch_group_share(fmt):
    RUN[fmt](dict(N=32, k=4, d=288, f=224, T=260, logits="domains", Q=5), 3, 1, 4, "per_group",
             groups=4, local=2, label=f"group share {fmt}")


# every staged partial-step instance, after whole steps and alone, with 1 to 32 rows an expert
# (batches of up to 32 tokens never take the large-batch launches)
PARTIAL_DIMS = [(160, 288), (288, 160), (352, 480), (416, 352), (544, 608), (1056, 224)]
PARTIAL_ROWS = [(9, 4, 2, 2), (16, 4, 2, 3), (24, 5, 2, 4), (32, 4, 2, 2)]     # T, N, k, M


@FORMATS
@pytest.mark.parametrize("d,f", PARTIAL_DIMS)
def test_partial_steps_by_rows(fmt, d, f):
    for T, N, k, M in PARTIAL_ROWS:
        _case(fmt, T, N, k, d, f, M, "partial step rows")


# one expert with more rows than a staged pass holds (32) in a batch whose others hold few, so that
# it stays on the staged launches: a block takes its rows in two passes
TWO_PASS_DIMS = [(352, 480), (384, 256), (544, 224), (512, 512)]
TWO_PASS = dict(T=60, N=24, k=2, M=16)


@FORMATS
@pytest.mark.parametrize("d,f", TWO_PASS_DIMS)
def test_two_staged_passes(fmt, d, f):
    import numpy as np
    import workloads as W
    from helpers import oracle_route
    cfg = dict(N=TWO_PASS["N"], k=TWO_PASS["k"], d=d, f=f, T=TWO_PASS["T"], logits="domains", Q=1)
    ids = oracle_route(W.make_logits(cfg, 5)[0], cfg["k"], 1, TWO_PASS["M"]).ids
    assert np.bincount(ids.ravel()).max() > 32
    RUN[fmt](cfg, 5, 1, TWO_PASS["M"], label=f"two passes {fmt} d{d} f{f}")
