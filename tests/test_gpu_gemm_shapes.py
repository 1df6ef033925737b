"""The expert GEMMs at the edges of their launches, in every weight format, against the float64
oracle: reductions with a partial last step (and shorter than one step), under one- and
two-tile gate/up launches and narrow and wide down launches, and the launches of large batches
at every count of token tiles, with experts in several slots, shared experts and GPU groups."""
import numpy as np
import pytest
import torch

import test_gpu_ffn
import test_gpu_fp8
import test_gpu_mxfp4
import workloads as W
from helpers import oracle_route

pytestmark = pytest.mark.gpu
RUN = {"bf16": test_gpu_ffn._run, "fp8": test_gpu_fp8._run, "mxfp4": test_gpu_mxfp4._run}
FORMATS = pytest.mark.parametrize("fmt", list(RUN))


def _case(fmt, T, N, k, d, f, M, label, Q=3):
    RUN[fmt](dict(N=N, k=k, d=d, f=f, T=T, logits="domains", Q=Q), 5, 1, M,
             label=f"{label} {fmt} T{T} N{N} d{d} f{f} M{M}")


# the steps are 64, 128 or 256 elements: every count of 32-element groups in a partial step,
# alone (d or f below one step) and after whole ones
@FORMATS
@pytest.mark.parametrize("d,f", [(32, 32), (64, 96), (96, 224), (160, 192), (224, 288),
                                 (288, 320), (352, 480), (544, 160), (480, 416)])
def test_partial_steps(fmt, d, f):
    # (the second batch runs the large-batch launches; test_partial_steps_by_rows has the staged
    # ones with more rows)
    for T, N, k, M in [(5, 6, 2, 3), (41, 5, 2, 3)]:      # 1-8 rows an expert; up to 41
        _case(fmt, T, N, k, d, f, M, "partial step")


# grids of at least 768 blocks: two column tiles per gate/up wave, wide down waves
@FORMATS
def test_partial_steps_wide_launches(fmt):
    _case(fmt, 40, 120, 16, 288, 928, 110, "two tiles")
    _case(fmt, 40, 120, 16, 1760, 160, 110, "wide down")


# whole half steps (format, T, N, k, d, f, M; kernel and its instance): bf16 gate/up with 257 to
# 512 blocks, FP8 down with 513 to 768, MXFP4 at odd multiples of 128 in two-tile gate/up and
# 64-row down waves; and 64-row down waves whose reduction is shorter than a step, which take the
# 32-row instance
HALF_STEPS = [("bf16", 12, 40, 8, 384, 512, 34, "gate_up_kernel<4, false, 0, 1, false>"),
              ("fp8", 12, 48, 8, 1664, 192, 40, "down_kernel<2, 1, 2, false, 4>"),
              ("mxfp4", 40, 120, 16, 384, 928, 110, "gate_up_kernel<4, false, 2, 2, false>"),
              ("mxfp4", 40, 120, 16, 1760, 384, 110, "down_kernel<4, 2, 4, false, 2>"),
              ("fp8", 40, 120, 16, 1760, 96, 110, "down_kernel<4, 1, 2, true, 4>"),
              ("mxfp4", 40, 120, 16, 1760, 96, 110, "down_kernel<4, 2, 2, true, 4>"),
              ("bf16", 40, 120, 16, 1760, 32, 110, "down_kernel<2, 0, 2, true, 4>")]


@pytest.mark.parametrize("fmt,T,N,k,d,f,M,kernel", HALF_STEPS)
def test_half_steps_and_short_reductions(fmt, T, N, k, d, f, M, kernel):
    _case(fmt, T, N, k, d, f, M, kernel)


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


# experts of 1 to 128 rows side by side; the first with 256 weight rows a gate/up block (2475
# blocks), over reductions of one or two steps
@FORMATS
def test_large_batch_uneven_experts(fmt):
    _case(fmt, 130, 64, 16, 160, 4128, 60, "uneven")
    _case(fmt, 400, 12, 2, 608, 224, 12, "uneven")


@pytest.mark.parametrize("T", [40, 129, 260])
def test_large_batch_shared_experts(T):
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


def _rows(T, N, k, M, Q):
    """Routed rows of each expert of a batch that `_case` (with Q domains) runs."""
    h = W.make_logits(dict(N=N, k=k, T=T, logits="domains", Q=Q), 5)[0]
    return np.bincount(oracle_route(h, k, 1, M).ids.ravel(), minlength=N)


@FORMATS
@pytest.mark.parametrize("d,f", TWO_PASS_DIMS)
def test_two_staged_passes(fmt, d, f):
    assert _rows(**TWO_PASS, Q=1).max() > 32
    _case(fmt, *(TWO_PASS[a] for a in ("T", "N", "k")), d, f, TWO_PASS["M"], "two passes", Q=1)


# the same with every length of the last pass (8 rows more each) and with four passes
STAGED_PASSES = [(T, 24, 2, 16) for T in (40, 46, 60, 62)] + [(128, 40, 2, 28)]


@FORMATS
@pytest.mark.parametrize("T,N,k,M", STAGED_PASSES)
def test_staged_passes_by_length(fmt, T, N, k, M):
    rows = _rows(T, N, k, M, 1).max()
    assert rows > (96 if T == 128 else 32)
    _case(fmt, T, N, k, 320, 192, M, f"passes of {rows} rows", Q=1)


# the persistent down launch with one unit a block (256 units), experts of up to 39 rows: two
# passes a unit
PERSISTENT = (39, 64, 8, 7168, 256, 16)                                         # T, N, k, d, f, M


def test_persistent_down_one_round():
    T, N, k, _, _, M = PERSISTENT
    assert _rows(T, N, k, M, 3).max() > 32
    _case("bf16", *PERSISTENT, "persistent down, one round")


# large batches with 256 weight rows a gate/up block, through pairs of steps of the pipelined
# loop, with and without a remainder, for every count of token tiles (1 to 128 rows an expert)
WIDE_256 = dict(T=130, N=36, k=10, M=32)
WIDE_256_DIMS = [(512, 4128), (800, 4128), (1056, 4128)]


@FORMATS
@pytest.mark.parametrize("d,f", WIDE_256_DIMS)
def test_large_batch_256_rows_a_block(fmt, d, f):
    rows = _rows(**WIDE_256, Q=3)
    for lo, hi in ((0, 16), (16, 32), (32, 48), (48, 64), (64, 96), (96, 128)):
        assert np.any((rows > lo) & (rows <= hi)), (lo, hi, sorted(rows))
    _case(fmt, *(WIDE_256[a] for a in ("T", "N", "k")), d, f, WIDE_256["M"], "256 rows")


# FP8 splits d over the waves of a block also where d is an odd multiple of 128, so that a wave's
# part is an odd number of 32-element groups: one to five of them
ODD_PARTS = [(1, 16, 4, 128, 96, 4), (6, 24, 2, 384, 32, 12), (16, 40, 2, 640, 160, 16),
             (9, 20, 1, 896, 64, 9)]


@pytest.mark.parametrize("T,N,k,d,f,M", ODD_PARTS)
def test_waves_split_odd_d(T, N, k, d, f, M):
    _case("fp8", T, N, k, d, f, M, "waves split odd d")
