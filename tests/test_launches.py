"""Which kernels the built library launches for which calls, and what registers they take (on the
CPU: tests/launches.py)."""
import re

import pytest

import test_gpu_gemm_shapes as shapes
from launches import kernels, launches, short_names


def route(T, N, k, **more):
    return dict(op="route", T=T, N=N, k=k, d=32, f=32, M=max(k, min(N, 3 * k)), **more)


def _names(cases):
    return [[n for n, _, _ in one] for one in launches(cases)]


FOUR = ["route_tokens_kernel", "route_scores_kernel", "route_refine_kernel", "route_lists_kernel"]


def test_selection_of_few_ranks_takes_one_launch():
    """Batches of tokens of few ranks whose one-workgroup selection is the faster one (four
    launches cost 24 us in a stream of calls; one workgroup took 17 to 21 us on these), and the
    first ones past it."""
    one = [(41, 256, 1), (72, 256, 1), (48, 256, 3), (64, 128, 2), (57, 128, 6), (100, 128, 1),
           (128, 60, 1), (65, 8, 2), (40, 512, 2), (52, 512, 1), (24, 1024, 2), (32, 1024, 1)]
    four = [(73, 256, 1), (61, 256, 2), (41, 256, 5), (57, 128, 8), (113, 128, 1), (129, 60, 1), (65, 8, 5),
            (53, 512, 1), (25, 512, 8), (33, 1024, 1), (17, 1024, 8), (1024, 8, 2)]
    got = _names([route(*c) for c in one + four])
    for c, names in zip(one, got):
        assert len(names) == 1 and names[0].startswith("route_kernel<"), (c, names)
    for c, names in zip(four, got[len(one):]):
        assert [re.sub("<.*", "", n) for n in names] == FOUR, (c, names)


@pytest.mark.parametrize("score,reqs", [("dense", 0), ("topk", 8)])
def test_every_batch_size_has_an_instance_for_its_tokens(score, reqs):
    """The few-rank instances are for batches past the others' tokens, and never for dense scores
    or more than four ranks."""
    limit = {1: (64, 128), 2: (64, 112), 4: (40, 72), 8: (24, 52), 16: (16, 32)}
    cases = [route(T, N, k, score=score, **(dict(reqs=reqs, m_r=1) if reqs else {}))
             for N in (8, 64, 128, 200, 256, 500, 1000) for k in (1, 2, 4, 5, 8)
             for T in (8, 16, 17, 24, 25, 32, 33, 40, 41, 52, 53, 56, 57, 64, 65, 72, 73, 112, 113, 128, 129)]
    for c, names in zip(cases, _names(cases)):
        m = re.fullmatch(r"route_kernel<(\d+), (\w+)>", names[0])
        if not m:
            continue
        few = m[2] == "true"
        assert c["T"] <= limit[int(m[1])][few], (c, names)
        assert not few or (c["k"] <= 4 and score != "dense" and c["T"] > limit[int(m[1])][0]), c


def layer(T, N, k, M, d, f, fmt="bf16", **more):
    return dict(T=T, N=N, k=k, M=M, d=d, f=f, fmt=fmt, **more)


def _instance(names, kernel):
    """Template arguments of the one launch of `kernel`."""
    found = [re.fullmatch(kernel + r"<(.*)>", n) for n in names]
    found = [m for m in found if m]
    assert len(found) == 1, (kernel, names)
    return found[0][1].split(", ")


@pytest.mark.parametrize("T,N,M,d,f", [(4, 96, 20, 4224, 2944), (32, 96, 48, 4224, 2944),
                                       (32, 64, 48, 2688, 1408), (32, 96, 48, 5120, 1664)])
def test_mxfp4_whole_half_steps(T, N, M, d, f):
    """Reductions of odd multiples of 128 with MXFP4 weights run whole 128-element steps: the
    partial-step instances are 10 to 12 % slower there."""
    (names,) = _names([layer(T, N, 6, M, d, f, "mxfp4")])
    for kernel, args, K in (("gate_up_kernel", slice(0, 5, 4), d), ("down_kernel", slice(0, 4, 3), f)):
        step, rest = _instance(names, kernel)[args]
        assert rest == "false" and K % (32 * int(step)) == 0, (kernel, names)


@pytest.mark.parametrize("fmt", ["bf16", "fp8", "mxfp4"])
def test_split_reductions_run_whole_steps(fmt):
    """The parts of a split reduction are multiples of 128."""
    cases = [layer(T, 16, 2, M, d, f, fmt) for T in (20, 32) for M in (3, 6, 8)
             for d in (512, 768, 1024, 1536, 2304, 2816) for f in (256, 768, 1408)]
    seen = 0
    for c, one in zip(cases, launches(cases)):
        for name, grid, _ in one:
            m = re.fullmatch(r"gate_up_kernel<(\d+), (\w+), \d+, \d+, (\w+)>", name)
            if m and grid[2] > 1:
                seen += 1
                assert m[2] == "true" and m[3] == "false", (c, name)
                assert (c["d"] // grid[2]) % (32 * int(m[1])) == 0, (c, name, grid)
    assert seen > 10


def _registers():
    meta = kernels()
    return dict(zip(short_names(list(meta)), meta.values()))


def test_no_kernel_spills():
    """No kernel keeps vector registers in scratch memory.  The two-tile FP8 gate/up, which is
    held to three waves a SIMD, and the partial-step instances come closest."""
    regs = _registers()
    for name, k in regs.items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, (name, k)
    assert regs["gate_up_kernel<4, false, 1, 2, false>"][".vgpr_count"] <= 168
    assert sum(n.endswith("true>") or "true, " in n for n in regs) >= 8


@pytest.mark.parametrize("fmt", list(shapes.RUN))
def test_partial_step_cases_run_the_partial_step(fmt):
    """The GPU tests of the partial steps reach the instances that they are for."""
    for names in _names([layer(T, N, k, M, d, f, fmt) for d, f in shapes.PARTIAL_DIMS
                         for T, N, k, M in shapes.PARTIAL_ROWS]):
        assert _instance(names, "gate_up_kernel")[4] == "true", names
        assert _instance(names, "down_kernel")[3] == "true", names
    for names in _names([layer(d=d, f=f, fmt=fmt, **shapes.TWO_PASS)
                         for d, f in shapes.TWO_PASS_DIMS] +
                        [layer(T, N, k, M, 320, 192, fmt) for T, N, k, M in shapes.STAGED_PASSES]):
        assert _instance(names, "gate_up_kernel") and _instance(names, "down_kernel")


def test_whole_half_steps_by_rounds_of_blocks():
    """bf16 gate/up at odd multiples of 128 and FP8 down at odd multiples of 64: the plain
    instances of half the step where they make the shorter launch, and only there."""
    case = lambda T, M, d, f, fmt: layer(T, 96, 6, M, d, f, fmt)     # noqa: E731
    gate_up = [(case(16, 24, 4992, 768, "bf16"), "4"), (case(4, 12, 2688, 1664, "bf16"), "4"),
               (case(32, 40, 2688, 768, "bf16"), "4"), (case(16, 12, 4992, 768, "bf16"), "8"),
               (case(2, 12, 2688, 1664, "bf16"), "8"), (case(4, 20, 2688, 1664, "bf16"), "8"),
               (case(32, 40, 4992, 1664, "bf16"), "8")]
    down = [(case(16, 24, 2752, 832, "fp8"), "2"), (case(8, 32, 2752, 1472, "fp8"), "2"),
            (case(4, 20, 2752, 1472, "fp8"), "4"), (case(16, 40, 2752, 1472, "fp8"), "4"),
            (case(16, 24, 2752, 1440, "fp8"), "4")]
    for kernel, rest, want in (("gate_up_kernel", 4, gate_up), ("down_kernel", 3, down)):
        full = "8" if kernel == "gate_up_kernel" else "4"
        for (c, step), names in zip(want, _names([c for c, _ in want])):
            args = _instance(names, kernel)
            assert args[0] == step and args[rest] == ("true" if step == full else "false"), (c, names)


def test_large_batch_launches_by_rounds_of_blocks():
    """Few rows more than a staged pass holds, in a grid of the large-batch launch whose last round
    is not full: staged, which measured 5 to 15 % faster; in whole rounds and with more rows the
    large-batch launches."""
    def c(T, N, k, M, d, f, fmt): return layer(T, N, k, M, d, f, fmt)     # noqa: E704
    staged = [c(64, 64, 8, 32, 3072, 1536, "fp8"), c(36, 64, 8, 18, 1024, 2048, "fp8"),
              c(64, 48, 6, 24, 2048, 1408, "fp8"), c(96, 8, 2, 8, 4096, 14336, "mxfp4"),
              c(64, 16, 2, 5, 4096, 8192, "mxfp4"), c(96, 96, 8, 32, 5120, 1536, "mxfp4"),
              c(64, 96, 8, 21, 5120, 1536, "mxfp4")]
    wide = [c(64, 256, 8, 32, 7168, 2048, "fp8"), c(64, 96, 8, 32, 2048, 768, "fp8"),
            c(64, 8, 2, 8, 4096, 14336, "fp8"), c(52, 64, 8, 19, 3072, 1536, "fp8"),
            c(96, 16, 2, 8, 4096, 8192, "mxfp4"), c(112, 8, 2, 8, 4096, 14336, "mxfp4"),
            c(256, 128, 8, 64, 2048, 768, "mxfp4"), c(128, 96, 8, 42, 5120, 1536, "mxfp4"),
            c(64, 96, 8, 21, 2048, 768, "mxfp4"), c(64, 8, 2, 5, 4096, 14336, "bf16")]
    got = _names(staged + wide)
    for case, names in zip(staged + wide, got):
        is_wide = any(n.startswith("gate_up_wide_kernel") for n in names)
        assert is_wide == (case in wide), (case, names)


def test_large_batch_and_split_cases_run_the_kernels_they_name():
    cases = [layer(T, N, k, M, d, f, fmt) for fmt, T, N, k, d, f, M, _ in shapes.HALF_STEPS]
    for case, names in zip(shapes.HALF_STEPS, _names(cases)):
        assert case[-1] in names, (case, names)
    weight = {"bf16": "0", "fp8": "1", "mxfp4": "2"}
    for fmt, w in weight.items():
        for names in _names([layer(d=d, f=f, fmt=fmt, **shapes.WIDE_256)
                             for d, f in shapes.WIDE_256_DIMS]):
            assert _instance(names, "gate_up_wide_kernel") == [w, "256"], names
            assert _instance(names, "down_wide_kernel") == [w, "256"], names
    for names in _names([layer(T, N, k, M, d, f, "fp8") for T, N, k, d, f, M in shapes.ODD_PARTS]):
        assert _instance(names, "gate_up_narrow_kernel") == ["4", "1"], names
    # the persistent down launch of the guard test and of the multi-pass test (M = 32 of them)
    T, N, k, d, f, M = shapes.PERSISTENT
    for names in _names([layer(64, 64, 8, 32, 7168, 256), layer(T, N, k, M, d, f)]):
        assert _instance(names, "down_seq_kernel") == ["4", "0", "7", "4"], names
