"""Which kernels the built library launches for which calls, and what registers they take (on the
CPU: tests/launches.py)."""
import re

import pytest

from launches import launches


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
