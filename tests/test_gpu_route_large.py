"""The four-kernel selection (batches past the one-workgroup kernel) against the oracle, bit
for bit, at the edges of its sizes: the first batch that takes it for each range of N, batches
that leave a partial wave, block or 64-entry piece, the largest T * k and T."""
import numpy as np
import pytest

from helpers import assert_route_equal, gpu_route, oracle_route, say

pytestmark = pytest.mark.gpu

SHAPES = [(65, 8, 2), (65, 64, 3), (57, 65, 8), (64, 128, 20), (41, 129, 5), (63, 256, 8),
          (33, 300, 7), (17, 513, 8), (256, 1024, 32), (129, 1, 1), (1024, 40, 8),
          (4096, 300, 2), (273, 30, 30)]


@pytest.mark.parametrize("T,N,k", SHAPES)
def test_large_batches_equal_the_oracle(T, N, k):
    rng = np.random.default_rng(T * 7 + N)
    h = rng.standard_normal((T, N)).astype(np.float32)
    if N % 2:                                    # ties and signed zeros
        h = (np.round(h * 8) / 8).astype(np.float32)
        h[rng.random(h.shape) < 0.1] = np.float32(-0.0)
    cuts = np.sort(rng.choice(np.arange(1, T), min(T // 3, 40), replace=False)) if T > 3 else []
    off = np.concatenate([[0], cuts, [T]]).astype(np.int32)
    k0 = min(1, k)
    for label, args, more in [
            ("total", (k0, min(N, k + 5), "total", "topk"), {}),
            ("extra", (0, 3, "extra", "topk"), {}),
            ("dense", (k0, min(N, k + 9), "total", "dense"), {}),
            ("threshold", (k0, 0, "threshold", "topk"), dict(tau=0.7)),
            ("requests", (k0, min(N, k + 12), "total", "topk"), dict(offsets=off, m_r=2)),
            ("dense requests", (0, 2, "extra", "dense"), dict(offsets=off, m_r=3))]:
        say(f"large route {label} T={T} N={N} k={k}")
        got = gpu_route(h, k, *args, **more)
        assert_route_equal(got, oracle_route(h, k, *args, **more), label)


# the instances for few ranks (token sets of two words past 64) and the first batches past them
@pytest.mark.parametrize("T,N,k", [
    (65, 8, 1), (128, 64, 1), (129, 64, 1), (116, 20, 2), (117, 20, 2), (92, 64, 4), (93, 33, 4),
    (65, 65, 2), (112, 128, 1), (113, 128, 1), (80, 100, 3), (81, 100, 3), (41, 129, 4),
    (72, 256, 1), (73, 256, 1), (60, 200, 2), (41, 256, 3), (25, 257, 4), (52, 512, 1),
    (53, 512, 1), (17, 513, 1), (32, 1024, 1), (33, 1024, 1), (20, 1000, 4), (21, 1000, 4)])
def test_few_ranks_equal_the_oracle(T, N, k):
    test_large_batches_equal_the_oracle(T, N, k)


@pytest.mark.parametrize("T,N,k", [(65, 64, 1), (100, 128, 1), (72, 256, 1), (40, 300, 2)])
def test_few_ranks_refuse_bad_offsets(T, N, k):
    h = np.random.default_rng(3).standard_normal((T, N)).astype(np.float32)
    for off in ([0, 5, 5, T], [1, T], [0, 9, T + 1], [0, T - 1]):
        got = gpu_route(h, k, 1, 8, offsets=off, m_r=1, device_offsets_only=True)
        assert got["stats"][0] == -1 and not got["sel_mask"].any()
        assert (got["ids"] == -1).all() and not got["w"].any()


@pytest.mark.parametrize("T", [65, 500])
def test_large_batches_refuse_bad_offsets_and_groups(T):
    """Offsets and group maps seen only on the device: nothing is selected."""
    import torch
    from paper_2602_07265_amd import xshare as X
    h = np.random.default_rng(3).standard_normal((T, 64)).astype(np.float32)
    for off in ([0, 5, 5, T], [1, T], [0, 9, T + 1], [0, T - 1]):
        got = gpu_route(h, 4, 1, 8, offsets=off, m_r=1, device_offsets_only=True)
        assert got["stats"][0] == -1 and not got["sel_mask"].any()
        assert (got["ids"] == -1).all() and not got["w"].any()
    groups = torch.zeros(64, dtype=torch.int32, device="cuda")
    groups[63] = 4
    got = X.select_ep(torch.from_numpy(h).cuda(), X.GroupMap(4, groups), 4, 1, 3)
    torch.cuda.synchronize()
    assert int(got["stats"][0]) == -1 and not bool(got["sel_mask"].any())
    assert bool((got["ids"] == -1).all()) and not bool(got["group_load"].any())


@pytest.mark.parametrize("T,N,G", [(65, 64, 8), (300, 256, 8), (130, 96, 3), (1024, 128, 128)])
def test_large_batches_over_gpu_groups(T, N, G):
    import torch
    from oracle import route as OR
    from paper_2602_07265_amd import xshare as X
    rng = np.random.default_rng(T)
    h = rng.standard_normal((T, N)).astype(np.float32)
    g = rng.integers(0, G, N) if G == 3 else np.arange(N) // (N // G)
    for k0, m in ((1, 2), (0, 5)):
        say(f"large route groups T={T} N={N} G={G} m_g={m}")
        got = X.select_ep(torch.from_numpy(h).cuda(), X.GroupMap(G, list(g)), 8, k0, m)
        torch.cuda.synchronize()
        got = {a: v.cpu().numpy() for a, v in got.items()}
        ref = OR.select_ep(h, 8, k0, m, g, G)
        assert_route_equal(got, ref, "groups")
        assert np.array_equal(got["group_load"], np.bincount(g[ref.sel_mask.astype(bool)],
                                                             minlength=G))
