"""The grid-wide round loop at the edges of its branches: holders per lane
(C up to 256, up to 512, above), experts merged by one wave or by the block,
more bids for a block's experts than its list holds, one- and two-byte expert
indices, several experts per block, free slots filled and holders displaced in
one round. And the score summaries the bids read."""
import numpy as np
import pytest
import torch

import oracle
import paper_2103_16716_amd as pb
import workloads as wl
from gpu_common import dev, eps_expected, host, rounding_slack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "the GPU tests need an MI355X"
    pb.lib()


def _scores(T, E, kind, seed):
    if kind == "int16":
        return wl.random_scores(T, E, seed, "int16")
    S = wl.random_scores(T, E, seed)
    if kind == "crowd":      # every token wants the same expert first
        S[:, E // 2] += 6.0
    if kind == "eight":      # eight experts everyone prefers: many large rounds
        S[:, :8] += 3.0
    if kind == "tied":       # many equal scores, also at the end of a summary
        S = np.round(S * 4.0) / np.float32(4.0)
    if kind == "close":      # scores that differ in their last bits only
        S = (np.float32(1.0) + wl.random_scores(T, E, seed + 1) * np.float32(2e-6))
    return S.astype(np.float32)


@pytest.mark.parametrize("kind", ["normal", "crowd", "int16"])
@pytest.mark.parametrize("T,E", [(2048, 128), (2048, 8), (2044, 4), (2048, 2), (1000, 250),
                                 (2047, 23), (2048, 32), (2015, 31)])
def test_same_rounds_as_the_single_workgroup_solver(monkeypatch, T, E, kind):
    """The single-workgroup solver runs the same rounds with code of its own:
    assignment, sort vector, prices and round count agree bit for bit. (Without
    early phase ends, which the two routes take at different rounds; integer
    solves without the duality checks, which the routes make in other phases.)"""
    monkeypatch.setenv("BASE_EARLY_END_DIV", "0")
    S = dev(_scores(T, E, kind, seed=T + E))
    res = []
    for route in ("1", "0"):
        monkeypatch.setenv("BASE_SMALL_PATH", route)
        res.append(pb.assign(S, flags=pb.BASE_ASSIGN_FULL_SCHEDULE if kind == "int16" else 0))
    for name in ("assign", "perm", "prices"):
        np.testing.assert_array_equal(host(getattr(res[0], name)), host(getattr(res[1], name)))
    assert (res[0].stats.rounds, res[0].stats.bids) == (res[1].stats.rounds, res[1].stats.bids)


@pytest.mark.parametrize("T,E,kind", [(16384, 32, "crowd"), (6000, 600, "normal"),
                                      (6000, 600, "crowd"), (12288, 8, "crowd"),
                                      (4097, 17, "crowd"),
                                      # experts of more than 512 tokens: bids with their
                                      # keys in the bucket, with positions only, beyond it
                                      (16416, 32, "normal"), (4104, 8, "eight"),
                                      (16416, 32, "crowd"), (135200, 260, "normal"),
                                      # the score summaries: rows of part groups and
                                      # of whole ones, ties at the 8th and 9th score
                                      (264, 33, "tied"), (512, 64, "tied"), (2000, 100, "close"),
                                      (2064, 129, "tied"), (4096, 256, "close"),
                                      (1028, 257, "tied"), (4096, 512, "tied")])
def test_optimality_bound(T, E, kind):
    """Weak duality at the returned prices certifies the bound, whatever path
    the merges took; every expert is full and perm is the stable sort."""
    Sh = _scores(T, E, kind, seed=3 * T + E)
    res = pb.assign(dev(Sh))
    a, p = host(res.assign), host(res.prices).astype(np.float64)
    assert oracle.balanced_counts_ok(a, E)
    np.testing.assert_array_equal(host(res.perm), oracle.stable_perm(a, E))
    S = Sh.astype(np.float64)
    gap = oracle.dual_bound(S, p) - oracle.objective(S, a)
    assert gap <= T * eps_expected(Sh, 1e-4) + rounding_slack(T, S, p)


@pytest.mark.parametrize("B,T,E", [(160, 4096, 256), (640, 2560, 64), (128, 4096, 512),
                                   (136, 2048, 1024), (12, 4096, 2048)])
def test_large_batches_keep_the_loop(B, T, E):
    """Batches that leave a problem few blocks, down to one that owns every
    expert, or that exceed the device run their large rounds in the loop too.
    The problems are those of a batch of four, so the results repeat and the
    bids placed in the engine (rounds of at most 256 tokens) add up. One phase,
    so one slot: without the loop it would end in the tail, with no bid in the
    engine. (Above 512 experts there is no engine: the loop runs every round,
    the experts of a block numbered beyond 256.)"""
    kw = dict(eps_initial=0.02, eps_final=0.02)
    four = torch.stack([dev(_scores(T, E, "eight", seed=T + E + b)) for b in range(4)])
    ref = pb.assign_batched(four, **kw)
    assert ref.stats.phases == 1 and (ref.stats.engine_bids > 0 or E > 512)
    res = pb.assign_batched(four.repeat(B // 4, 1, 1), **kw)
    for name in ("assign", "perm", "prices"):
        x, y = getattr(res, name), getattr(ref, name)
        assert torch.equal(x.view(B // 4, 4, -1), y.view(1, 4, -1).expand(B // 4, 4, -1))
    assert res.stats.bids == B // 4 * ref.stats.bids
    assert res.stats.engine_bids == B // 4 * ref.stats.engine_bids


@pytest.mark.parametrize("B,T,E", [(24, 4096, 64), (3, 8192, 128), (1, 16384, 128), (64, 8192, 16)])
def test_four_solves_at_once(B, T, E):
    """Four solves on streams of their own, their loops' waiting blocks side by
    side: each ends balanced, with the results it has alone. (The last shape
    has more positions a block than its token list holds.)"""
    S = [torch.stack([dev(_scores(T, E, "normal", seed=1000 * i + b % 5)) for b in range(B)])
         for i in range(4)]
    one = [pb.assign_batched(s) for s in S]
    ws = [torch.empty(pb.assign_batched_workspace_size(B, T, E), dtype=torch.uint8, device="cuda")
          for _ in S]
    out = [[torch.empty_like(x) for x in (r.assign, r.perm, r.prices)] for r in one]
    streams = [torch.cuda.Stream() for _ in S]
    torch.cuda.synchronize()
    for _ in range(3):
        for s, w, o, st in zip(S, ws, out, streams):
            pb.assign_batched(s, workspace=w, out_assign=o[0], out_perm=o[1], out_prices=o[2],
                              sync_stats=False, stream=st)
    for w, o, st, r in zip(ws, out, streams, one):
        code, stats = pb.assign_status(w, T, E, B=B, stream=st)
        assert code == pb.BASE_OK and stats.converged == 1
        for x, y in zip(o, (r.assign, r.perm, r.prices)):
            assert torch.equal(x, y)


def test_tokens_of_a_block_beyond_its_list():
    """Blocks with more positions than their token list in LDS holds (two blocks
    for 8192 tokens) against the problems' own solves (128 blocks)."""
    B, T, E = 96, 8192, 16
    S = torch.stack([dev(_scores(T, E, ("normal", "eight", "crowd")[b % 3], seed=b)) for b in range(6)])
    res = pb.assign_batched(S.repeat(B // 6, 1, 1))
    for b in range(6):
        ref = pb.assign(S[b].contiguous())
        for k in (b, b + 48, B - 6 + b):
            for name in ("assign", "perm", "prices"):
                assert torch.equal(getattr(res, name)[k], getattr(ref, name))
