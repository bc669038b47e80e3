"""EvictionPass.evict with budgets of the caller's own: calls issued one behind another without a wait, on a
stream of the caller's, and captured; each must work with its own counts and places."""
import numpy as np
import pytest
import torch

from gpu_util import load_cake, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
L, B, H_Q, H_KV, D, N, S_W = 3, 2, 4, 2, 64, 700, 32


def _make(cake, layers=L, n=N, total=None):
    gen = torch.Generator(device=DEV).manual_seed(3)
    mk = lambda heads, rows: [torch.randn(B, heads, rows, D, device=DEV, generator=gen) for _ in range(layers)]
    ev = cake.EvictionPass(mk(H_Q, S_W), mk(H_KV, n), mk(H_KV, n), total or layers * 150)
    ev.scores()
    return ev


def _budgets(*per_layer):
    return np.stack([np.asarray(per_layer), np.asarray(per_layer)[::-1]], axis=1).astype(np.int64) + S_W


def _outputs(ev, placed):
    """Copies of an evict's per-layer results, cut to the rows each sequence keeps."""
    keep, idx, k, v, ind = placed
    return [t[l][b, :, : int(keep[l, b]) + extra].clone() for t, extra in ((idx, 0), (k, S_W), (v, S_W), (ind, 0))
            for l in range(len(keep)) for b in range(B)]


def _expected(ev, budgets):
    """The same from torch: stable descending sort, ascending positions, window rows behind."""
    keep = budgets - S_W
    pick = [[[torch.sort(torch.sort(ev.indicator[l, b, h], descending=True, stable=True)[1][: int(keep[l, b])])[0] for h in range(H_KV)]
             for b in range(B)] for l in range(len(keep))]
    window = torch.arange(ev.N_p, ev.N, device=DEV)
    stack = lambda f: [torch.stack([f(l, b, h, pick[l][b][h]) for h in range(H_KV)]) for l in range(len(keep)) for b in range(B)]
    return (stack(lambda l, b, h, p: p.int()) + stack(lambda l, b, h, p: ev.k[l][b, h][torch.cat([p, window])])
            + stack(lambda l, b, h, p: ev.v[l][b, h][torch.cat([p, window])]) + stack(lambda l, b, h, p: ev.indicator[l, b, h][p]))


def _check(got, want):
    for i, (a, b) in enumerate(zip(got, want, strict=True)):
        assert torch.equal(a, b), i


@pytest.mark.parametrize("side", [False, True])
def test_evictions_one_behind_another_keep_their_own_counts(side):
    cake = load_cake()
    say(f"two evictions without a wait, side stream {side}")
    ev = _make(cake)
    first, second = _budgets(150, 20, 100), _budgets(5, 180, 60)
    want = _expected(ev, first), _expected(ev, second)
    busy = torch.randn(8192, 8192, device=DEV)
    stream = torch.cuda.Stream() if side else torch.cuda.current_stream()
    torch.cuda.synchronize()
    got = []
    with torch.cuda.stream(stream):
        for _ in range(4):
            busy @ busy                             # the stream is behind the host while both calls are made
    for budgets in (first, second):
        placed = ev.evict(budgets, stream if side else None)
        with torch.cuda.stream(stream):
            got.append(_outputs(ev, placed))
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        _check(g, w)


def test_captured_evictions_replay_with_their_own_counts():
    cake = load_cake()
    say("captured evictions")
    ev = _make(cake)
    budgets = _budgets(150, 20, 100), _budgets(5, 180, 60)
    want = [_expected(ev, b) for b in budgets]
    ev.evict(budgets[0])
    torch.cuda.synchronize()
    graphs, placed = [torch.cuda.CUDAGraph() for _ in budgets], []
    side = torch.cuda.Stream()
    for graph, b in zip(graphs, budgets):
        with torch.cuda.graph(graph, stream=side):
            placed.append(ev.evict(b))
    for replay in range(3):
        for graph, p, w in zip(graphs, placed, want):
            for pool in (ev.pool_k, ev.pool_v, ev.pool_ind, ev.pool_idx):
                pool.zero_()
            ev.evict(_budgets(40, 40, 40))
            graph.replay()
            torch.cuda.synchronize()
            _check(_outputs(ev, p), w)


def test_places_of_more_layers_than_one_launch_holds():
    cake = load_cake()
    say("300 layers")
    ev = _make(cake, layers=300, n=S_W + 8, total=300 * (S_W + 5))
    budgets = np.tile(_budgets(0, 5, 3), (100, 1))
    got = _outputs(ev, ev.evict(budgets))
    torch.cuda.synchronize()
    _check(got, _expected(ev, budgets))


def test_budgets_beyond_the_pools_are_refused_before_anything_is_launched():
    cake = load_cake()
    say("budgets that fill the pools and one row more")
    ev = _make(cake, total=L * (S_W + 50))
    fits = np.repeat(_budgets(150, 100, 50)[:, :1], B, axis=1)       # 300 = B * 3 * 50 rows: all there are
    want = _outputs(ev, ev.evict(fits))
    _check(want, _expected(ev, fits))
    before = [t.clone() for t in (ev.pool_k, ev.pool_v, ev.pool_idx, ev.pool_ind, ev.tbl_out)]
    over = fits.copy()
    over[2, 1] += 1
    for call in (ev.evict, ev.evict_launch):
        with pytest.raises(ValueError, match="pools"):
            call(over)
    torch.cuda.synchronize()
    for t, b in zip((ev.pool_k, ev.pool_v, ev.pool_idx, ev.pool_ind, ev.tbl_out), before):
        assert torch.equal(t, b)
    _check(_outputs(ev, ev.evict(fits)), want)
