"""The device-chained cascade's lists (csrc/cascade_stage.hip, select_stage_kernel) as a model on the host: counts, places, stack of
free places, rows of the store, gather.  The kernels hold an index at its buffer's ends; the model lets none pass that lies
outside, and checks that no place is held twice and every kept row is where its list says."""
import numpy as np
import pytest

from oracle import cake_oracle as co


class _Buffer:
    """Words that are read only where something was written, and only inside."""

    def __init__(self, size):
        self.data = np.full(max(size, 1), -1, dtype=np.int64)

    def put(self, at, value):
        assert 0 <= at < self.data.size, (at, self.data.size)
        self.data[at] = value

    def get(self, at):
        assert 0 <= at < self.data.size, (at, self.data.size)
        assert self.data[at] >= 0, at
        return int(self.data[at])


def _cascade(rng, L, B, N, S_w, total, prefs, kept_all_at):
    """Runs L stages of B sequences of one head; returns how many stages it checked."""
    n_p = N - S_w
    most = min(total, L * N)
    prefix_rows = max(most - S_w, 1)
    words = B * B * prefix_rows                                # a list holds [B, cap_l] per layer, cap_l the largest count of the batch
    slots = [_Buffer(words), _Buffer(words)]
    scores = [_Buffer(words), _Buffer(words)]                  # of each held row, as a whole number
    free = [_Buffer(prefix_rows) for _ in range(B)]
    for f in free:
        f.data[:] = np.arange(prefix_rows)
    store = [_Buffer(prefix_rows + L * S_w) for _ in range(B)]    # which row of which layer lies there
    row_id = lambda l, p: l * N + p
    keep_before, held = np.zeros((0, B), dtype=np.int64), []   # held[l][b]: kept positions, the reference
    offsets_before = np.zeros(0, dtype=np.int64)
    for m in range(L):
        cur = np.concatenate([keep_before, np.full((1, B), n_p)])
        budgets = np.array([co.cascade_allocate(prefs[b][:m + 1], total, S_w, N) for b in range(B)]).T
        keep = np.minimum(np.maximum(budgets - S_w, 0), cur)
        caps_in, caps_out = np.append(keep_before.max(axis=1), n_p), keep.max(axis=1)
        offsets = B * np.concatenate([[0], np.cumsum(caps_out)[:-1]])
        old, new, s_old, s_new = slots[(m & 1) ^ 1], slots[m & 1], scores[(m & 1) ^ 1], scores[m & 1]
        fresh = rng.integers(0, 4 if rng.random() < 0.5 else 10 ** 6, size=(B, n_p))       # with many ties, or few
        held.append([np.arange(n_p) for _ in range(B)])
        for b in range(B):
            for l in range(m + 1):
                c, k = int(cur[l, b]), int(keep[l, b])
                at_in = 0 if l == m else int(offsets_before[l]) + b * int(caps_in[l])
                at_out = int(offsets[l]) + b * int(caps_out[l])
                value = [int(fresh[b, p]) if l == m else s_old.get(at_in + p) for p in range(c)]
                chosen = co.select_topk(np.array(value, dtype=np.float64), k) if k < c else np.arange(c)
                if l < m:
                    # the stack's height: what was free, then what the layers before drop
                    top = prefix_rows - int(cur[:m, b].sum()) + int((cur[:l, b] - keep[:l, b]).sum())
                    stay = np.zeros(c, dtype=bool)
                    stay[chosen] = True
                    r = 0
                    for p in range(c):
                        if stay[p]:
                            new.put(at_out + r, old.get(at_in + p))
                            s_new.put(at_out + r, value[p])
                            r += 1
                        else:
                            free[b].put(top + p - r, old.get(at_in + p))
                    assert r == k
                held[l][b] = held[l][b][chosen]
            # the new layer's rows, after the lists
            c, k, top = int(cur[m, b]), int(keep[m, b]), prefix_rows - int(keep[:m, b].sum())
            for r in range(k):
                slot = free[b].get(top - 1 - r)
                assert slot < prefix_rows
                at = int(offsets[m]) + b * int(caps_out[m]) + r
                new.put(at, slot)
                s_new.put(at, int(fresh[b, held[m][b][r]]))
                store[b].put(slot, row_id(m, int(held[m][b][r])))
            for w in range(S_w):
                store[b].put(prefix_rows + m * S_w + w, row_id(m, n_p + w))
            # every kept row is where its list says, no place is held twice
            places = []
            for l in range(m + 1):
                for r in range(int(keep[l, b])):
                    slot = new.get(int(offsets[l]) + b * int(caps_out[l]) + r)
                    assert slot < prefix_rows + l * S_w                # what the gather clamps to
                    assert store[b].get(slot) == row_id(l, int(held[l][b][r])), (m, b, l, r)
                    places.append(slot)
                for w in range(S_w):
                    assert store[b].get(prefix_rows + l * S_w + w) == row_id(l, n_p + w)
            assert len(set(places)) == len(places)
        kept_all_at.append(bool((keep == cur).all()))
        keep_before, offsets_before = keep, offsets
    return L


def test_lists_of_random_cascades():
    rng = np.random.default_rng(7)
    stages, whole = 0, []
    for trial in range(120):
        B, S_w = int(rng.integers(1, 4)), int(rng.integers(1, 5))
        L = int(rng.integers(1, 9)) if trial % 8 else int(rng.integers(60, 71))      # more layers than a wave has lanes
        N = S_w + int(rng.integers(1, 30 if L < 20 else 8))
        kind = trial % 5
        total = L * S_w if kind == 0 else L * N + int(rng.integers(0, 9)) if kind == 1 else int(rng.integers(L * S_w, L * N + 1))
        prefs = np.exp(2.0 * rng.standard_normal((B, L)))
        if kind == 2:
            prefs[:, rng.random(L) < 0.4] = 0.0
        if kind == 3:
            prefs[0] = prefs[0, 0]
        stages += _cascade(rng, L, B, N, S_w, total, prefs, whole)
    assert stages > 900 and any(whole) and not all(whole)


@pytest.mark.parametrize("bad", [-1, 5])
def test_the_model_refuses_an_index_outside(bad):
    with pytest.raises(AssertionError):
        _Buffer(5).put(bad, 1)
