"""DeviceCascade keeps a row where its layer's admission put it: lists of places, a stack of free places
per head, one gather for the result.  Its caches must equal those of CascadeSession, which copies every
layer at every stage, also where rows change hands often, and a result taken between two stages must
neither disturb the next ones nor change afterwards."""
import re

import numpy as np
import pytest
import torch

from gpu_util import kernels_of, load_cake, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # L, B, H_q, H_kv, d, N, S_w, total, dtype
    "one_layer": (1, 1, 4, 2, 64, 300, 32, 100, torch.float32),
    "windows_only": (6, 1, 4, 4, 64, 257, 32, 6 * 32, torch.bfloat16),
    "one_row_each": (5, 2, 8, 2, 128, 400, 32, 5 * 33, torch.float32),
    "fits": (3, 2, 4, 2, 64, 130, 64, 3 * 130, torch.bfloat16),
    "overflows_late": (7, 1, 8, 8, 128, 301, 32, 4 * 301 + 17, torch.bfloat16),
    "ragged_batch": (9, 3, 10, 2, 64, 999, 64, 9 * 150 + 5, torch.float32),
    "long_gaps": (4, 1, 4, 2, 128, 5003, 32, 4 * 90, torch.bfloat16),
}


def _same(got, want, S_w):
    np.testing.assert_array_equal(got.budgets, want.budgets)
    np.testing.assert_array_equal(got.keep, want.keep)
    np.testing.assert_array_equal(got.pref, want.pref)
    np.testing.assert_array_equal(got.hv, want.hv)
    for l in range(len(got.keep)):
        for b in range(got.keep.shape[1]):
            n = int(want.keep[l, b])
            for name, rows in (("k_out", n + S_w), ("v_out", n + S_w), ("ind_out", n)):
                assert torch.equal(getattr(got, name)[l][b, :, :rows], getattr(want, name)[l][b, :, :rows]), (l, b, name)


@pytest.mark.parametrize("name", CASES)
def test_rows_of_the_store_are_those_of_the_copying_cascade(name):
    cake = load_cake()
    L, B, H_q, H_kv, d, N, S_w, total, dt = CASES[name]
    say(f"cascade store: {name}")
    gen = torch.Generator(device=DEV).manual_seed(7)
    dev, host = cake.DeviceCascade(L, total), cake.CascadeSession(L, total, track_positions=False)
    early = None
    for l in range(L):
        q = (torch.randn(B, H_q, S_w, d, device=DEV, generator=gen) * (0.5 + l % 3)).to(dt)
        # rows of several heads side by side, as a projection leaves them
        k, v = [torch.randn(B, N, H_kv, d, device=DEV, generator=gen).to(dt).transpose(1, 2) for _ in range(2)]
        dev.admit(q, k, v)
        host.admit(q, k, v)
        if l == L // 2:
            early, early_want = dev.result(), host.result()
            kept = [t.clone() for t in early.k_out + early.v_out + early.ind_out]
            _same(early, early_want, S_w)
    _same(dev.result(), host.result(), S_w)
    for a, b in zip(early.k_out + early.v_out + early.ind_out, kept, strict=True):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


# rows at the edges of the stage's kernels; the last with more rows than compute units
@pytest.mark.parametrize("N,H_kv,L", [(1021 + 32, 2, 3), (1022 + 32, 2, 3), (2045 + 32, 2, 3), (2046 + 32, 2, 3), (4094 + 32, 2, 3),
                                      (8189 + 32, 1, 3), (8190 + 32, 1, 3), (16381 + 32, 1, 3), (4093 + 32, 46, 7), (8189 + 32, 46, 7)])
def test_kernels_of_a_stage(N, H_kv, L):
    cake = load_cake()
    say(f"cascade stage: {L} layers of {H_kv} heads of {N} keys")
    gen = torch.Generator(device=DEV).manual_seed(N)
    total = L * N // 6
    dev, host = cake.DeviceCascade(L, total), cake.CascadeSession(L, total, track_positions=False)
    for l in range(L):
        q = (torch.randn(1, H_kv, 32, 64, device=DEV, generator=gen) * (0.5 + l % 3)).bfloat16()
        k, v = [torch.randn(1, H_kv, N, 64, device=DEV, generator=gen).bfloat16() for _ in range(2)]
        dev.admit(q, k, v)
        host.admit(q, k, v)
    _same(dev.result(), host.result(), 32)


def test_threads_of_a_stage_by_its_rows():
    """A row has as many threads as it can use while there is a compute unit for each, 256 of them."""
    cake = load_cake()
    L, H_kv, N = 33, 8, 3032
    say(f"cascade stage: kernels of {L} layers of {H_kv} heads of {N} keys")
    gen = torch.Generator(device=DEV).manual_seed(N)
    q, k = (torch.randn(1, H_kv, rows, 64, device=DEV, generator=gen).bfloat16() for rows in (32, N))
    dev = cake.DeviceCascade(L, L * N // 6)

    def admit():
        for _ in range(L):
            dev.admit(q, k, k)
    names = [n for n in kernels_of(admit) if "select_stage" in n]
    threads = [int(re.search(r"(?:<|Li)(\d+)", n[n.index("select_stage"):])[1]) for n in names]
    assert threads == [1024] * 32 + [512], names
