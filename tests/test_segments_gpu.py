"""Key-axis segments (cake_window_scores_segment / _finish): a layer whose keys arrive a range
of positions at a time must give what the resident call gives, bit for bit, and therefore the
oracle's values within the same bars; misaligned segments are rejected on the host."""
import numpy as np
import pytest
import torch

from synth import CONFIGS, make_config_inputs

from gpu_util import assert_close, load_cake, oracle_layer, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def cake():
    return load_cake()


def _pass(cake, cfg, inp, mode=None):
    L = cfg.n_layers
    params = cake.make_params() if mode is None else cake.make_params(indicator_mode=mode)
    return cake.EvictionPass([inp["q_win"][l] for l in range(L)], [inp["k"][l] for l in range(L)],
                             [inp["v"][l] for l in range(L)], cfg.total_budget, params=params)


@pytest.mark.parametrize("cid,over,segments", [
    (1, dict(seq_len=1024 + 77), (256, 512, 768)),                                # fp32, S_w = 32, ragged last chunk
    (2, dict(n_layers=2, seq_len=2048 + 300, total_budget=2 * 300), (512, 1536)),    # bf16, G = 4, S_w = 32
    (4, dict(n_layers=2, seq_len=8192 + 64 + 5, total_budget=2 * 300), (1024, 3072)),  # bf16, S_w = 64 (pipelined pass 2)
    (5, dict(n_layers=2, batch=2, seq_len=2048 + 511, total_budget=2 * 200), (512, 1024)),  # G = 5, batch of 2
])
def test_segmented_scores_equal_resident_scores_bit_for_bit(cake, cid, over, segments):
    cfg = CONFIGS[cid].scaled(**over)
    inp = make_config_inputs(cfg, device=DEV)
    ref = _pass(cake, cfg, inp)
    ref.scores()
    torch.cuda.synchronize()
    want_ind, want_pref, want_hv = ref.indicator.clone(), ref.pref.clone(), ref.hv.clone()
    assert cake.cake_scores_chunk_keys(ref.shape) == min(segments)
    for seg in segments:
        say(f"segments of {seg} keys: config {cid} {over}")
        ep = _pass(cake, cfg, inp)
        ep.workspace.fill_(0xFF)                        # stale bytes must not leak into the result
        ep.indicator.fill_(float("nan"))
        ep.scores_segmented(seg)
        torch.cuda.synchronize()
        assert torch.equal(ep.indicator, want_ind)
        assert torch.equal(ep.pref, want_pref) and torch.equal(ep.hv, want_hv)
    # and against the oracle, one (layer, sequence), on the last segmented result
    l, b = cfg.n_layers - 1, cfg.batch - 1
    o = oracle_layer(inp["q_win"][l][b], inp["k"][l][b], ep.params)
    assert_close(ep.indicator[l, b].cpu().numpy(), o["indicator"], "segmented indicator vs oracle")
    assert_close(ep.hv[b, l, 0].item(), o["H"], "segmented H vs oracle")
    assert_close(ep.hv[b, l, 1].item(), o["V"], "segmented V vs oracle")


def test_segments_in_any_order_and_variance_mode(cake):
    """Pass-1 and pass-2 segments written in reverse order, for the variance-only indicator
    (pivoted column sums): still the resident result."""
    from paper_2503_12491_amd import binding as C
    from paper_2503_12491_amd.driver import _strides3
    cfg = CONFIGS[2].scaled(n_layers=1, seq_len=2048 + 40, total_budget=300)
    inp = make_config_inputs(cfg, device=DEV)
    ref = _pass(cake, cfg, inp, mode=cake.CAKE_IND_VAR)
    ref.scores()
    torch.cuda.synchronize()
    ep = _pass(cake, cfg, inp, mode=cake.CAKE_IND_VAR)
    N, N_p, seg = cfg.seq_len, cfg.seq_len - cfg.window, 512
    k = inp["k"][0]
    for which, end in ((1, N), (2, N_p)):
        for lo in reversed(range(0, end, seg)):
            hi = min(lo + seg, N)
            part = k[:, :, lo:hi].contiguous()          # its own allocation: nothing beyond the segment exists
            C.cake_window_scores_segment(ep.shape, ep.params, which, lo, hi - lo, ep.tbl_q, C.ptr_table([part]),
                                         _strides3(ep.q_win[0]), _strides3(part), ep.workspace)
            torch.cuda.synchronize()
        C.cake_window_scores_finish(ep.shape, ep.params, which, ep.tbl_ind if which == 2 else None, ep.workspace)
    C.cake_layer_preference(ep.shape, ep.params, ep.workspace, ep.pref, ep.hv)
    torch.cuda.synchronize()
    assert torch.equal(ep.indicator, ref.indicator) and torch.equal(ep.hv, ref.hv)


def test_misaligned_segments_are_rejected(cake):
    from paper_2503_12491_amd import binding as C
    from paper_2503_12491_amd.driver import _strides3
    cfg = CONFIGS[1]
    inp = make_config_inputs(cfg, device=DEV)
    ep = _pass(cake, cfg, inp)
    chunk = C.cake_scores_chunk_keys(ep.shape)
    qs, ks = _strides3(ep.q_win[0]), _strides3(ep.k[0])
    for lo, cnt in ((chunk // 2, chunk), (0, chunk + 1), (0, 0), (chunk, cfg.seq_len), (-chunk, chunk)):
        with pytest.raises(C.CakeError):
            C.cake_window_scores_segment(ep.shape, ep.params, 1, lo, cnt, ep.tbl_q, ep.tbl_k, qs, ks, ep.workspace)
    with pytest.raises(C.CakeError):
        C.cake_window_scores_segment(ep.shape, ep.params, 3, 0, chunk, ep.tbl_q, ep.tbl_k, qs, ks, ep.workspace)
    with pytest.raises(C.CakeError):
        C.cake_window_scores_finish(ep.shape, ep.params, 2, None, ep.workspace)
    torch.cuda.synchronize()


@pytest.mark.parametrize("spread,n", [(20.0, 4096 + 32), (16.0, 16384 + 32), (20.0, 1000)])
def test_row_normalisers_of_peaked_rows(cake, spread, n):
    """Rows whose largest logits lie some 40 to 100 (log2 units) above 0: the normalisers, which the segmented form leaves
    at the start of the workspace, against float64.  One-hot queries make every logit a stored number times the scale.
    Bound: the result's own rounding (half an ulp) and, of a sum relative to a reference that no term outruns by more
    than 2^24, the rounding of the exponents (2^-20) and of the exponentials, partial sums and merges (some eight of 2^-23 / ln 2: few terms count)."""
    say(f"normalisers of peaked rows, N={n}")
    B, H, S_w, d = 2, 8, 32, 64
    c = np.float32(0.125 * 1.4426950408889634)                   # the default scale of d = 64, in log2 units
    rng = np.random.default_rng(n)
    acc = np.zeros((B, H, n, d), dtype=np.float32)
    acc[..., :S_w] = rng.standard_normal((B, H, n, S_w)) * spread / c
    q = torch.eye(S_w, d, device=DEV).expand(B, H, S_w, d).contiguous()
    k = torch.from_numpy(acc).to(DEV)
    ev = cake.EvictionPass([q], [k], [k], S_w + n // 4)
    ev.scores_segmented(cake.cake_scores_chunk_keys(ev.shape))
    torch.cuda.synchronize()
    got = ev.workspace[: B * H * S_w * 4].view(torch.float32).view(B, H, S_w).cpu().double().numpy()
    t = acc[..., :S_w].transpose(0, 1, 3, 2).astype(np.float64) * float(c)
    t = np.where(np.arange(n) <= n - S_w + np.arange(S_w)[:, None], t, -np.inf)       # key j is visible to row r up to n - S_w + r
    top = t.max(axis=-1, keepdims=True)
    want = top[..., 0] + np.log2(np.exp2(t - top).sum(axis=-1))
    bound = 0.5 * np.spacing(np.abs(want).astype(np.float32)).astype(np.float64) + 2.0 ** -20 + 8 * 2.0 ** -23 * 1.4427
    assert top.max() > 60.0 and np.all(np.abs(got - want) <= bound), np.max(np.abs(got - want) / bound)
