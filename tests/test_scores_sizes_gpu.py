"""The score passes at the sizes where their forms change: element types and row blocks, and launches of a few
workgroups (which combine pass 1's pairs inside pass 2) against launches of many (some of which stream)."""
import re

import pytest
import torch

from gpu_util import assert_close, kernels_of, load_cake, oracle_layer, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(layers, h_q, h_kv, d, n, window, dtype, seed, peak=1.0):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    mk = lambda h, rows, t: [(torch.randn(1, h, rows, d, device=DEV, generator=gen) * t).to(dtype) for _ in range(layers)]
    return mk(h_q, window, peak), mk(h_kv, n, 1.0), mk(h_kv, n, 1.0)


@pytest.mark.parametrize("window", [32, 64])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [97, 640 + 31])      # one key past a tile; a ragged last tile behind whole granules
def test_fp32_scores_against_the_oracle(d, window, n):
    cake = load_cake()
    say(f"scores fp32 d={d} S_w={window} N={n}")
    q, k, v = _inputs(1, 6, 2, d, n, window, torch.float32, d + window + n, 2.0)
    params = cake.make_params()
    ev = cake.EvictionPass(q, k, v, 2 * window, params)
    ev.scores()
    want = oracle_layer(q[0][0], k[0][0], params)
    # fp32 sums of d products and of n exponentials, whose arguments (up to some 30) are rounded to 2^-24 of themselves;
    # gamma = 200 times a variance that is a difference of sums: 1e-4 leaves a factor of ten over what that adds up to
    assert_close(ev.indicator[0, 0].cpu().numpy(), want["indicator"], "indicator", rtol=1e-4)
    pref, hv = ev.preferences_to_host()
    assert_close(hv[0, 0, 0], want["H"], "H", rtol=1e-5)
    assert_close(hv[0, 0, 1], want["V"], "V", rtol=1e-4)


def _granules(n, window):
    """(chunk, granule) in keys of a layer of n keys."""
    chunk = 2048 if n >= 32768 else 1024 if n >= 8192 else 512 if n >= 2048 else 256
    return chunk, 2048 if n >= 65536 else 1024 if n >= 16384 else 256 if n >= 2048 else 128 if window > 32 else 64


def _combines(slices, dtype, window, group, n):
    """Whether pass 2 combines the pairs of pass 1 by itself in a call of so many slices: None where that hangs on how many
    granules a workgroup takes (one at least, a chunk at most)."""
    chunk, granule = _granules(n, window)
    n_p = n - window
    if dtype == torch.bfloat16 and window == 32 and group in (5, 6) and slices * n_p >= 2048 * 256:
        return False                               # packed slices and waves that stream do not
    pairs = group * window * -(-n // granule) * 8
    piped = dtype == torch.bfloat16 and window == 64
    fits = lambda workgroups: workgroups * pairs <= 16 << 20 and (not piped or workgroups <= 256)
    fewest, most = fits(slices * -(-n_p // chunk)), fits(slices * -(-n_p // granule))
    return fewest if fewest == most else None


@pytest.mark.parametrize("peak", [1.0, 12.0])      # references all 0; references of their own
@pytest.mark.parametrize("dtype,window,group,d,n,layers", [
    (torch.bfloat16, 32, 4, 128, 160, 700),        # 3 granules of 64
    (torch.bfloat16, 32, 5, 64, 32 * 64, 160),     # 8 granules of 256, streaming where there are many
    (torch.bfloat16, 32, 6, 128, 33 * 256 - 7, 60),    # 33 granules: one more than a sweep of the pairs
    (torch.bfloat16, 32, 1, 128, 8192, 70),        # 32 granules: one sweep
    (torch.bfloat16, 64, 4, 128, 31 * 256 + 1, 64),    # 32 granules of the software-pipelined form, one key in the last
    (torch.float32, 64, 3, 64, 1999, 160),         # 16 granules of 128
    (torch.float32, 32, 2, 128, 2100, 100),
])
def test_a_layer_alone_scores_to_the_same_bits_as_among_many(dtype, window, group, d, n, layers, peak):
    """A layer alone has its pairs combined inside pass 2, among many by the kernel in between."""
    cake = load_cake()
    say(f"scores alone and among many {dtype} S_w={window} G={group} d={d} N={n} peak={peak}")
    h_kv = 8
    assert _combines(h_kv, dtype, window, group, n) is True
    assert _combines(h_kv * layers, dtype, window, group, n) is False
    q, k, v = _inputs(2, h_kv * group, h_kv, d, n, window, dtype, n, peak)
    many = cake.EvictionPass([q[i % 2] for i in range(layers)], [k[i % 2] for i in range(layers)], [v[i % 2] for i in range(layers)],
                             layers * window)
    assert cake.cake_scores_chunk_keys(many.shape) == _granules(n, window)[0]
    many.scores()
    for l in range(2):
        alone = cake.EvictionPass(q[l:l + 1], k[l:l + 1], v[l:l + 1], window)
        alone.scores()
        assert torch.equal(alone.indicator[0], many.indicator[l])
        assert torch.equal(alone.indicator[0], many.indicator[l + 2 * ((layers - 1 - l) // 2)])
        assert torch.equal(alone.hv[0, 0], many.hv[0, l]) and torch.equal(alone.pref[0, 0], many.pref[0, l])


def _form(names, pass_, group):
    """Which form of a score pass ran: streaming, slices packed by the kernel's last argument, or a wave per head."""
    mine = [n for n in names if f"_pass{pass_}" in n]
    assert len(mine) == 1, names
    if "stream_pass" in mine[0]:
        return "stream"
    m = re.search(r"Li(\d+)EEEv|, (\d+)>\(", mine[0])
    slices = int(m[1] or m[2])
    assert slices in (1, {5: 3, 6: 2}.get(group, 1)), mine
    return "packed" if slices > 1 else "head"


@pytest.mark.parametrize("mode", [0, 2])            # sums of the weights; about a pivot
@pytest.mark.parametrize("window,group,d,h_kv,n,layers,forms", [
    (32, 5, 128, 8, 1025, 60, ("stream", "stream")),     # a tile with one key in its second half, keys past the prefix in the same one
    (32, 5, 128, 8, 4093, 30, ("stream", "stream")),     # whole granules of 256 and a ragged one
    (32, 5, 128, 8, 2100, 19, ("head", "packed")),       # 152 slices: the last workgroup repeats one
    (32, 6, 128, 8, 8231, 28, ("stream", "stream")),
    (32, 6, 128, 9, 16384 + 31, 13, ("packed", "stream")),     # granules of 1024; 117 slices, one repeated
    (32, 6, 128, 9, 225, 17, ("packed", "packed")),
    (32, 5, 64, 8, 4093, 29, ("stream", "stream")),
    (32, 5, 64, 8, 2100, 34, ("head", "packed")),
    (32, 6, 64, 8, 4093, 16, ("packed", "stream")),
    (32, 6, 64, 9, 225, 17, ("packed", "packed")),
    (32, 4, 128, 8, 16384 + 31, 32, ("head", "stream")),
    (32, 4, 128, 8, 4128, 61, ("head", "head")),
    (64, 3, 128, 8, 4093, 25, ("head", "stream")),
    (64, 4, 64, 8, 2047, 29, ("head", "stream")),
])
def test_every_form_of_the_passes_gives_the_bits_of_a_layer_alone(window, group, d, h_kv, n, layers, forms, mode):
    """Launches that stream, or pack slices, against a layer alone with a wave per head, and against the oracle; their queries and
    keys in the order [B, N, H, d], the layer's alone contiguous."""
    cake = load_cake()
    say(f"forms of the score passes S_w={window} G={group} d={d} N={n} layers={layers} mode={mode}")
    q, k, v = _inputs(2, h_kv * group, h_kv, d, n, window, torch.bfloat16, n + group, 6.0)
    tokens_first = lambda xs: [x.transpose(1, 2).contiguous().transpose(1, 2) for x in xs]
    qt, kt, vt = tokens_first(q), tokens_first(k), tokens_first(v)
    params = cake.make_params(indicator_mode=mode)
    many = cake.EvictionPass([qt[i % 2] for i in range(layers)], [kt[i % 2] for i in range(layers)], [vt[i % 2] for i in range(layers)],
                             layers * window, params)
    assert many.k[0].stride(2) == h_kv * d
    names = kernels_of(many.scores)
    assert (_form(names, 1, group), _form(names, 2, group)) == forms, names
    for l in range(2):
        alone = cake.EvictionPass(q[l:l + 1], k[l:l + 1], v[l:l + 1], window, params)
        names = kernels_of(alone.scores)
        assert (_form(names, 1, group), _form(names, 2, group)) == ("head", "head"), names
        assert torch.equal(alone.indicator[0], many.indicator[l])
        assert torch.equal(alone.indicator[0], many.indicator[l + 2 * ((layers - 1 - l) // 2)])
        assert torch.equal(alone.hv[0, 0], many.hv[0, l]) and torch.equal(alone.pref[0, 0], many.pref[0, l])
    want = oracle_layer(q[1][0], k[1][0], params)
    assert_close(many.indicator[1, 0].cpu().numpy(), want["indicator"], "indicator")
    assert_close(many.hv[0, 1].cpu().numpy(), [want["H"], want["V"]], "H, V")


def test_streamed_segments_give_the_bits_of_the_resident_call():
    """Key segments long enough to stream, against the whole layer at once."""
    cake = load_cake()
    layers, h_kv, group, d, n, window = 16, 8, 5, 128, 3 * 8192 + 77, 32
    say(f"streamed segments {layers} layers of {n} keys")
    q, k, v = _inputs(1, h_kv * group, h_kv, d, n, window, torch.bfloat16, 5, 3.0)
    ev = cake.EvictionPass(q * layers, k * layers, v * layers, layers * window)
    ev.scores()
    torch.cuda.synchronize()
    want, want_hv = ev.indicator.clone(), ev.hv.clone()
    ev.workspace.fill_(0xFF)
    ev.indicator.fill_(float("nan"))
    names = kernels_of(lambda: ev.scores_segmented(8192))
    for pass_ in (1, 2):
        assert sum(f"stream_pass{pass_}" in n for n in names) >= 3, names
    assert torch.equal(ev.indicator, want) and torch.equal(ev.hv, want_hv)


def test_streamed_end_of_the_longest_layer():
    """The last segment of a layer of nearly 2^31 keys, whose last workgroup has waves beyond them: the sums of the same keys in
    short segments, and nothing written behind the last granule."""
    from paper_2503_12491_amd import binding as C
    cake = load_cake()
    n, window, group, d = 2**31 - 2048 - 31, 32, 5, 64
    lo, short = 2**31 - 4091 * 2048, 128 * 2048
    say(f"streamed segment [{lo}, {n})")
    q, k, _ = _inputs(1, group, 1, d, n - lo, window, torch.bfloat16, 3, 3.0)
    k = k[0]
    shape, params = C.make_shape(1, 1, group, 1, d, n, window, torch.bfloat16), cake.make_params()
    assert C.cake_scores_chunk_keys(shape) == 2048
    strides = lambda x: [x.stride(i) for i in range(3)]
    ws = [torch.zeros(C.cake_workspace_bytes(shape), dtype=torch.uint8, device=DEV) for _ in range(2)]

    def run(pass_, begin, end, to):
        part = k[:, :, begin - lo:end - lo]
        C.cake_window_scores_segment(shape, params, pass_, begin, end - begin, C.ptr_table(q), C.ptr_table([part]), strides(q[0]), strides(part), to)

    for pass_ in (1, 2):
        names = kernels_of(lambda: run(pass_, lo, n, ws[0]))
        assert len(names) == 1 and f"stream_pass{pass_}" in names[0], names
        for begin in range(lo, n, short):
            run(pass_, begin, min(begin + short, n), ws[1])
        torch.cuda.synchronize()
        assert torch.equal(ws[0], ws[1]), pass_
        if pass_ == 1:
            for w in ws:
                C.cake_window_scores_finish(shape, params, 1, None, w)
