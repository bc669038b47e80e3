"""The score passes at the sizes where their forms change: element types and row blocks, and launches of a few
workgroups (which combine pass 1's pairs inside pass 2) against launches of many (some of which stream)."""
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
        return False                               # waves that stream do not
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


@pytest.mark.parametrize("mode", [0, 2])            # sums of the weights; about a pivot
@pytest.mark.parametrize("window,group,d,n,layers", [
    (32, 4, 128, 1000, 545),       # 8 x 545 x 968 keys: where groups of four begin to stream
    (32, 5, 128, 32 + 97, 1010),   # a tile with one key in its second half, keys past the prefix in the same one
    (32, 5, 128, 4093, 34),        # whole granules of 256 and a ragged one
    (32, 6, 128, 16384 + 31, 6),   # granules of 1024
    (32, 5, 64, 193, 700),
    (32, 6, 64, 2048, 66),
    (64, 3, 128, 2100, 70),        # pass 2 alone streams
    (64, 4, 64, 193 + 64, 820),
])
def test_waves_that_stream_give_the_bits_of_a_layer_alone(window, group, d, n, layers, mode):
    """Launches beyond the line of the streaming kernels against one layer, which is below it."""
    cake = load_cake()
    say(f"streaming scores S_w={window} G={group} d={d} N={n} layers={layers} mode={mode}")
    h_kv, n_p = 8, n - window
    line = 2048 * (512 if window == 64 else 2048 if group == 4 else 256)
    assert h_kv * n < line <= h_kv * layers * n_p
    q, k, v = _inputs(2, h_kv * group, h_kv, d, n, window, torch.bfloat16, n + group, 6.0)
    params = cake.make_params(indicator_mode=mode)
    many = cake.EvictionPass([q[i % 2] for i in range(layers)], [k[i % 2] for i in range(layers)], [v[i % 2] for i in range(layers)],
                             layers * window, params)
    many.scores()
    for l in range(2):
        alone = cake.EvictionPass(q[l:l + 1], k[l:l + 1], v[l:l + 1], window, params)
        alone.scores()
        assert torch.equal(alone.indicator[0], many.indicator[l])
        assert torch.equal(alone.indicator[0], many.indicator[l + 2 * ((layers - 1 - l) // 2)])
        assert torch.equal(alone.hv[0, 0], many.hv[0, l]) and torch.equal(alone.pref[0, 0], many.pref[0, l])


def test_streamed_segments_give_the_bits_of_the_resident_call():
    """Key segments long enough to stream, against the whole layer at once."""
    cake = load_cake()
    layers, h_kv, group, d, n, window = 16, 8, 5, 128, 3 * 8192 + 77, 32
    say(f"streamed segments {layers} layers of {n} keys")
    q, k, v = _inputs(1, h_kv * group, h_kv, d, n, window, torch.bfloat16, 5, 3.0)
    ev = cake.EvictionPass(q * layers, k * layers, v * layers, layers * window)
    assert layers * h_kv * 8192 >= 2048 * 256
    ev.scores()
    torch.cuda.synchronize()
    want, want_hv = ev.indicator.clone(), ev.hv.clone()
    ev.workspace.fill_(0xFF)
    ev.indicator.fill_(float("nan"))
    ev.scores_segmented(8192)
    torch.cuda.synchronize()
    assert torch.equal(ev.indicator, want) and torch.equal(ev.hv, want_hv)


def test_streamed_end_of_the_longest_layer():
    """The last segment of a layer of nearly 2^31 keys, whose last workgroup has waves beyond them: the sums of the same keys in
    short segments, and nothing written behind the last granule."""
    from paper_2503_12491_amd import binding as C
    cake = load_cake()
    n, window, group, d = 2**31 - 2048 - 31, 32, 5, 64
    lo, short = 2**31 - 4098 * 2048, 128 * 2048
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
