"""cake_decode_step at the edges of its kernels: caches whose rows just fill and just exceed a chunk, the
longest lists one workgroup per head finishes, and longer ones; through DecodeSlots and through the
binding; against the oracle's update, every buffer."""
import numpy as np
import pytest
import torch

from oracle import cake_oracle as co

from gpu_util import assert_close, host64, load_cake, oracle_params, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STEP_WHOLE_BYTES = 128 << 10      # keys of a head that one workgroup takes in


@pytest.fixture(scope="module")
def cake():
    return load_cake()


def _result(cake, cap, B, H_kv, d, S_w, dtype, gen):
    keep = np.array([[cap if b == 0 else max(cap - 7 * b, 0) for b in range(B)]])
    mk = lambda: torch.randn(B, H_kv, cap + S_w, d, generator=gen).to(dtype).to(DEV)
    ind = torch.exp(torch.randn(B, H_kv, cap, generator=gen) - 6.0).to(DEV)
    return cake.PassResult(keep + S_w, keep, None, None, [], [], [mk()], [mk()], [ind])


@pytest.mark.parametrize("cap,G,d,S_w,dtype,B,pool", [
    (0, 4, 128, 32, "bf16", 1, 7), (1, 1, 64, 32, "bf16", 1, 7), (222, 4, 128, 32, "bf16", 1, 7), (223, 3, 128, 32, "bf16", 2, 7),
    (224, 8, 64, 32, "f32", 1, 13), (1000, 5, 128, 64, "f32", 2, 7), (4063, 4, 128, 32, "bf16", 1, 1), (4064, 4, 128, 32, "bf16", 1, 7),
    (8159, 2, 64, 32, "bf16", 1, 7), (8160, 2, 64, 32, "bf16", 1, 129)])
def test_steps_match_the_oracle_at_every_list_length(cake, cap, G, d, S_w, dtype, B, pool):
    say(f"decode step: {cap} rows, G = {G}, d = {d}, {dtype}, batch {B}")
    H_kv, dt = 2, torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(cap + G)
    res = _result(cake, cap, B, H_kv, d, S_w, dt, gen)
    params = cake.make_params(pool_kernel=pool)
    slots = cake.DecodeSlots(res, G * H_kv, S_w, params)
    plain = cake.DecodeSlots(res, G * H_kv, S_w, params)
    p = oracle_params(params)
    for step in range(3):
        qn = (torch.randn(B, G * H_kv, d, generator=gen) * 2).to(dt).to(DEV)
        kn, vn = (torch.randn(B, H_kv, d, generator=gen).to(dt).to(DEV) for _ in range(2))
        before = [tuple(host64(x) for x in slots.logical(0, b)[:3]) for b in range(B)]
        slots.step(0, qn, kn, vn)
        t = plain.tbl
        cake.cake_decode_step(plain.shape1, params, qn, [0, *qn.stride()[:2]], kn, vn, [0, *kn.stride()[:2]], t["k"], t["v"],
                              plain.slot_strides, t["ind"], t["order"], t["state"], plain.cap, plain.ws)
        torch.cuda.synchronize()
        for name in ("k", "v", "ind", "order", "state"):
            assert torch.equal(getattr(slots, name)[0], getattr(plain, name)[0]), (step, name)
        for b in range(B):
            k0, v0, i0 = before[b]
            cur = i0.shape[1]
            k_full = np.concatenate([k0, host64(kn[b])[:, None]], axis=1)
            upd = co.decode_update(host64(qn[b]), k_full, np.concatenate([i0, np.zeros((H_kv, 1))], axis=1), S_w, p)
            k1, v1, i1, evicted = slots.logical(0, b)
            for g in range(H_kv):
                e = int(evicted[g])
                assert upd[g, e] <= upd[g].min() * (1 + 2e-3)
                sel = np.delete(np.arange(cur + 1), e)
                np.testing.assert_array_equal(host64(k1[g]), co.compact(k_full[g], sel, S_w))
                v_full = np.concatenate([v0[g], host64(vn[b])[g][None]], axis=0)
                np.testing.assert_array_equal(host64(v1[g]), co.compact(v_full, sel, S_w))
                assert_close(host64(i1[g]), upd[g][sel], f"indicator step {step} b={b} g={g}")


@pytest.mark.parametrize("G", [1, 5])
def test_weights_below_the_normal_range_still_order_the_rows(cake, G):
    """Weights of 2^-126 .. 2^-146 are kept: rows whose indicators are still 0 differ by them alone.  A logit's fp32
    rounding at 146 is 1.7e-5 of the weight, the weight's own rounding at most a step of 2^-149."""
    say(f"decode step: weights below 2^-126, G = {G}")
    cap, S_w, d = 40, 32, 64
    log2w = np.random.default_rng(2).permutation(-126.0 - 0.5 * np.arange(cap))
    rows = np.concatenate([log2w, [-130.0], [-200.0] * (S_w - 2), [0.0]])       # the oldest window row leaves; the newest takes all the weight
    k = torch.zeros(1, 1, cap + S_w, d)
    k[0, 0, :, 0] = torch.tensor(rows * np.log(2.0), dtype=torch.float32)
    keep = np.array([[cap]])
    res = cake.PassResult(keep + S_w, keep, None, None, [], [], [k.to(DEV)], [k.to(DEV)], [torch.zeros(1, 1, cap, device=DEV)])
    slots = cake.DecodeSlots(res, G, S_w, cake.make_params(pool_kernel=1))
    q = torch.zeros(1, G, d)
    q[..., 0] = 8.0                                                             # scale 1/8: the logit is the key's first entry
    new = torch.zeros(1, 1, d)
    new[..., 0] = -200.0 * np.log(2.0)
    slots.step(0, q.to(DEV), new.to(DEV), new.to(DEV))
    torch.cuda.synchronize()
    _, _, ind, evicted = slots.logical(0, 0)
    want = np.exp2(rows[:cap + 1])
    e = int(np.argmin(want))
    assert int(evicted[0]) == e
    want = np.delete(want, e)
    assert np.all(np.abs(host64(ind[0]) - want) <= 2.0 ** -149 + 3e-5 * want)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_queries_may_start_at_any_element(cake, dtype):
    """Only the strides of q_new are multiples of 16 bytes: its address is any element's."""
    say(f"decode step: q_new off 16 bytes, {dtype}")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(4)
    G, H_kv, d, S_w, B = 3, 2, 64, 32, 2
    res = _result(cake, 300, B, H_kv, d, S_w, dt, gen)
    q = torch.randn(B, G * H_kv, d, generator=gen).to(dt).to(DEV)
    kn, vn = (torch.randn(B, H_kv, d, generator=gen).to(dt).to(DEV) for _ in range(2))
    want = cake.DecodeSlots(res, G * H_kv, S_w)
    want.step(0, q, kn, vn)
    for off in (1, 3):
        moved = torch.empty(q.numel() + off, dtype=dt, device=DEV)[off:].view(q.shape)
        moved.copy_(q)
        assert moved.data_ptr() % 16 != 0
        got = cake.DecodeSlots(res, G * H_kv, S_w)
        got.step(0, moved, kn, vn)
        torch.cuda.synchronize()
        for name in ("k", "v", "ind", "order", "state"):
            assert torch.equal(getattr(got, name)[0], getattr(want, name)[0]), (off, name)


@pytest.mark.parametrize("L,B,H_kv,G,d,S_w,dtype,cap", [
    (12, 1, 8, 4, 128, 32, "bf16", 1000),      # one call for all layers is large, a layer is not
    (3, 16, 4, 1, 64, 64, "bf16", 767),        # a layer's call is large too, a sequence alone is not
    (3, 5, 8, 6, 64, 32, "f32", 1400),
    (2, 2, 8, 8, 128, 32, "bf16", 4063),       # 4096 rows: the longest lists of the small form
    (3, 9, 4, 4, 64, 32, "bf16", 8300)])       # lists longer than a workgroup holds (8192 rows) beside others that are not
def test_a_step_is_the_same_whatever_else_the_call_holds(cake, L, B, H_kv, G, d, S_w, dtype, cap):
    """Every buffer of a call for all layers equals that of calls layer by layer, and every sequence's rows those of a
    batch of one, bit for bit: calls of more than 256 workgroups of 256 rows, and calls of fewer, which take 64 rows each."""
    say(f"decode step alone and among others: L={L} B={B} H_kv={H_kv} G={G} d={d} S_w={S_w} {dtype} {cap} rows")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    workgroups = lambda layers, batch: -(-(cap + S_w + 1) // 256) * layers * batch * H_kv
    assert workgroups(L, B) > 256 >= workgroups(1, 1)
    gen = torch.Generator().manual_seed(cap + L)
    keep = np.array([[max(cap - 90 * l - 7 * b, 1) for b in range(B)] for l in range(L)])
    mk = lambda l: torch.randn(B, H_kv, int(keep[l].max()) + S_w, d, generator=gen).to(dt).to(DEV)
    k, v = [mk(l) for l in range(L)], [mk(l) for l in range(L)]
    ind = [torch.exp(torch.randn(B, H_kv, int(keep[l].max()), generator=gen) - 6.0).to(DEV) for l in range(L)]

    def slots(b=slice(None)):
        kept = keep[:, b]
        cut = lambda t, extra: [x[b, :, : int(kept[l].max()) + extra] for l, x in enumerate(t)]
        return cake.DecodeSlots(cake.PassResult(kept + S_w, kept, None, None, [], [], cut(k, S_w), cut(v, S_w), cut(ind, 0)), G * H_kv, S_w)

    together, by_layer, alone = slots(), slots(), [slots(slice(b, b + 1)) for b in range(B)]
    for step in range(3):
        qn = (torch.randn(L, B, G * H_kv, d, generator=gen) * 2).to(dt).to(DEV)
        kn, vn = (torch.randn(L, B, H_kv, d, generator=gen).to(dt).to(DEV) for _ in range(2))
        together.step_all(qn, kn, vn)
        for l in range(L):
            by_layer.step(l, qn[l], kn[l], vn[l])
            for b in range(B):
                alone[b].step(l, qn[l, b:b + 1], kn[l, b:b + 1], vn[l, b:b + 1])
        for l in range(L):
            for name in ("k", "v", "ind", "order", "state"):
                assert torch.equal(getattr(together, name)[l], getattr(by_layer, name)[l]), (step, l, name)
            for b in range(B):
                for x, y in zip(by_layer.logical(l, b), alone[b].logical(l, 0)):
                    assert np.array_equal(x, y) if isinstance(x, np.ndarray) else torch.equal(x, y), (step, l, b)


@pytest.mark.parametrize("G,d,S_w,dtype,B,pool", [(4, 128, 32, "bf16", 1, 7), (5, 128, 64, "bf16", 2, 129), (8, 64, 32, "bf16", 3, 13),
                                                  (1, 128, 32, "f32", 1, 7), (7, 64, 64, "f32", 2, 1)])
def test_short_lists_in_one_launch_equal_two(cake, G, d, S_w, dtype, B, pool):
    """A call whose longest list is short does the step in one launch, beside a longer list in two: the same bits in every
    buffer, at the edges of a wave's 64 rows, of 256 and of the longest list the one launch takes (counted with the window and the new row)."""
    dt, eb = (torch.bfloat16, 2) if dtype == "bf16" else (torch.float32, 4)
    longest = min(STEP_WHOLE_BYTES // (d * eb), 1024)
    rows = [S_w + 1, S_w + 2, 127, 128, 129, 256, 257, longest - 1, longest, longest + 1, longest + 700]
    caps = sorted({r - S_w - 1 for r in rows if r > S_w})
    say(f"decode step in one launch and in two: G={G} d={d} S_w={S_w} {dtype} batch {B}, rows {rows}")
    gen = torch.Generator().manual_seed(G + d)
    H_kv, L = 2, len(caps)
    keep = np.array([[max(c - 5 * b, 0) for b in range(B)] for c in caps])
    mk = lambda c: torch.randn(B, H_kv, c + S_w, d, generator=gen).to(dt).to(DEV)
    res = cake.PassResult(keep + S_w, keep, None, None, [], [], [mk(c) for c in caps], [mk(c) for c in caps],
                          [torch.exp(torch.randn(B, H_kv, c, generator=gen) - 6.0).to(DEV) for c in caps])
    together, by_layer = (cake.DecodeSlots(res, G * H_kv, S_w, cake.make_params(pool_kernel=pool)) for _ in range(2))
    for step in range(4):
        qn = (torch.randn(L, B, G * H_kv, d, generator=gen) * 2).to(dt).to(DEV)
        kn, vn = (torch.randn(L, B, H_kv, d, generator=gen).to(dt).to(DEV) for _ in range(2))
        together.step_all(qn, kn, vn)
        for l in range(L):
            by_layer.step(l, qn[l], kn[l], vn[l])
        torch.cuda.synchronize()
        for l in range(L):
            for name in ("k", "v", "ind", "order", "state"):
                assert torch.equal(getattr(together, name)[l], getattr(by_layer, name)[l]), (step, caps[l], name)
