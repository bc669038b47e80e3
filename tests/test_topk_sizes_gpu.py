"""cake_select_topk at the edges of its kernels: rows that just fit and just exceed each register
kernel, rows long enough for the list in LDS, counts beyond the list, constant and few-valued rows,
row starts at every alignment; against the oracle's ordered selection, exactly."""
import numpy as np
import pytest
import torch

from oracle import cake_oracle as co

from gpu_util import kernels_of, load_cake, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def cake():
    return load_cake()


def _values(kind, heads, n, rng):
    if kind == "pooled":                                          # runs of equal values over many binary exponents
        x = np.exp(3.0 * rng.standard_normal((heads, n)) - 9.0)
        p = np.pad(x, ((0, 0), (3, 3)), constant_values=0.0)
        return np.max([p[:, i: i + n] for i in range(7)], axis=0)
    if kind == "constant":
        return np.full((heads, n), 0.25)
    if kind == "few":                                             # a handful of distinct values, both signs, both zeros
        return rng.choice([-1.0, -0.0, 0.0, 1e-30, 3.0], size=(heads, n))
    if kind == "narrow":                                          # neighbouring floats: every interval but the last rounds is one key
        return 1.0 + rng.integers(0, 40, size=(heads, n)) * 2.0 ** -23
    if kind == "pair":                                            # two neighbouring floats: more than the list of either
        return 1.0 + rng.integers(0, 2, size=(heads, n)) * 2.0 ** -23
    if kind == "zeros":                                           # 0 nearly everywhere, the entries above it anywhere
        return np.where(rng.random((heads, n)) < 0.999, 0.0, rng.random((heads, n)))
    return rng.standard_normal((heads, n)) * 10.0 ** rng.integers(-30, 30, size=(heads, n))     # the whole range of a float


@pytest.mark.parametrize("n,ks", [(1, (1,)), (5, (1, 4, 5)), (129, (1, 64, 128)), (4093, (1, 300, 4092)), (4094, (2000,)),
                                  (16381, (1, 1000)), (16382, (16000,)), (32765, (1048,)), (32766, (5, 31000)),
                                  (65533, (2048, 65532)), (65534, (1, 2048)), (131008, (2048, 14336, 20000, 131007))])
def test_selection_is_the_ordered_top_k(cake, n, ks):
    say(f"top-k of rows of {n}")
    rng = np.random.default_rng(n)
    heads = 4                                                     # odd n: the four rows start at all four alignments
    for kind in ("pooled", "constant", "few", "narrow", "pair", "zeros", "wide"):
        vals = _values(kind, heads, n, rng).astype(np.float32)
        ind = torch.tensor(vals, device=DEV)[None]
        for k in ks:
            idx = torch.full((1, heads, k), -1, dtype=torch.int32, device=DEV)
            shape = cake.make_shape(1, 1, heads, heads, 64, n + 32, 32, torch.float32)
            cake.cake_select_topk(shape, cake.ptr_table([ind]), [n], [k], cake.ptr_table([idx]))
            torch.cuda.synchronize()
            for h in range(heads):
                want = co.select_topk(vals[h].astype(np.float64), k)
                np.testing.assert_array_equal(idx[0, h].cpu().numpy(), want, err_msg=f"{kind} n={n} k={k} head {h}")


@pytest.mark.parametrize("n", [200, 5000, 40000, 70001])
def test_rows_of_nan_with_all_bits_set(cake, n):
    # The smallest keys there are: still entries of the row, kept in order of position behind all numbers.
    say(f"top-k of rows of {n} with NaN of all bits")
    for k in (1, n // 2, n - 1):
        vals = np.random.default_rng(n + k).standard_normal((2, n)).astype(np.float32)
        vals[0] = np.uint32(0xFFFFFFFF).view(np.float32)
        vals[1, n // 3:] = vals[0, 0]
        ind = torch.from_numpy(vals.view(np.int32).copy()).to(DEV).view(torch.float32)[None]
        idx = torch.full((1, 2, k), -1, dtype=torch.int32, device=DEV)
        shape = cake.make_shape(1, 1, 2, 2, 64, n + 32, 32, torch.float32)
        cake.cake_select_topk(shape, cake.ptr_table([ind]), [n], [k], cake.ptr_table([idx]))
        torch.cuda.synchronize()
        np.testing.assert_array_equal(idx[0, 0].cpu().numpy(), np.arange(k))
        want = co.select_topk(np.where(np.isnan(vals[1]), -1e30, vals[1]).astype(np.float64), k)
        np.testing.assert_array_equal(idx[0, 1].cpu().numpy(), want)


@pytest.mark.parametrize("n", [200, 1000, 5000, 40000, 70001])
def test_rows_of_the_largest_key(cake, n):
    # NaN of the bits 0x7fffffff has the largest key there is, and an interval of the search that holds it may reach
    # past the keys' end: the absent entries behind a row are not in it.  More of them than are ranked, beside numbers.
    say(f"top-k of rows of {n} with the largest key")
    for m in (129, 190):
        for k in (1, 100, m, m + 3):
            vals = np.exp(np.random.default_rng(n + k).standard_normal((2, n))).astype(np.float32)
            vals[:, n - m:] = np.uint32(0x7FFFFFFF).view(np.float32)
            vals[1] = vals[1, ::-1]
            ind = torch.from_numpy(vals.view(np.int32).copy()).to(DEV).view(torch.float32)[None]
            idx = torch.full((1, 2, k), -1, dtype=torch.int32, device=DEV)
            shape = cake.make_shape(1, 1, 2, 2, 64, n + 32, 32, torch.float32)
            cake.cake_select_topk(shape, cake.ptr_table([ind]), [n], [k], cake.ptr_table([idx]))
            torch.cuda.synchronize()
            for h in range(2):
                want = co.select_topk(np.where(np.isnan(vals[h]), 1e30, vals[h]).astype(np.float64), k)
                np.testing.assert_array_equal(idx[0, h].cpu().numpy(), want, err_msg=f"m={m} k={k} row {h}")


# the edges between the kernels of up to 16381 entries, which hang on the number of rows as well
@pytest.mark.parametrize("n,layers", [(1021, 1), (1022, 1), (1022, 32), (2045, 1), (2045, 32), (2046, 32), (4094, 2), (6141, 1), (6142, 1),
                                      (8189, 2), (8190, 2), (8190, 17), (16381, 17)])
def test_kernels_of_short_rows(cake, n, layers):
    say(f"top-k of {layers} layers of rows of {n}")
    heads, batch = 3, 3                                           # 9 rows a layer: at most 32 layers, 288 rows, a launch
    rng = np.random.default_rng(n + layers)
    few = min(layers, 2)
    vals = [np.stack([_values(kind, heads, n, rng) for kind in ("pooled", "few", "wide")]).astype(np.float32) for _ in range(few)]
    ind = [torch.tensor(x, device=DEV) for x in vals]
    for k in (1, n // 5, n - 1):
        idx = torch.full((layers, batch, heads, k), -1, dtype=torch.int32, device=DEV)
        shape = cake.make_shape(batch, layers, heads, heads, 64, n + 32, 32, torch.float32)
        cake.cake_select_topk(shape, cake.ptr_table([ind[l % few] for l in range(layers)]), [n] * layers * batch, [k] * layers * batch,
                              cake.ptr_table(list(idx)))
        torch.cuda.synchronize()
        for l in range(few):
            for b in range(batch):
                for h in range(heads):
                    want = co.select_topk(vals[l][b, h].astype(np.float64), k)
                    np.testing.assert_array_equal(idx[l, b, h].cpu().numpy(), want, err_msg=f"n={n} k={k} layer {l} row {b} {h}")
            for again in range(l + few, layers, few):
                assert torch.equal(idx[again], idx[l]), (n, k, again)


@pytest.mark.parametrize("layers,n,threads,slots", [(32, 2000, 512, 1), (33, 2000, 256, 2), (16, 9000, 1024, 4), (17, 9000, 512, 8)])
def test_kernels_of_a_pass_by_its_rows(cake, layers, n, threads, slots):
    """256 rows are 256 and 128 are 128, also where more workgroups write the host's copy of the plan beside them."""
    say(f"top-k of a pass of {layers} x 8 rows of {n}")
    gen = torch.Generator(device=DEV).manual_seed(n)
    k = torch.randn(1, 8, n + 32, 64, device=DEV, generator=gen).bfloat16()
    q = torch.randn(1, 8, 32, 64, device=DEV, generator=gen).bfloat16()
    ev = cake.EvictionPass([q] * layers, [k] * layers, [k] * layers, layers * 128)
    ev.run()
    names = [x for x in kernels_of(ev.run) if "select_topk" in x]
    assert len(names) == 1 and (f"<true, {threads}, {slots}>" in names[0] or f"Li{threads}ELi{slots}E" in names[0]), names
