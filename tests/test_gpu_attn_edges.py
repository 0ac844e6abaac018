"""Attention at the edges of its tiles: key counts around the 32-key blocks
and the tiles loaded into LDS (32 keys at head_dim 128, 64 at 64), with NaN
rows before and after K and V so that a read outside the range shows, and
the longest sequence at head_dim 64."""

import numpy as np
import pytest

from oracle import attention as oa
from paper_2606_16135_amd import workloads as W

from _gpu_util import bits_to_f64, compare_attention, require_gpu, to_u16

pytestmark = pytest.mark.gpu


def _single(sc, p, n, hq, hkv, d, dtype, seed, noalloc=False):
    """One call over K/V with 80 NaN rows on both sides; output and lse
    against the oracle."""
    import torch
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    q = torch.randn((n, hq, d), generator=g, device="cuda").to(td)
    kv = torch.full((2, p + n + 160, hkv, d), float("nan"), dtype=td, device="cuda")
    kv[:, 80:80 + p + n] = torch.randn((2, p + n, hkv, d), generator=g, device="cuda").to(td)
    k, v = kv[0, 80:80 + p + n], kv[1, 80:80 + p + n]
    out = torch.full((n, hq, d), float("nan"), dtype=td, device="cuda")
    lse = torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda")
    f = (sc.sc_prefill_attn_noalloc if noalloc else
         sc.sc_prefill_attn if dtype == "bf16" else sc.sc_prefill_attn_f16)
    f(q.data_ptr(), k.data_ptr(), v.data_ptr(), p, n, hq, hkv, d, out.data_ptr(), lse=lse.data_ptr(),
      stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    o_ref, l_ref = oa.attention(bits_to_f64(to_u16(q), dtype), bits_to_f64(to_u16(k), dtype),
                                bits_to_f64(to_u16(v), dtype), [p], [n])
    what = f"P={p} N={n} heads {hq}/{hkv} D={d} {dtype}"
    compare_attention(to_u16(out), o_ref, what, dtype)
    # The row sums are fp32 sums of unrounded probabilities.
    assert np.abs(lse.cpu().numpy() - l_ref).max() <= 1e-5 * (1 + np.abs(l_ref).max()), what


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_key_counts_around_tile_edges(d, dtype):
    sc = require_gpu()
    for i, keys in enumerate([1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191, 193, 255, 257, 321, 385]):
        for n in {1, min(keys, 5), keys}:
            print(f"[edges] D={d} {dtype} keys={keys} N={n}", flush=True)
            _single(sc, keys - n, n, 8, 2, d, dtype, 100 * i + n)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("keys", [20, 32, 65, 90, 96, 150, 215, 280, 345, 410])
def test_reference_moves_in_half_a_tile(keys, dtype):
    """Unsplit calls at head_dim 64 whose last tile has keys in its first
    half only; one of those keys leaves the safe range of one row's sum."""
    sc = require_gpu()
    import torch
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    n, hq, hkv, d = 20, 128, 32, 64
    p = keys - n
    spike = (keys - 1) // 64 * 64                 # first key of the last tile
    assert sc.sc_attn_plan_query([p], [n], hq, hkv)[1] == [1] and keys - spike <= 32
    assert sc.sc_attn_plan_kinds([p], [n], hq, hkv, d)[0] == 0
    print(f"[half tile] keys={keys} N={n} heads {hq}/{hkv} {dtype}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(keys)
    q = (4 * torch.randn((n, hq, d), generator=g, device="cuda")).to(td)
    k = torch.randn((keys, hkv, d), generator=g, device="cuda").to(td)
    v = torch.randn((keys, hkv, d), generator=g, device="cuda").to(td)
    k[spike] = (q[n - 1, ::hq // hkv].float() * 0.75).to(td)
    out = torch.full((n, hq, d), float("nan"), dtype=td, device="cuda")
    f = sc.sc_prefill_attn if dtype == "bf16" else sc.sc_prefill_attn_f16
    f(q.data_ptr(), k.data_ptr(), v.data_ptr(), p, n, hq, hkv, d, out.data_ptr(),
      stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ref, _ = oa.attention(*(bits_to_f64(to_u16(t), dtype) for t in (q, k, v)), [p], [n])
    compare_attention(to_u16(out), ref, f"keys={keys}", dtype)


def test_longest_sequence_head_dim_64():
    """2 GiB of keys less 256 tokens at 8 KV heads x 64 dims: tiles of 64
    keys past the last one would start beyond the signed 32-bit offsets."""
    sc = require_gpu()
    import torch
    hq, hkv, d, n = 32, 8, 64, 4096
    tokens = (1 << 31) // (hkv * d * 2) - 256 - 1
    p = tokens - n
    assert sc.sc_attn_plan_query([p], [n], hq, hkv)[1] == [1]
    q, k, v = W.long_sequence_torch(302, p, n, hq, hkv, d, "cuda")
    out = torch.full((n, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    print(f"[longest] P={p} N={n} heads {hq}/{hkv} D={d}", flush=True)
    sc.sc_prefill_attn(q.data_ptr(), k.data_ptr(), v.data_ptr(), p, n, hq, hkv, d, out.data_ptr(),
                       stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for h in (0, hq - 1):
        g = h // (hq // hkv)
        kg, vg = (bits_to_f64(to_u16(t[:, g:g + 1])) for t in (k, v))
        rows = [(0, i, 0) for i in (0, n - 1)]
        o_ref, _ = oa.attention_rows(bits_to_f64(to_u16(q[:, h:h + 1])), kg, vg, [p], [n], rows)
        for r, (_, i, _) in enumerate(rows):
            compare_attention(to_u16(out)[i, h][None, :], o_ref[r][None, :], f"longest row {i} head {h}")


# One query tile per KV head and more than 16 key splits: (P, N, Hq, Hkv).
MANY_SPLITS = [(4100, 50, 8, 2), (16001, 3, 16, 4), (6000, 60, 8, 4), (9001, 17, 40, 8)]


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (64, "f16"), (128, "bf16"), (128, "f16")])
def test_more_than_16_splits(d, dtype):
    sc = require_gpu()
    for i, (p, n, hq, hkv) in enumerate(MANY_SPLITS):
        splits = sc.sc_attn_plan_query([p], [n], hq, hkv)[1][0]
        assert 16 < splits <= 32 and splits * hkv <= 256, (p, n, splits)
        for noalloc in ([False, True] if dtype == "bf16" else [False]):
            print(f"[splits] D={d} {dtype} P={p} N={n} splits={splits} noalloc={noalloc}", flush=True)
            _single(sc, p, n, hq, hkv, d, dtype, 7000 + i, noalloc)


def _stack(seed, p, n, hq, hkv, d, rc=0.0, dtype="bf16"):
    """A three-layer overlapped stack, every layer against the oracle: merges
    deferred to the next layer's kernel and the last layer's own."""
    sc = require_gpu()
    import torch
    from oracle import kvcache as ok
    from _gpu_util import DevicePool, from_u16, new_active
    L = 3
    wl = W.small_workload(seed, p, n, L, hq, hkv, d, rc_fraction=rc, dtype=dtype)
    pool = W.pool_numpy(wl)
    dp = DevicePool(sc, wl, pool)
    try:
        ins = [W.layer_inputs_numpy(wl, l) for l in range(L)]
        dev = [[from_u16(x, "cuda", wl.dtype) for x in t] for t in ins]
        td = torch.bfloat16 if dtype == "bf16" else torch.float16
        outs = [torch.full((wl.total_q, hq, d), float("nan"), dtype=td, device="cuda") for _ in range(L)]
        slots = [new_active(sc, wl) for _ in range(2)]
        copy = torch.cuda.Stream()
        sc.sc_prefill_stack(dp.handle, dp.table, *([x[i].data_ptr() for x in dev] for i in range(3)),
                            [o.data_ptr() for o in outs], [s[2] for s in slots], hq,
                            compute_stream=torch.cuda.current_stream().cuda_stream, copy_stream=copy.cuda_stream)
        torch.cuda.synchronize()
        for l, (q, kn, vn) in enumerate(ins):
            ka, va = ok.gather_layer(pool, wl.block_ids, wl.cu_blocks, wl.prefix_len, wl.new_len, l)
            kf, vf = ok.append_new(ka, va, kn, vn, wl.prefix_len, wl.new_len)
            ref, _ = oa.attention(*(bits_to_f64(x, dtype) for x in (q, kf, vf)), wl.prefix_len, wl.new_len)
            compare_attention(to_u16(outs[l]), ref, f"layer {l}", dtype)
    finally:
        dp.close()


@pytest.mark.parametrize("d", [64, 128])
def test_more_than_16_splits_in_a_stack(d):
    sc = require_gpu()
    assert sc.sc_attn_plan_query([5000], [21], 16, 4)[1][0] > 16
    _stack(7100, [5000], [21], 16, 4, d)


# Deferred merges of a layer stack: by workgroups of their own, one chunk of
# rows each or up to two, or (too few idle CUs: no groups) by the items'
# workgroups; with at most four splits a row and with more; beside narrow
# items, items of the regular cache, and both.
# (P, N, Hq, Hkv, D, regular-cache fraction, narrow rows, merge groups)
MERGES = [([378], [10], 10, 2, 64, 0, 0, 2), ([378], [10], 10, 2, 128, 0, 0, 4), ([304], [66], 32, 8, 64, 0, 0, 9),
          ([304], [66], 32, 8, 128, 0, 0, 17), ([490], [111], 10, 2, 64, 0, 0, 16), ([847], [53], 10, 2, 128, 0, 0, 16),
          ([616, 323, 694], [150, 71, 110], 32, 8, 128, 0, 32, 64), ([918], [55], 10, 2, 64, 0, 0, 0),
          ([918], [55], 10, 2, 128, 0, 0, 0), ([807, 1250, 1308], [109, 140, 130], 32, 8, 64, 0, 32, 0),
          ([648, 515, 670], [75, 9, 78], 32, 8, 64, 0.25, 64, 21),
          ([336, 450, 484, 109], [27, 20, 63, 90], 32, 8, 64, 0.5, 0, 25),
          ([573, 182, 578, 51, 199, 81], [1, 27, 60, 46, 47, 71], 8, 8, 64, 0.25, 32, 32),
          ([622, 101, 861, 342], [66, 53, 73, 57], 32, 8, 64, 0.5, 32, 0),
          ([299, 379, 429, 422, 667, 197], [9, 72, 85, 86, 2, 72], 32, 8, 64, 0.25, 64, 40),
          ([679, 767, 762, 273], [39, 56, 34, 67], 14, 2, 128, 0.5, 32, 86),
          ([550, 272, 254, 894], [3, 14, 9, 73], 32, 8, 128, 0.25, 64, 99),
          ([221, 844, 675, 91, 593], [69, 82, 54, 80, 25], 32, 8, 128, 0.25, 32, 72),
          ([653, 292, 343, 622, 554], [32, 31, 90, 75, 85], 32, 8, 128, 0.5, 64, 0),
          ([629, 447, 628, 267, 374], [88, 4, 36, 78, 86], 14, 2, 128, 0.25, 0, 64)]


@pytest.mark.parametrize("i", range(len(MERGES)))
def test_deferred_merges(i):
    sc = require_gpu()
    p, n, hq, hkv, d, rc, narrow, groups = MERGES[i]
    rc_keys = [16 * int(rc * (x // 16)) for x in p]
    assert max(sc.sc_attn_plan_query(p, n, hq, hkv, rc_keys=rc_keys)[1]) > 1
    assert sc.sc_attn_plan_kinds(p, n, hq, hkv, d, rc_keys=rc_keys) == (narrow, groups)
    dtype = "f16" if rc and i % 2 else "bf16"
    print(f"[merges] P={p} N={n} heads {hq}/{hkv} D={d} rc={rc} {dtype}", flush=True)
    _stack(7200 + i, p, n, hq, hkv, d, rc, dtype)


# Short turns, alone or as the tail tile of a longer one, over key counts
# around the iterations of a narrow item, with one and several splits: where
# the planner takes narrow items and where it does not.  (N, Hq, Hkv)
NARROW = [(1, 8, 2), (8, 8, 2), (6, 32, 8), (9, 14, 2), (16, 8, 2), (64, 4, 4), (66, 8, 2), (52, 10, 2), (257, 3, 3)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_narrow_items(d, dtype):
    sc = require_gpu()
    for i, (n, hq, hkv) in enumerate(NARROW):
        for p in (0, 31, 64, 127, 128, 129, 255, 257, 500, 513, 1100, 4000):
            print(f"[narrow] D={d} {dtype} P={p} N={n} heads {hq}/{hkv}", flush=True)
            _single(sc, p, n, hq, hkv, d, dtype, 9000 + 100 * i + p)


# Calls that run narrow items (at most 64 rows of a query tile): one and two
# row blocks, a last one of few rows, key counts around their iterations (4
# tiles of 32 keys, or of 64 at head_dim 64), as the tail tile of a longer
# turn (all it has are 2 to 32 rows), one and several splits.
# (N, Hq, Hkv, narrow rows): prefixes
RUN_NARROW = {
    (1, 8, 2, 32): (99, 126, 127, 143, 254, 255, 256, 382, 383, 384, 510, 511, 1100, 4000),
    (8, 8, 2, 32): (92, 120, 136, 247, 248, 249, 375, 377, 504, 1100, 4000),
    (6, 32, 8, 32): (250, 251, 506, 507, 1100, 4000),
    (16, 8, 2, 64): (183, 239, 240, 241, 367, 368, 3057, 4000),
    (9, 14, 2, 64): (190, 246, 247, 248, 374, 375, 4000),
    (40, 4, 4, 64): (159, 215, 216, 217, 344, 2600),
    (60, 8, 8, 64): (139, 195, 196, 197, 324, 451, 452, 4000),
    (66, 8, 2, 32): (33, 61, 62, 77, 189, 190, 191, 205, 4000),
    (257, 3, 3, 32): (0, 23, 1300, 4000),
}


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_calls_that_run_narrow_items(d, dtype):
    sc = require_gpu()
    for (n, hq, hkv, rows), prefixes in RUN_NARROW.items():
        for p in prefixes:
            assert sc.sc_attn_plan_kinds([p], [n], hq, hkv, d)[0] == rows, (p, n, hq, hkv)
            print(f"[run narrow] D={d} {dtype} P={p} N={n} heads {hq}/{hkv}", flush=True)
            _single(sc, p, n, hq, hkv, d, dtype, 12000 + p + n)


# Narrow, unsplit (the last: 16 splits), with one or two row blocks.
# (P, N, Hq, Hkv, narrow rows)
NARROW_VALUES = [(500, 1, 8, 2, 32), (500, 8, 8, 2, 32), (368, 16, 8, 2, 64), (4000, 16, 8, 2, 64)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_narrow_items_move_their_reference(d, dtype):
    """Peaky scores: tile sums that leave the safe range (the reference moves
    within a key group), and key groups whose references differ by more than
    the exponent range of a probability."""
    sc = require_gpu()
    import torch
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    for p, n, hq, hkv, rows in NARROW_VALUES:
        assert sc.sc_attn_plan_kinds([p], [n], hq, hkv, d)[0] == rows
        for name, lean_max in (("growing", 6), ("shrinking", -6), ("growing apart", 200), ("shrinking apart", -200)):
            what = f"{name} P={p} N={n} heads {hq}/{hkv} D={d} {dtype}"
            print(f"[reference] {what}", flush=True)
            g = torch.Generator(device="cuda")
            g.manual_seed(9999)
            q = torch.randn((n, hq, d), generator=g, device="cuda").to(td)
            k = torch.randn((p + n, hkv, d), generator=g, device="cuda")
            # Each key leans towards the queries' mean by an amount that grows
            # (or shrinks) with its position.
            lean = torch.linspace(-lean_max, lean_max, p + n, device="cuda")[:, None, None]
            k = (k + lean * q.float().reshape(n, hkv, hq // hkv, d).mean(dim=(0, 2))[None]).to(td)
            v = torch.randn((p + n, hkv, d), generator=g, device="cuda").to(td)
            q = (q.float() * 4).to(td)
            out = torch.full((n, hq, d), float("nan"), dtype=td, device="cuda")
            f = sc.sc_prefill_attn if dtype == "bf16" else sc.sc_prefill_attn_f16
            f(q.data_ptr(), k.data_ptr(), v.data_ptr(), p, n, hq, hkv, d, out.data_ptr(),
              stream=torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            ref, _ = oa.attention(*(bits_to_f64(to_u16(t), dtype) for t in (q, k, v)), [p], [n])
            compare_attention(to_u16(out), ref, what, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_narrow_items_keep_nan_and_infinity_where_they_belong(d, dtype):
    """A NaN or infinity in one key group's K or V, or in one query row,
    reaches the outputs that the oracle says and no others."""
    sc = require_gpu()
    import torch
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    nan, inf = float("nan"), float("inf")
    for p, n, hq, hkv, rows in NARROW_VALUES:
        assert sc.sc_attn_plan_kinds([p], [n], hq, hkv, d)[0] == rows
        # (tensor, index, value); keys in the first and in a later iteration.
        for t, at, x in (("k", (3, 0, 1), nan), ("k", (p - 40, 1, 2), nan), ("k", (70, 0, 0), inf),
                         ("k", (p - 5, 1, 0), -inf), ("v", (5, 0, 7), inf), ("v", (p - 70, 1, 9), -inf),
                         ("v", (p - 1, 0, 3), nan), ("q", (n - 1, 2, 0), nan)):
            what = f"{t}{list(at)}={x} P={p} N={n} heads {hq}/{hkv} D={d} {dtype}"
            print(f"[nan] {what}", flush=True)
            g = torch.Generator(device="cuda")
            g.manual_seed(9998)
            a = {"q": torch.randn((n, hq, d), generator=g, device="cuda").to(td),
                 "k": torch.randn((p + n, hkv, d), generator=g, device="cuda").to(td),
                 "v": torch.randn((p + n, hkv, d), generator=g, device="cuda").to(td)}
            a[t][at] = x
            out = torch.zeros((n, hq, d), dtype=td, device="cuda")
            f = sc.sc_prefill_attn if dtype == "bf16" else sc.sc_prefill_attn_f16
            f(a["q"].data_ptr(), a["k"].data_ptr(), a["v"].data_ptr(), p, n, hq, hkv, d, out.data_ptr(),
              stream=torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            with np.errstate(invalid="ignore"):
                ref, _ = oa.attention(*(bits_to_f64(to_u16(a[i]), dtype) for i in "qkv"), [p], [n])
            got = bits_to_f64(to_u16(out), dtype)
            finite = np.isfinite(ref)
            assert not finite.all() or t == "k", what   # a score of -inf is a weight of 0
            assert np.array_equal(np.isnan(got), np.isnan(ref)), what
            assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]), what
            compare_attention(np.where(finite, to_u16(out), 0), np.where(finite, ref, 0), what, dtype)
