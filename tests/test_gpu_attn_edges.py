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


def _stack(seed, p, n, hq, hkv, d):
    """A three-layer overlapped stack, every layer against the oracle: merges
    deferred to the next layer's kernel and the last layer's own."""
    sc = require_gpu()
    import torch
    from oracle import kvcache as ok
    from _gpu_util import DevicePool, from_u16, new_active
    L = 3
    wl = W.small_workload(seed, p, n, L, hq, hkv, d)
    pool = W.pool_numpy(wl)
    dp = DevicePool(sc, wl, pool)
    try:
        ins = [W.layer_inputs_numpy(wl, l) for l in range(L)]
        dev = [[from_u16(x, "cuda", wl.dtype) for x in t] for t in ins]
        outs = [torch.full((wl.total_q, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(L)]
        slots = [new_active(sc, wl) for _ in range(2)]
        copy = torch.cuda.Stream()
        sc.sc_prefill_stack(dp.handle, dp.table, *([x[i].data_ptr() for x in dev] for i in range(3)),
                            [o.data_ptr() for o in outs], [s[2] for s in slots], hq,
                            compute_stream=torch.cuda.current_stream().cuda_stream, copy_stream=copy.cuda_stream)
        torch.cuda.synchronize()
        for l, (q, kn, vn) in enumerate(ins):
            ka, va = ok.gather_layer(pool, wl.block_ids, wl.cu_blocks, wl.prefix_len, wl.new_len, l)
            kf, vf = ok.append_new(ka, va, kn, vn, wl.prefix_len, wl.new_len)
            ref, _ = oa.attention(bits_to_f64(q), bits_to_f64(kf), bits_to_f64(vf), wl.prefix_len, wl.new_len)
            compare_attention(to_u16(outs[l]), ref, f"layer {l}")
    finally:
        dp.close()


@pytest.mark.parametrize("d", [64, 128])
def test_more_than_16_splits_in_a_stack(d):
    sc = require_gpu()
    assert sc.sc_attn_plan_query([5000], [21], 16, 4)[1][0] > 16
    _stack(7100, [5000], [21], 16, 4, d)


# Deferred merges of a layer stack: by workgroups of their own, one chunk of
# rows each or up to two, or (too few idle CUs) by the items' workgroups; with
# at most four splits a row and with more.  (P, N, Hq, Hkv, D)
MERGES = [([378], [10], 10, 2, 64), ([378], [10], 10, 2, 128), ([304], [66], 32, 8, 64), ([304], [66], 32, 8, 128),
          ([490], [111], 10, 2, 64), ([847], [53], 10, 2, 128), ([616, 323, 694], [150, 71, 110], 32, 8, 128),
          ([918], [55], 10, 2, 64), ([918], [55], 10, 2, 128), ([807, 1250, 1308], [109, 140, 130], 32, 8, 64)]


@pytest.mark.parametrize("i", range(len(MERGES)))
def test_deferred_merges(i):
    p, n, hq, hkv, d = MERGES[i]
    print(f"[merges] P={p} N={n} heads {hq}/{hkv} D={d}", flush=True)
    _stack(7200 + i, p, n, hq, hkv, d)


# Narrow items (at most 64 rows of a query tile): one and two row blocks,
# key counts around their iterations (4 tiles of 32 keys, or of 64 at
# head_dim 64), alone and as the tail tile of a longer turn, one and several
# splits.  (N, Hq, Hkv)
NARROW = [(1, 8, 2), (8, 8, 2), (6, 32, 8), (9, 14, 2), (16, 8, 2), (64, 4, 4), (66, 8, 2), (52, 10, 2), (257, 3, 3)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [64, 128])
def test_narrow_items(d, dtype):
    sc = require_gpu()
    for i, (n, hq, hkv) in enumerate(NARROW):
        for p in (0, 31, 64, 127, 128, 129, 255, 257, 500, 513, 1100, 4000):
            print(f"[narrow] D={d} {dtype} P={p} N={n} heads {hq}/{hkv}", flush=True)
            _single(sc, p, n, hq, hkv, d, dtype, 9000 + 100 * i + p)


def test_narrow_items_move_their_reference():
    """Peaky scores: key groups whose references differ by more than the
    exponent range of a probability, and tile sums that leave the safe range
    (the reference moves within a group)."""
    sc = require_gpu()
    import torch
    p, n, hq, hkv, d = 700, 7, 8, 2, 128
    for name, scale in (("growing", 1.0), ("shrinking", -1.0)):
        g = torch.Generator(device="cuda")
        g.manual_seed(9999)
        q = torch.randn((n, hq, d), generator=g, device="cuda").to(torch.bfloat16)
        k = torch.randn((p + n, hkv, d), generator=g, device="cuda")
        # Each key leans towards the queries' mean by an amount that grows
        # (or shrinks) with its position.
        lean = torch.linspace(-6, 6, p + n, device="cuda")[:, None, None] * scale
        k = (k + lean * q.float().reshape(n, hkv, hq // hkv, d).mean(dim=(0, 2))[None]).to(torch.bfloat16)
        v = torch.randn((p + n, hkv, d), generator=g, device="cuda").to(torch.bfloat16)
        q = (q.float() * 4).to(torch.bfloat16)
        out = torch.full((n, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        sc.sc_prefill_attn(q.data_ptr(), k.data_ptr(), v.data_ptr(), p, n, hq, hkv, d, out.data_ptr(),
                           stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        ref, _ = oa.attention(*(bits_to_f64(to_u16(t)) for t in (q, k, v)), [p], [n])
        compare_attention(to_u16(out), ref, name)
