"""Kernel variants that the dispatch picks by size or geometry, at the sizes where each can go
wrong (tile edges, remainders, the smallest call), against the fp64 oracle."""

import pytest

from test_gpu_prefill import _prefill_case

pytestmark = pytest.mark.gpu


# 8 query heads per KV head on MFMA: a q-tile is 32 rows at head_dim 64 / 128 and two sets of 4
# heads by 32 rows at 256.
GROUP8_CASES = [
    # dtype, D, Hq, Hkv, ctx_lens, chunk, q sigma_log2, needle divisor, windows
    ("bf16", 64, 8, 1, [0, 63], 33, -1, 0, (0, 0)),
    ("bf16", 128, 16, 2, [64, 5], 1, -1, 0, (0, 40)),
    ("bf16", 128, 8, 1, [130], 97, 2, 2, (0,)),            # harsh needles
    ("bf16", 256, 16, 2, [0, 500], 65, -1, 0, (0, 100)),
    ("bf16", 256, 8, 1, [77], 31, 2, 2, (0,)),
    ("fp8", 256, 8, 1, [64], 32, -1, 0, (0,)),
    ("fp8", 128, 16, 2, [0, 31], 64, -1, 0, (0, 33)),
    ("fp8", 64, 8, 1, [200], 5, -1, 0, (0,)),
    # several 512-key segments: boundaries inside the chunk, windows starting inside a segment
    ("bf16", 128, 8, 1, [1023, 511], 2, -1, 0, (0, 600)),
    ("bf16", 256, 8, 1, [1100], 40, -1, 0, (0, 513)),
]


@pytest.mark.parametrize("dtype,D,Hq,Hkv,ctxs,chunk,qsig,div,windows", GROUP8_CASES)
def test_group8_prefill(dtype, D, Hq, Hkv, ctxs, chunk, qsig, div, windows):
    _prefill_case(dtype, D, Hq, Hkv, ctxs, chunk, qsig, windows, div)


# fp32 caches: tiles of 32 (row, head) pairs, key blocks of 32, waves of 128, splits of 512
F32_CASES = [
    (64, 4, 2, [0, 31], 1, -1, 0, (0, 0)),
    (64, 2, 2, [511, 100], 33, -1, 0, (0, 40)),
    (128, 8, 1, [512], 65, 2, 2, (0,)),
    (128, 8, 2, [127, 128], 17, -1, 0, (0, 150)),
    (256, 4, 1, [1100], 40, -1, 0, (0, 513)),
    (256, 8, 1, [0, 30], 31, 2, 2, (0,)),
]


@pytest.mark.parametrize("D,Hq,Hkv,ctxs,chunk,qsig,div,windows", F32_CASES)
def test_f32_prefill(D, Hq, Hkv, ctxs, chunk, qsig, div, windows):
    _prefill_case("f32", D, Hq, Hkv, ctxs, chunk, qsig, windows, div)


def test_f32_prefill_unit_per_workgroup():
    # one layer's call is small (a workgroup per 128 keys), the same layer among others is not
    import numpy as np
    import torch

    from paper_2607_14431_amd import kvg
    D, Hq, Hkv, ctx, chunk, L = 128, 8, 4, 1100, 40, 8
    windows = tuple(100 * i for i in range(L))
    g = torch.Generator(device="cuda").manual_seed(5)
    n_pages = (ctx + chunk + 15) // 16
    cache = kvg.Cache.allocate(L, n_pages, Hq, Hkv, D, torch.float32, windows=windows)
    cache.k_pool.normal_(generator=g)
    cache.v_pool.normal_(generator=g)
    table = torch.randperm(n_pages, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()[None]
    seqs = kvg.Seqs(table, torch.tensor([ctx], dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda"), ctx)
    q, k, v = (torch.randn((L, 1, chunk, h, D), device="cuda", generator=g) for h in (Hq, Hkv, Hkv))
    rp = kvg.rope(10000.0, kvg.KVG_ROPE_HALF)

    def run(l0, n, ws_bytes=None):
        out = torch.empty((n, 1, chunk, Hq, D), device="cuda")
        ws_bytes = ws_bytes or kvg.kvg_prefill_workspace_bytes(cache, seqs, n, chunk)
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
        s = slice(l0, l0 + n)
        kvg.kvg_prefill_attn(cache, seqs, rp, l0, n, chunk, q[s], k[s], v[s], 1.0 / np.sqrt(D), out, ws)
        return out

    together = run(0, L)
    for layer in range(L):
        assert torch.equal(run(layer, 1)[0], together[layer])
    # a workspace without room for the units' partials: one partial per split and row
    rows, splits = chunk * Hq, (ctx + chunk + 511) // 512
    small = rows * D * 4 + rows * splits * (D + 2) * 4
    assert small % 256 == 0 and small < kvg.kvg_prefill_workspace_bytes(cache, seqs, 1, chunk)
    assert torch.equal(run(3, 1, small)[0], together[3])
    with pytest.raises(kvg.KvgError):
        run(3, 1, small - 1)


# Small fp32 calls take two (row, head) pairs a workgroup on the vector ALUs: the bytes of the same rows in a call of
# 32-pair tiles.  Odd pair counts, blocks and units partly and wholly masked, one unit (no combine) and several.
@pytest.mark.parametrize("D,Hq,Hkv", [(64, 4, 2), (64, 3, 3), (128, 8, 1), (128, 4, 2), (256, 2, 2), (256, 8, 1)])
@pytest.mark.parametrize("window", [0, 1, 40, 200])
def test_f32_prefill_pairs_are_tiles(D, Hq, Hkv, window):
    import torch

    from paper_2607_14431_amd import kvg
    G, long = Hq // Hkv, 400
    for ctx in (0, 30, 31, 97, 127, 128, 300, 505):
        n_pages = (ctx + long + 15) // 16
        g = torch.Generator(device="cuda").manual_seed(ctx)
        cache = kvg.Cache.allocate(1, n_pages, Hq, Hkv, D, torch.float32, windows=(window,))
        for pool in (cache.k_pool, cache.v_pool):
            pool.normal_(generator=g)
            pool[:, ctx // 16 + 1:] = float("nan")        # nothing beyond the chunk is read into a result
        table = torch.arange(n_pages, dtype=torch.int32, device="cuda")[None]
        seqs = kvg.Seqs(table, torch.tensor([ctx], dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda"), ctx)
        q, k, v = (torch.randn((1, 1, long, h, D), device="cuda", generator=g) for h in (Hq, Hkv, Hkv))

        def run(rows):
            units = (ctx + rows + 127) // 128
            assert (2 * Hkv * ((rows * G + 1) // 2) * units + 64 * units <= {64: 1152, 128: 640, 256: 1024}[D]) == (rows < long)
            out = torch.full((1, 1, rows, Hq, D), float("nan"), device="cuda")
            ws = torch.empty(kvg.kvg_prefill_workspace_bytes(cache, seqs, 1, rows), dtype=torch.uint8, device="cuda")
            kvg.kvg_prefill_attn(cache, seqs, kvg.rope(), 0, 1, rows, *(x[:, :, :rows].contiguous() for x in (q, k, v)), 3.0 * D ** -0.5, out, ws)
            return out

        small = [(rows, run(rows)) for rows in (1, 2, 5, 7)]
        together = run(long)
        assert torch.isfinite(together).all()
        for rows, out in small:
            assert torch.equal(out, together[:, :, :rows]), (ctx, rows)


# The comparison's single pass: a wave, 4 and 16 waves a row, rows read as vectors and element by element, fewer elements
# than lanes, references that have to be raised (spread > e^300), infinities.
@pytest.mark.parametrize("rows,V,scale", [(1, 1, 1.0), (3, 7, 1.0), (2, 64, 1.0), (3, 4095, 5.0), (2, 4100, 5.0),
                                          (2, 33_000, 300.0), (1, 10_001, 2000.0), (5, 512, 5.0),
                                          (2, 513, 300.0), (6, 511, 2000.0), (2, 12_288, 5.0), (2, 12_289, 5.0)])
def test_logit_compare_pass(rows, V, scale):
    import numpy as np
    import torch

    from oracle.logits import argmax, kl_divergence, log_softmax
    from paper_2607_14431_amd import harness as h
    rng = np.random.default_rng(V)
    a = (rng.normal(size=(rows, V)) * scale).astype(np.float32)
    b = (a + rng.normal(size=(rows, V)) * 0.1).astype(np.float32)
    kl, ia, ib = h.compare_logits(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda())
    want = kl_divergence(a.astype(np.float64), b.astype(np.float64))
    # T / A and lse_a - lse_b are each off by at most gamma_V of their terms' magnitudes (u = 2^-53):
    # sum p |a - b| and |max| + log V for the two references and logarithms
    p = np.exp(log_softmax(a.astype(np.float64)))
    mag = (p * np.abs(a.astype(np.float64) - b)).sum(axis=1) + np.abs(a).max(axis=1) + np.abs(b).max(axis=1) + np.log(V)
    assert np.all(np.abs(kl - want) <= 4 * (V + 16) * 2.0 ** -53 * mag)
    assert np.array_equal(ia, argmax(a)) and np.array_equal(ib, argmax(b))


def test_logit_compare_special_values():
    import numpy as np
    import torch

    from paper_2607_14431_amd import harness as h
    inf = np.inf
    a = np.array([[-inf] * 8, [1, 2, -inf, 0, 0, 0, 0, 0], [1, 2, 3, 4, 5, 6, 7, 7], [np.nan] * 8, [1, inf, 0, 0, 0, 0, 0, 0],
                  [3, 1, 2, 0, 0, 0, 0, 0]], np.float32)
    b = np.array([[0] * 8, [1, 2, 0, 0, 0, 0, 0, 0], [1, 2, 3, 4, 5, 6, 7, 7], [0] * 8, [1, 2, 0, 0, 0, 0, 0, 0],
                  [3, -inf, 2, 0, 0, 0, 0, 0]], np.float32)
    kl, ia, ib = h.compare_logits(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda())
    assert np.isnan(kl[[0, 1, 3, 4]]).all() and kl[2] == 0.0 and kl[5] == inf
    assert list(ia) == [0, 1, 6, 8, 1, 0] and list(ib) == [0, 1, 6, 0, 1, 0]


# Decode of bf16 and fp8 caches: units of 128 keys, splits of 512, windows that start inside a page
# and a unit; groups of 1 to 8 heads.  Small calls take a wave per unit.
DECODE_CASES = [
    # dtype, D, Hq, Hkv, ctx_lens, steps, windows
    ("bf16", 256, 2, 1, [126, 127, 128], 3, (0, 0)),
    ("bf16", 64, 4, 2, [0, 15, 640], 2, (0, 127)),
    ("bf16", 128, 2, 2, [511, 1151], 3, (0, 513)),
    ("fp8", 256, 8, 1, [129, 1030], 2, (0, 128)),
    ("fp8", 128, 4, 1, [255, 31], 2, (0, 17)),
    ("fp8", 64, 16, 2, [639, 383], 2, (0, 600)),
    # windows of whole splits that start inside a page: the last unit holds up to 143 keys
    ("bf16", 256, 2, 1, [520, 1037, 1200], 3, (1024, 512)),
    ("bf16", 64, 4, 2, [1039, 523], 2, (512, 1024)),
    ("bf16", 128, 8, 1, [1036], 2, (512, 128)),
    ("fp8", 256, 4, 2, [1550, 527], 2, (1536, 512)),
    ("fp8", 64, 8, 1, [1033, 1023], 2, (512, 1024)),
    ("f32", 64, 4, 2, [1033, 700], 2, (512, 513)),
]


@pytest.mark.parametrize("dtype,D,Hq,Hkv,ctxs,steps,windows", DECODE_CASES)
def test_decode_units(dtype, D, Hq, Hkv, ctxs, steps, windows):
    from test_gpu_prefill import _decode_case
    _decode_case(dtype, D, Hq, Hkv, ctxs, steps, windows)


@pytest.mark.parametrize("B", [12, 16])
@pytest.mark.parametrize("dtype,D,window", [("bf16", 256, 0), ("bf16", 256, 700), ("bf16", 128, 700), ("bf16", 64, 100), ("fp8", 256, 100),
                                            ("fp8", 128, 0), ("fp8", 64, 700)])
def test_decode_wave_per_unit_is_wave_per_split(dtype, D, window, B):
    """B sequences together take a wave per split (rows of 256 bytes and more: with 12 sequences two stages in flight,
    with 16 three), each alone a wave per 128-key unit, or, in a call of its own length below 256 keys, a wave per
    split that needs no merge.  Same bytes, for contexts of one unit to many splits."""
    import torch

    from gpu_helpers import TORCH_DTYPE
    from paper_2607_14431_amd import kvg
    L, Hq, Hkv, long = 2, 8, 4, 9000
    ctxs = [0, 100, 130, 511, 512, long, 255, 256, 127, 1023, 1200, 3000][:B] + [600] * (B - 12)
    per_seq = (long + 16) // 16
    g = torch.Generator(device="cuda").manual_seed(D + window)
    cache = kvg.Cache.allocate(L, B * per_seq, Hq, Hkv, D, TORCH_DTYPE[dtype], windows=(window, 0))
    for pool in (cache.k_pool, cache.v_pool):
        pool.copy_((torch.randn(pool.shape, generator=g, device="cuda") * 0.5).to(pool.dtype))
    tables = torch.randperm(B * per_seq, generator=g, device="cuda").to(torch.int32).view(B, per_seq)
    lens = torch.tensor(ctxs, dtype=torch.int32, device="cuda")
    start = torch.full((B,), 777, dtype=torch.int64, device="cuda")
    raw = [torch.randn((L, B, 1, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv)]

    def splits(n_seqs, max_ctx):                      # of the call: a windowed layer's are those its window touches
        n = (max_ctx + 512) // 512
        return n_seqs * Hkv * (n + (min(n, (window + 511) // 512) if window else n))

    def decode(rows, max_ctx):
        seqs = kvg.Seqs(tables[rows].contiguous(), lens[rows].contiguous(), start[rows].contiguous(), max_ctx)
        out = torch.full((L, len(rows), 1, Hq, D), float("nan"), device="cuda")
        ws = kvg.decode_workspace(cache, seqs, L)
        kvg.kvg_decode_attn(cache, seqs, kvg.rope(), 0, L, *(t[:, rows].contiguous() for t in raw), D ** -0.5, out, ws)
        return out

    row_bytes = D * cache.k_pool.element_size()
    resident = 1280 if row_bytes >= 256 else 2560     # one-wave workgroups
    n = splits(B, long)
    assert n * 4 > resident >= splits(1, long) * 4
    assert row_bytes < 256 or (768 < n < 2304 and 0 < n % 768 <= 256) == (B == 12)
    together = decode(list(range(B)), long)
    assert torch.isfinite(together).all()
    for b in range(B):
        want = together[:, b:b + 1].view(torch.int32)
        assert torch.equal(want, decode([b], long).view(torch.int32)), f"context {ctxs[b]}"
        assert torch.equal(want, decode([b], ctxs[b]).view(torch.int32)), f"context {ctxs[b]} in a call of its length"


# A shared window: the other splits of a small call take a wave per unit, of a larger one a wave per split (each row has
# a partial per shared split, four or one per other split).  Same bytes, for own keys of no whole unit to three splits.
@pytest.mark.parametrize("dtype,D,Hq,Hkv", [("bf16", 256, 4, 2), ("bf16", 128, 8, 2), ("fp8", 256, 2, 2), ("fp8", 64, 8, 2)])
def test_decode_beside_shared_splits(dtype, D, Hq, Hkv):
    import torch

    from gpu_helpers import TORCH_DTYPE
    from paper_2607_14431_amd import kvg
    L, B, shared = 48, 4, 1100 // 16 * 16
    ctxs = [2600, shared + 1, 1500, 1024 + 200]
    n_sh, per = shared // 16, max(ctxs) // 16 + 1
    g = torch.Generator(device="cuda").manual_seed(D)
    n_pages = n_sh + B * (per - n_sh)
    cache = kvg.Cache.allocate(L, n_pages, Hq, Hkv, D, TORCH_DTYPE[dtype])
    for pool in (cache.k_pool, cache.v_pool):
        pool.copy_((torch.randn(pool.shape, generator=g, device="cuda") * 0.5).to(pool.dtype))
    perm = torch.randperm(n_pages, generator=g, device="cuda").to(torch.int32)
    tables = torch.stack([torch.cat([perm[:n_sh], perm[n_sh + b * (per - n_sh):n_sh + (b + 1) * (per - n_sh)]]) for b in range(B)])
    seqs = kvg.Seqs(tables, torch.tensor(ctxs, dtype=torch.int32, device="cuda"), torch.zeros(B, dtype=torch.int64, device="cuda"),
                    max(ctxs), shared)
    plain = kvg.Seqs(seqs.block_tables, seqs.ctx_lens, seqs.start_pos, max(ctxs))
    raw = [torch.randn((L, B, 1, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv)]

    def decode(l0, n, ws_bytes=None, s=seqs):
        out = torch.full((n, B, 1, Hq, D), float("nan"), device="cuda")
        ws = torch.empty(ws_bytes or kvg.kvg_decode_workspace_bytes(cache, s, n), dtype=torch.uint8, device="cuda")
        kvg.kvg_decode_attn(cache, s, kvg.rope(), l0, n, *(t[l0:l0 + n] for t in raw), D ** -0.5, out, ws)
        return out

    own = (max(ctxs) + 512) // 512 - shared // 512
    limit = 1280 if D * cache.k_pool.element_size() >= 256 else 2560
    assert 2 * B * Hkv * own * 4 <= limit < L * B * Hkv * own * 4
    together = decode(0, L)
    assert torch.isfinite(together).all()
    for l0 in (0, 7, L - 2):
        assert torch.equal(decode(l0, 2), together[l0:l0 + 2])
    # room for one partial a split only
    rows, splits = 2 * B * Hq, (max(ctxs) + 512) // 512
    up = lambda x: -(-x // 256) * 256
    small = max(up(rows * splits * 8) + up(rows * splits * D * 4) + 2 * up(rows * D * 2), kvg.kvg_decode_workspace_bytes(cache, plain, 2))
    assert torch.equal(decode(7, 2, small), together[7:9])
    # attended per sequence: the shared splits' bf16 weights apart (2^-9 each)
    alone = decode(7, 2, s=plain)
    assert ((alone - together[7:9]).norm() / alone.norm()).item() < 4e-3


# An append of many values a token requests a thread's first items together, of few one after the other: a head's rows
# are the same bytes among others and alone.  More items than lanes, layers of several to a workgroup.
@pytest.mark.parametrize("dtype", ["bf16", "fp8", "f32"])
@pytest.mark.parametrize("D,Hkv", [(64, 40), (128, 9), (256, 17)])
@pytest.mark.parametrize("pairing", [0, 1])
def test_append_of_a_head_among_others(dtype, D, Hkv, pairing):
    import torch

    from gpu_helpers import INT_VIEW, TORCH_DTYPE
    from paper_2607_14431_amd import kvg
    L, n = 7, 1500                                    # L n > 8192: two layers a workgroup
    n_pages = (n + 15) // 16
    g = torch.Generator(device="cuda").manual_seed(D)
    table = torch.randperm(n_pages, generator=g, device="cuda").to(torch.int32)[None]
    seqs = kvg.Seqs(table, torch.zeros(1, dtype=torch.int32, device="cuda"), torch.full((1,), 33, dtype=torch.int64, device="cuda"), 0)
    wide = kvg.Cache.allocate(L, n_pages, Hkv, Hkv, D, TORCH_DTYPE[dtype])
    k, v = (torch.randn((L, 1, n, Hkv, D), generator=g, device="cuda").to(wide.raw_dtype) for _ in range(2))
    assert Hkv * D * k.element_size() > 128 * 16 >= D * k.element_size()
    kvg.kvg_append(wide, seqs, kvg.rope(10000.0, pairing), 0, L, n, k, v)
    for h in (0, 1, Hkv // 2, Hkv - 1):
        one = kvg.Cache.allocate(L, n_pages, 1, 1, D, TORCH_DTYPE[dtype])
        kvg.kvg_append(one, seqs, kvg.rope(10000.0, pairing), 0, L, n, *(t[:, :, :, h:h + 1].contiguous() for t in (k, v)))
        for a, b in ((wide.k_pool, one.k_pool), (wide.v_pool, one.v_pool)):
            for page in (0, n // 32):                 # whole pages of the sequence
                at = int(table[0, page])
                assert torch.equal(a.view(INT_VIEW[dtype])[:, at, h], b.view(INT_VIEW[dtype])[:, at, 0]), (h, page)


# Two waves per 64 leaves (up to 512 x 64 leaves of equal length): one set and two sets a workgroup, partial
# sets, one and several blocks; a ragged last leaf and one leaf too many take a lane per leaf
@pytest.mark.parametrize("n,leaf,short", [(1, 64, 0), (65, 128, 0), (65, 128, 9), (16_384, 64, 0), (16_385, 64, 0),
                                          (32_767, 64, 0), (32_768, 64, 64), (32_769, 64, 0)])
def test_few_leaves(n, leaf, short):
    import hashlib

    import numpy as np
    import torch

    from paper_2607_14431_amd import kvg
    data = np.random.default_rng(n).integers(0, 256, size=n * leaf - short, dtype=np.uint8)
    got = torch.zeros(((n * leaf - short + leaf - 1) // leaf, 32), dtype=torch.uint8, device="cuda")
    kvg.kvg_leaf_digests(torch.from_numpy(data).cuda(), leaf, got)
    raw = data.tobytes()
    want = [hashlib.sha256(raw[i:i + leaf]).digest() for i in range(0, len(raw), leaf)]
    assert got.cpu().numpy().tobytes() == b"".join(want)


# Subtrees of 512 nodes (odd counts at every level, one launch, two, three) and one level first
@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 1023, 1025, 131_072, 131_073, 262_145, 300_001])
def test_merkle_subtrees(n):
    import numpy as np
    import torch

    from oracle.digest import merkle_root
    from paper_2607_14431_amd import kvg
    leaves = np.random.default_rng(n).integers(0, 256, size=(n, 32), dtype=np.uint8)
    root = torch.zeros(32, dtype=torch.uint8, device="cuda")
    ws = torch.empty(kvg.kvg_merkle_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    kvg.kvg_merkle_root(torch.from_numpy(leaves).cuda(), n, root, ws)
    assert root.cpu().numpy().tobytes() == merkle_root(leaves)


def test_decode_workspace_serves_windowed_caches():
    # the size asked for without windows is enough with them (12B-class stack, 5 of 6 layers windowed)
    import torch

    from paper_2607_14431_amd import kvg
    for dtype in (torch.bfloat16, torch.float8_e4m3fn, torch.float32):
        for layers, ctx in ((1, 100), (6, 5000), (48, 4672)):
            seqs = kvg.Seqs(torch.zeros((1, 400), dtype=torch.int32, device="cuda"),
                            torch.tensor([ctx], dtype=torch.int32, device="cuda"),
                            torch.zeros(1, dtype=torch.int64, device="cuda"), ctx)
            sizes = [kvg.kvg_decode_workspace_bytes(kvg.Cache.allocate(layers, 1, 4, 2, 64, dtype, windows=w), seqs, layers)
                     for w in (None, tuple(0 if (i + 1) % 6 == 0 else 1024 for i in range(layers)))]
            assert sizes[0] == sizes[1] > 0


def test_decode_merge_grid_of_many_rows():
    """More rows (layers x sequences x query heads) than fit a grid of 1,024-lane workgroups, over more
    than 16 splits: the call runs, and a slice of its layers on its own gives the same bytes."""
    import torch

    from paper_2607_14431_amd import kvg
    L, Hq, Hkv, D, ctx, max_ctx = 1 << 19, 8, 1, 64, 700, 8192
    assert L * Hq * 1024 > 2 ** 32 - 1 >= L * Hq * 256
    g = torch.Generator(device="cuda").manual_seed(3)
    cache = kvg.Cache.allocate(L, 2, Hq, Hkv, D, torch.bfloat16)
    for pool in (cache.k_pool, cache.v_pool):
        pool.normal_(generator=g)
    # the new token's page is no other key's
    table = torch.zeros((1, max_ctx // 16 + 1), dtype=torch.int32, device="cuda")
    table[0, ctx // 16] = 1
    seqs = kvg.Seqs(table, torch.tensor([ctx], dtype=torch.int32, device="cuda"),
                    torch.zeros(1, dtype=torch.int64, device="cuda"), max_ctx)
    q, k, v = (torch.randn((L, 1, 1, h, D), generator=g, device="cuda", dtype=torch.bfloat16) for h in (Hq, Hkv, Hkv))

    def decode(l0, n):
        out = torch.full((n, 1, 1, Hq, D), float("nan"), device="cuda")
        ws = kvg.decode_workspace(cache, seqs, n)
        s = slice(l0, l0 + n)
        kvg.kvg_decode_attn(cache, seqs, kvg.rope(), l0, n, q[s], k[s], v[s], D ** -0.5, out, ws)
        return out

    together = decode(0, L)
    assert torch.isfinite(together).all()
    for l0 in (0, L // 2 - 1, L - 2):
        assert torch.equal(decode(l0, 2), together[l0:l0 + 2])


def test_logit_compare_of_many_rows():
    """More rows than fit a grid of 1,024-lane workgroups (2^22 of them): every row is compared."""
    import torch

    from paper_2607_14431_amd import kvg
    rows, V = (1 << 22) + 3, 2
    a = torch.randn((rows, V), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    b = a.flip(1).contiguous()
    kl = torch.full((rows,), float("nan"), dtype=torch.float64, device="cuda")
    ia, ib = (torch.full((rows,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    kvg.kvg_logit_compare(a, b, kl, ia, ib)
    d = a[:, 0].double() - a[:, 1].double()
    want = torch.tanh(d / 2) * d                     # two logits exchanged: (p0 - p1) (a0 - a1)
    # a handful of fp64 roundings (1.1e-16) of terms below |a| + |b| + 1 < 20
    assert torch.allclose(kl, want, rtol=0, atol=1e-13)
    assert torch.equal(ia.long(), a.argmax(1)) and torch.equal(ib.long(), b.argmax(1))


# The merges of a decode's splits: up to 512 rows (sequences x query heads) and more of them over more than
# 16 splits, at most 16 splits, and units (one sequence alone; not fp32).  Same bytes.
@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("fp8", 128), ("bf16", 256), ("f32", 64), ("f32", 256)])
def test_decode_merges_agree(dtype, D):
    import torch

    from gpu_helpers import TORCH_DTYPE
    from paper_2607_14431_amd import kvg
    Hq, Hkv, B, long = 32, 4, 20, 9000
    ctxs = [[8100, 511, 512, 1100, 5][b % 5] for b in range(B - 1)] + [long]
    per_seq = long // 16 + 1
    g = torch.Generator(device="cuda").manual_seed(D)
    cache = kvg.Cache.allocate(1, B * per_seq, Hq, Hkv, D, TORCH_DTYPE[dtype])
    for pool in (cache.k_pool, cache.v_pool):
        pool.copy_((torch.randn(pool.shape, generator=g, device="cuda") * 0.5).to(pool.dtype))
    tables = torch.randperm(B * per_seq, generator=g, device="cuda").to(torch.int32).view(B, per_seq)
    lens = torch.tensor(ctxs, dtype=torch.int32, device="cuda")
    start = torch.arange(B, device="cuda") * 100
    raw = [torch.randn((1, B, 1, h, D), generator=g, device="cuda").to(cache.raw_dtype) for h in (Hq, Hkv, Hkv)]

    def decode(rows):
        max_ctx = max(ctxs[b] for b in rows)
        seqs = kvg.Seqs(tables[rows].contiguous(), lens[rows].contiguous(), start[rows].contiguous(), max_ctx)
        out = torch.full((1, len(rows), 1, Hq, D), float("nan"), device="cuda")
        ws = kvg.decode_workspace(cache, seqs, 1)
        kvg.kvg_decode_attn(cache, seqs, kvg.rope(), 0, 1, *(t[:, rows].contiguous() for t in raw), D ** -0.5, out, ws)
        return out, len(rows) * Hq, (max_ctx + 512) // 512

    every = list(range(B))
    together, rows, splits = decode(every)
    assert torch.isfinite(together).all() and rows > 512 and splits > 16
    some, few_splits = every[10:], every[:11]
    for part, want in ((some, lambda r, s: r <= 512 and s > 16 and len(some) * Hkv * s * 4 > 2560),
                       (few_splits, lambda r, s: s <= 16 and len(few_splits) * Hkv * s * 4 > 2560),
                       ([3], lambda r, s: 1 < s <= 4), ([B - 1], lambda r, s: s > 16 and Hkv * s * 4 <= 1280)):
        out, r, s = decode(part)
        assert want(r, s)
        assert torch.equal(out.view(torch.int32), together[:, part].view(torch.int32)), part


# Rows of at most 64 keys: the weights are exact in fp32.  Position 0 leaves bf16 queries as they are, so what
# is left is fp32 arithmetic: a score is off by a few 2^-24 of the sum of its terms' magnitudes (below 8 here), an
# output by as much relatively; weights of 16 bits alone would leave 2^-18.6 = 2.5e-6.
@pytest.mark.parametrize("window", [0, 9, 64])
@pytest.mark.parametrize("call,dtype,D,Hq,Hkv", [
    ("decode", "bf16", 64, 8, 1), ("decode", "bf16", 128, 4, 2), ("decode", "bf16", 256, 2, 2), ("decode", "fp8", 64, 2, 1),
    ("decode", "fp8", 256, 8, 1), ("prefill", "bf16", 64, 8, 1), ("prefill", "bf16", 128, 16, 2), ("prefill", "bf16", 256, 8, 1),
    ("prefill", "fp8", 64, 8, 1), ("prefill", "fp8", 128, 8, 1), ("prefill", "fp8", 256, 8, 1)])
def test_few_keys_have_exact_weights(call, dtype, D, Hq, Hkv, window):
    import torch

    from gpu_helpers import TORCH_DTYPE
    from paper_2607_14431_amd import kvg
    ctxs = [0, 1, 7, 15, 16, 30, 63] + ([64, 73, 127, 200, 600] if window else [])
    B, per_seq, G = len(ctxs), max(ctxs) // 16 + 1, Hq // Hkv
    g = torch.Generator(device="cuda").manual_seed(D + window)
    cache = kvg.Cache.allocate(1, B * per_seq, Hq, Hkv, D, TORCH_DTYPE[dtype], windows=(window,))
    for pool in (cache.k_pool, cache.v_pool):
        pool.copy_((torch.randn(pool.shape, generator=g, device="cuda") * 0.5).to(pool.dtype))
    tables = torch.randperm(B * per_seq, generator=g, device="cuda").to(torch.int32).view(B, per_seq)
    lens = torch.tensor(ctxs, dtype=torch.int32, device="cuda")
    q, k, v = (torch.randn((1, B, 1, h, D), generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    out = torch.full((1, B, 1, Hq, D), float("nan"), device="cuda")
    seqs = kvg.Seqs(tables, lens, -lens.long(), max(ctxs))
    if call == "decode":
        ws = kvg.decode_workspace(cache, seqs, 1)
        kvg.kvg_decode_attn(cache, seqs, kvg.rope(), 0, 1, q, k, v, 3.0 * D ** -0.5, out, ws)
    else:
        ws = torch.empty(kvg.kvg_prefill_workspace_bytes(cache, seqs, 1, 1), dtype=torch.uint8, device="cuda")
        kvg.kvg_prefill_attn(cache, seqs, kvg.rope(), 0, 1, 1, q, k, v, 3.0 * D ** -0.5, out, ws)
    for b, n in enumerate(ctxs):
        lo = max(0, n + 1 - window) if window else 0
        rows = [cache.k_pool, cache.v_pool]
        kk, vv = (p[0][tables[b].long()].float().transpose(1, 2).reshape(-1, Hkv, D)[lo:n + 1].double() for p in rows)
        for h in range(Hq):
            s = kk[:, h // G] @ q[0, b, 0, h].double() * (3.0 * D ** -0.5)
            want = torch.softmax(s, 0) @ vv[:, h // G]
            got = out[0, b, 0, h].double()
            assert ((got - want).norm() / want.norm()).item() <= 1e-6, (n, h)
            if n + 1 - lo == 1:
                assert torch.equal(got, want)


# Inf and NaN among the values (and NaN among the keys) of tokens that a row does not see leave it as it is:
# later tokens of its chunk, tokens below its window in the same key block, page or tile.
@pytest.mark.parametrize("dtype,D,Hq,Hkv,windows", [
    ("f32", 64, 4, 2, (0, 40)), ("f32", 128, 4, 4, (0, 9)), ("f32", 256, 8, 1, (0, 300)),
    ("bf16", 64, 8, 1, (0, 40)), ("bf16", 128, 16, 2, (0, 300)), ("bf16", 256, 8, 1, (0, 70)),
    ("fp8", 64, 8, 1, (33, 300)), ("fp8", 128, 8, 1, (40, 9)), ("fp8", 256, 8, 1, (600, 70))])
def test_prefill_rows_take_nothing_from_masked_values(dtype, D, Hq, Hkv, windows):
    import torch

    from gpu_helpers import TORCH_DTYPE, attention_close
    from paper_2607_14431_amd import kvg
    L, ctx, chunk = 2, 700, 75
    n_pages = (ctx + chunk + 15) // 16
    g = torch.Generator(device="cuda").manual_seed(D)
    cache = kvg.Cache.allocate(L, n_pages, Hq, Hkv, D, TORCH_DTYPE[dtype], windows=windows)
    for pool in (cache.k_pool, cache.v_pool):
        pool.copy_((torch.randn(pool.shape, generator=g, device="cuda") * 0.5).to(pool.dtype))
    table = torch.randperm(n_pages, generator=torch.Generator().manual_seed(1)).to(torch.int32).cuda()[None]
    seqs = kvg.Seqs(table, torch.tensor([ctx], dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda"), ctx)
    q, k, v = (torch.randn((L, 1, chunk, h, D), device="cuda", generator=g).to(cache.raw_dtype) for h in (Hq, Hkv, Hkv))

    def run():
        out = torch.full((L, 1, chunk, Hq, D), float("nan"), device="cuda")
        ws = torch.empty(kvg.kvg_prefill_workspace_bytes(cache, seqs, L, chunk), dtype=torch.uint8, device="cuda")
        kvg.kvg_prefill_attn(cache, seqs, kvg.rope(), 0, L, chunk, q, k, v, D ** -0.5, out, ws)
        return out

    clean = run()
    assert torch.isfinite(clean).all()
    # chunk rows (an fp8 cache's appended values saturate) and cached tokens
    bad = {680, 693} | (set() if dtype == "fp8" else {ctx + 40, ctx + 57})
    for n in bad:
        if n >= ctx:
            v[:, 0, n - ctx, :, ::3] = float("inf") if n % 2 else float("nan")
        else:
            pool = cache.v_pool.view(torch.uint8) if dtype == "fp8" else cache.v_pool
            pool[:, int(table[0, n // 16]), :, n % 16, 1::3] = 0x7F if dtype == "fp8" else float("-inf")
    got = run()
    for layer, w in enumerate(windows):
        for i in range(chunk):
            sees = any(n <= ctx + i and (w == 0 or n > ctx + i - w) for n in bad)
            row, want = got[layer, 0, i], clean[layer, 0, i]
            if sees:
                assert not torch.isfinite(row).all(), (layer, i)
            elif dtype == "f32":
                assert torch.equal(row, want), (layer, i)
            else:
                attention_close(row.cpu().numpy(), want.cpu().numpy(), dtype)


@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 256), ("fp8", 64), ("fp8", 128), ("f32", 64), ("f32", 256)])
def test_windowed_decode_takes_nothing_from_below_its_window(dtype, D):
    import torch

    from gpu_helpers import INT_VIEW, TORCH_DTYPE
    from paper_2607_14431_amd import kvg
    Hq, Hkv, window, ctxs = 8, 2, 100, [104, 1000, 1011, 1012]
    B, per_seq = len(ctxs), max(ctxs) // 16 + 1
    g = torch.Generator(device="cuda").manual_seed(D)
    cache = kvg.Cache.allocate(1, B * per_seq, Hq, Hkv, D, TORCH_DTYPE[dtype], windows=(window,))
    for pool in (cache.k_pool, cache.v_pool):
        pool.copy_((torch.randn(pool.shape, generator=g, device="cuda") * 0.5).to(pool.dtype))
    tables = torch.randperm(B * per_seq, generator=g, device="cuda").to(torch.int32).view(B, per_seq)
    lens = torch.tensor(ctxs, dtype=torch.int32, device="cuda")
    raw = [torch.randn((1, B, 1, h, D), generator=g, device="cuda").to(cache.raw_dtype) for h in (Hq, Hkv, Hkv)]
    seqs = kvg.Seqs(tables, lens, torch.zeros(B, dtype=torch.int64, device="cuda"), max(ctxs))

    def run():
        out = torch.full((1, B, 1, Hq, D), float("nan"), device="cuda")
        kvg.kvg_decode_attn(cache, seqs, kvg.rope(), 0, 1, *raw, D ** -0.5, out, kvg.decode_workspace(cache, seqs, 1))
        return out

    clean = run()
    for b, ctx in enumerate(ctxs):
        for n in range((ctx + 1 - window) // 16 * 16, ctx + 1 - window):
            for pool in (cache.k_pool, cache.v_pool):
                pool.view(INT_VIEW[dtype])[:, int(tables[b, n // 16]), :, n % 16] = 0x7F if dtype == "fp8" else -1    # NaN
    assert torch.isfinite(clean).all() and torch.equal(run(), clean)
