"""Parity at the edges of the tiles and rules that choose a kernel: row counts around a tile's height, widths that leave
a partial last tile or one that straddles q | k | v, ranks that are no multiple of 16, short reductions, records
bounded by memory.  Everything against the oracle at the stated tolerances, cache bytes outside the new rows exact."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import alora_oracle as orc
from paper_2504_12397_amd import workloads as wl
from tests import helpers as H
from tests.test_gpu_parity import SMALL_BF16, SMALL_F32, check_case
from tests.test_zz_no_alloc import _both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ab():
    from paper_2504_12397_amd import binding
    return binding


@pytest.fixture()
def ctx(ab):
    c = ab.Context(0)
    yield c
    c.close()


def _split(T, n):
    """T rows as n sequences of uneven lengths"""
    cuts = [T * i * i // (n * n) for i in range(n + 1)]
    return [max(0, b - a) for a, b in zip(cuts, cuts[1:])]


# heads / kv heads give 6, 20, 32 columns of 256: tiles of 8, 12 and 16 rotation pairs, the 12-pair ones crossing heads and kinds
@pytest.mark.parametrize("hq,hkv,rank,T", [(8, 2, 8, 1), (8, 2, 24, 33), (32, 4, 64, 32), (32, 4, 8, 65), (32, 16, 16, 129),
                                           (32, 16, 40, 256), (32, 4, 16, 255),
                                           # more than 128 rows are streamed where tiles would leave most of the chip idle (up to 3200 columns)
                                           (16, 4, 16, 129), (8, 2, 24, 255), (16, 8, 8, 256)])
def test_few_rows_through_the_streaming_projection(ab, ctx, hq, hkv, rank, T):
    shape = wl.LayerShape(d=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=rank, n_adapters=4)
    n = min(T, 5)
    S = _split(T, n)
    P = [40, 0, 17, 90, 3][:n]
    case = H.make_case(shape, P, S, [P[b] + (S[b] // 2 if b % 2 else 0) for b in range(n)], [3, 1, -1, 2, 0][:n], seed=1000 + T,
                       prefix="random")
    check_case(ab, ctx, case)


@pytest.mark.parametrize("rank,T,few", [(8, 15, 2), (24, 31, 0), (40, 257, 0), (40, 257, 2), (64, 33, 0), (64, 2049, 1)])
def test_down_projection_in_one_kernel_or_two(ab, ctx, rank, T, few):
    """t = s A x_hat for every row from the kernel of few rows and from that of many; 3 * rank columns that end inside a tile."""
    ctx.set_option("prep_split", few)
    shape = wl.LayerShape(d=1024, n_q_heads=2, n_kv_heads=1, head_dim=128, rank=rank, n_adapters=3)
    S = _split(T, 4)
    case = H.make_case(shape, [5] * 4, S, [5, 5 + S[1] // 2, 5, 0], [0, 2, -1, 2], seed=1100 + rank + T, prefix="random")
    check_case(ab, ctx, case)


def _one_stack_layer(ab, ctx, shape, T, seed, ads=(1, -1, 2)):
    """A call of T rows in three sequences from empty caches through one whole layer, against the oracle"""
    rng = wl.Rng(seed)
    tensors = wl.make_layer(shape, rng, "L0")
    layer = H.oracle_layer(tensors, shape)
    S = _split(T, 3)
    ks = [S[0] // 2, 0, 0]
    xs = [H.f64(wl.make_hidden(rng, f"x{b}", S[b], shape)) for b in range(3)]
    cu = [0, S[0], S[0] + S[1], T]
    cache = [ab.KVCache([s + 1 for s in S], shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda")]
    xg = torch.from_numpy(np.concatenate(xs)).to(shape.torch_dtype).cuda().contiguous()
    out = ab.alora_stack_prefill(ctx, [H.gpu_layer(tensors, shape)], cache, xg, cu, ks, list(ads))
    torch.cuda.synchronize()
    for b in range(3):
        ref, _ = orc.ref_stack_full([layer], xs[b], ks[b], ads[b], shape.dtype)
        e = H.rel_err(H.f64(out[cu[b]:cu[b + 1]]), ref)
        H.report(check="one layer, large tiles", rows=T, sequence=b, err=e)
        assert e <= H.TOL[shape.dtype], f"sequence {b}: {e:.3e}"


# 1216 = 19 * 64: no large tiles for W_down (the reduction is no multiple of 128), 9.5 column tiles of gate | up;
# 1280: W_down split over two workgroups per tile
@pytest.mark.parametrize("T,inter,tile,rest,rank", [(257, 1280, 0, False, 16), (300, 1216, 2, True, 24), (511, 1280, 3, True, 8),
                                                    (513, 1216, 3, False, 8), (700, 1280, 0, True, 40), (700, 1280, 2, False, 16)])
def test_many_rows_through_the_large_tiles(ab, ctx, T, inter, tile, rest, rank):
    ctx.set_option("gemm_tile", tile)
    shape = dataclasses.replace(SMALL_BF16, intermediate=inter, rank=rank, adapt_rest=rest)
    _one_stack_layer(ab, ctx, shape, T, 1200 + T + inter)


@pytest.mark.parametrize("T,inter,rest,rank", [(33, 1280, True, 16), (129, 1280, True, 24), (256, 8192, False, 16), (640, 1280, True, 8), (1025, 2048, False, 40)])
def test_rows_through_the_tiles_of_128_rows(ab, ctx, T, inter, rest, rank):
    _one_stack_layer(ab, ctx, dataclasses.replace(SMALL_BF16, intermediate=inter, rank=rank, adapt_rest=rest), T, 2200 + T + inter)


# W_o and W_down (d x heads * 128 and d x inter) in tiles of 96, 128, 192, 256 columns, as fp32 partial sums of 8 or 4 segments and whole with
# the residual; 96 of 1280 and 1024 columns and 192 of 2560 and 1024 end inside a wave's part of the last tile.  The last: gate/up in 192 columns, three tiles a workgroup.
@pytest.mark.parametrize("T,d,heads,kv,inter,rest,rank", [(129, 1280, 32, 8, 4096, True, 16), (129, 2048, 32, 8, 4096, False, 8), (139, 2560, 32, 8, 4096, True, 24),
                                                          (150, 4096, 32, 8, 4096, True, 16),
                                                          (513, 1024, 16, 4, 2048, True, 16), (700, 1024, 16, 4, 2048, False, 8), (1100, 1024, 32, 8, 4096, True, 16), (1300, 1024, 4, 1, 5120, True, 24),
                                                          (1600, 1280, 4, 1, 512, True, 16), (2100, 1536, 4, 1, 512, False, 8), (1600, 2560, 4, 1, 512, True, 16), (2100, 3072, 4, 1, 512, True, 8),
                                                          (400, 512, 4, 1, 16448, True, 16)])
def test_linears_in_tiles_of_every_width(ab, ctx, T, d, heads, kv, inter, rest, rank):
    shape = wl.LayerShape(d=d, n_q_heads=heads, n_kv_heads=kv, head_dim=128, rank=rank, n_adapters=3, intermediate=inter, adapt_rest=rest)
    _one_stack_layer(ab, ctx, shape, T, 2800 + T + d)


# columns of a tile: 64, 64, 96, 96 (the last tile is part of one), 128, 192 (part of one), 256; 192 and three tiles a workgroup; 96, 128, 192 of 6144 columns
@pytest.mark.parametrize("hq,hkv,T,rank", [(16, 8, 129, 16), (8, 2, 257, 8), (32, 8, 257, 64), (64, 8, 129, 24), (32, 16, 257, 8), (64, 8, 400, 16), (64, 8, 513, 32), (32, 32, 1500, 16),
                                           (16, 4, 700, 24), (32, 8, 1000, 64), (32, 8, 1200, 16)])
def test_projection_in_tiles_of_every_width_gives_the_same_bits(ab, hq, hkv, T, rank):
    """Queries, keys and values of one running sum: the same from 256 x 256 tiles (gemm_tile 3) as from the tiles of 128 rows.  Both rotate and append by themselves."""
    shape = wl.LayerShape(d=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=rank, n_adapters=3)
    S = [T - 40, 17, 23]
    case = H.make_case(shape, [5, 33, 0], S, [5 + S[0] // 2, 33, 4], [1, 2, 0], seed=2300 + T + hq, prefix="random")
    layer, x = H.gpu_layer(case, shape), case.x_packed.cuda().contiguous()
    got = []
    for tile in (0, 3):
        c = ab.Context(0)
        c.set_option("gemm_tile", tile)
        c.set_option("profile", 1)
        cache = H.gpu_cache(case)
        out = ab.alora_prefill(c, layer, cache, x, case.cu, case.k, case.adapter)
        torch.cuda.synchronize()
        assert "rope_append" not in c.profile_read()      # (what takes over where the tiles cannot)
        got.append([t.clone() for t in (out, cache.k, cache.v)])
        c.close()
    assert all(torch.equal(p, q) for p, q in zip(*got))
    ref, _ = H.oracle_prefill(case)
    assert H.rel_err(H.f64(got[0][0]), ref) <= H.TOL["bf16"]


@pytest.mark.parametrize("T", [20, 300])
def test_weights_that_are_not_16_byte_aligned(ab, ctx, T):
    """Parameters that are views into one flat buffer, eight bytes off: the kernels whose weights go to LDS by request
    are passed by."""
    shape = dataclasses.replace(SMALL_BF16, intermediate=1280)
    case = H.make_case(shape, [30, 7], [T - 8, 8], [30, 7], [1, 2], seed=1300 + T, prefix="random")
    tensors = {}
    for name, t in case.tensors.items():
        if isinstance(t, torch.Tensor):
            flat = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
            flat[4:] = t.reshape(-1).cuda()
            t = flat[4:].view(t.shape)
            assert t.data_ptr() % 16 == 8
        tensors[name] = t
    layer = ab.Layer(tensors, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rms_eps, shape.rope_theta, shape.intermediate)
    x = case.x_packed.cuda().contiguous()
    for call in (ab.alora_prefill, ab.alora_stack_prefill):
        stack = call is ab.alora_stack_prefill
        cache, same = H.gpu_cache(case), H.gpu_cache(case)
        aligned = H.gpu_layer(case, shape)
        args = (x, case.cu, case.k, case.adapter)
        out = call(ctx, [layer], [cache], *args) if stack else call(ctx, layer, cache, *args)
        want = call(ctx, [aligned], [same], *args) if stack else call(ctx, aligned, same, *args)
        torch.cuda.synchronize()
        if not stack:
            ref, _ = H.oracle_prefill(case)
            assert H.rel_err(H.f64(out), ref) <= H.TOL["bf16"]
        # two correct results at half the tolerance each
        assert H.rel_err(H.f64(out), H.f64(want)) <= H.TOL["bf16"]


@pytest.mark.parametrize("T", [1, 3, 16, 17, 63, 65])
@pytest.mark.parametrize("d,hq,hkv,h", [(256, 4, 2, 64), (200, 6, 3, 36), (520, 16, 1, 48)])
def test_small_calls_on_the_plain_kernels(ab, ctx, T, d, hq, hkv, h):
    """One kernel for projection, rotation and append; hidden sizes that end inside its 256 values of k, pair counts that end
    inside a tile, head sizes with and without 16-byte loads, more query heads per kv head than one workgroup takes."""
    shape = dataclasses.replace(SMALL_F32, d=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, rank=5)
    S = _split(T, min(T, 3))
    n = len(S)
    case = H.make_case(shape, [64, 0, 129][:n], S, [64, S[1] // 2 if n > 1 else 0, 130][:n], [0, 1, -1][:n], seed=1400 + T + d,
                       prefix="random")
    check_case(ab, ctx, case)


@pytest.mark.parametrize("P", [[4000] + [60] * 20, [31, 32, 33, 1, 0, 127, 128, 129, 511, 513], [9000], [700] * 33])
def test_decode_key_ranges(ab, ctx, P):
    """Lists of uneven lengths: one long sequence among short ones, lengths around a step of 32 keys, one sequence alone."""
    shape = wl.LayerShape(d=512, n_q_heads=8, n_kv_heads=4, head_dim=128, rank=16, n_adapters=3)
    n = len(P)
    case = H.make_case(shape, P, [1] * n, [max(0, p - 10) for p in P], [b % 4 - 1 for b in range(n)], seed=1500 + n, prefix="random")
    check_case(ab, ctx, case, decode=True)


def test_static_decode_of_one_long_sequence_among_short_ones(ab, ctx):
    """64 sequences, one of them long: as many partial records per row as the long one alone would like do not fit the
    static scratch array; the call is taken with fewer, bit-identical to alora_decode."""
    shape = wl.LayerShape(d=512, n_q_heads=32, n_kv_heads=8, head_dim=128, rank=16, n_adapters=2)
    P = [16448] + [100 + b for b in range(63)]
    case = H.make_case(shape, P, [1] * 64, P, [b % 3 - 1 for b in range(64)], seed=1600, prefix="random")
    _both(ab, ctx, case)


# a range is 128 keys here: 16 records (the fewest that a workgroup merges), 64 with and without the next one, places that shorter
# rows leave without a record
@pytest.mark.parametrize("P", [[2047], [8191], [8192], [8063, 127, 0, 129], [9000, 8300, 5]])
def test_merge_of_many_records(ab, ctx, P):
    shape = wl.LayerShape(d=512, n_q_heads=4, n_kv_heads=2, head_dim=128, rank=16, n_adapters=3)
    n = len(P)
    case = H.make_case(shape, P, [1] * n, [max(0, p - 10) for p in P], [b % 4 - 1 for b in range(n)], seed=1700 + P[0], prefix="random")
    check_case(ab, ctx, case, decode=True)


def test_down_projection_of_more_rows_than_32_bit_offsets_reach(ab, ctx):
    """524544 rows of 4096: byte offsets of x_hat pass 2^31 at row 262144 and 2^32 at row 524288.  W_v = 0 and no RMSNorm, so the
    appended value rows are s B (A x) and nothing else."""
    n, each, d, r = 2049, 256, 4096, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(1800)
    T = n * each
    x = torch.empty((T, d), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    t = {"W_qkv": torch.zeros((384, d), dtype=torch.bfloat16, device="cuda"),
         "A": torch.empty((1, 3, r, d), dtype=torch.bfloat16, device="cuda").normal_(0, d ** -0.5, generator=g), "scale": [2.0], "rms_gain": None}
    for p in ("B_q", "B_k", "B_v"):
        t[p] = torch.empty((1, 128, r), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    cache = ab.KVCache([each] * n, 1, 128, torch.bfloat16, "cuda")
    ab.alora_prefill(ctx, ab.Layer(t, 1, 1, 128), cache, x, [each * i for i in range(n + 1)], [0] * n, [0] * n)
    torch.cuda.synchronize()
    for b in (0, 1023, 1024, 2047, 2048):
        xb = x[b * each:(b + 1) * each].cpu().double()
        ref = 2.0 * (xb @ t["A"][0, 2].cpu().double().T) @ t["B_v"][0].cpu().double().T
        e = H.rel_err(H.f64(cache.rows(b, 0, each)[1][:, 0]), ref.numpy())
        assert e <= H.TOL["bf16"], f"rows {b * each} ..: {e:.3e}"


def test_large_tiles_of_an_operand_just_short_of_2_gb(ab, ctx):
    """74241 rows of 14336 through W_down: the operand is below 2 GB but one row more than the kernel takes at once, and a narrow
    output asks for several workgroups per tile.  W_o = 0, so the layer is x + MLP(x)."""
    n, each, d, inter = 291, 256, 512, 14336
    S = [each] * (n - 1) + [1]
    T = sum(S)
    g = torch.Generator(device="cuda")
    g.manual_seed(1900)

    def normal(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)

    t = {"W_qkv": normal(384, d, std=d ** -0.5), "W_o": torch.zeros((d, 128), dtype=torch.bfloat16, device="cuda"), "rms_gain": None,
         "rms2_gain": torch.ones(d, dtype=torch.bfloat16, device="cuda"), "W_gate": normal(inter, d, std=d ** -0.5),
         "W_up": normal(inter, d, std=d ** -0.5), "W_down": normal(d, inter, std=4 * inter ** -0.5)}
    x = normal(T, d)
    cu = [0]
    for s in S:
        cu.append(cu[-1] + s)
    cache = [ab.KVCache(S, 1, 128, torch.bfloat16, "cuda")]
    out = ab.alora_stack_prefill(ctx, [ab.Layer(t, 1, 1, 128, 1e-5, 10000.0, inter)], cache, x, cu, [0] * n, [-1] * n)
    torch.cuda.synchronize()
    w = {k: v.cpu().double() for k, v in t.items() if v is not None}
    for lo, hi in ((0, 64), (30000, 30064), (T - 65, T)):
        h = x[lo:hi].cpu().double()
        hn = (h * torch.rsqrt((h * h).mean(1, keepdim=True) + 1e-5)).to(torch.bfloat16).double()
        act = (torch.nn.functional.silu(hn @ w["W_gate"].T) * (hn @ w["W_up"].T)).to(torch.bfloat16).double()
        e = H.rel_err(H.f64(out[lo:hi]), (h + act @ w["W_down"].T).numpy())
        assert e <= H.TOL["bf16"], f"rows {lo} ..: {e:.3e}"


@pytest.mark.parametrize("rank", [8, 24, 32, 64])
def test_rotation_fused_or_not_gives_the_same_bits_at_every_rank(ab, rank):
    """The low-rank term joins the sums in one order in every projection kernel: the large tiles, the one that leaves the rotation
    to another kernel and, given the same t (prep_split = 0), the one that streams the weights past few rows."""
    shape = dataclasses.replace(SMALL_BF16, rank=rank)
    case = H.make_case(shape, [30, 0, 64], [230, 190, 77], [40, 0, 100], [1, 2, -1], seed=2000 + rank, prefix="random")
    got = []
    for fuse in (1, 0):
        c = ab.Context(0)
        try:
            c.set_option("rope_fuse", fuse)
            out, cache = check_case(ab, c, case)
            got.append((out.clone(), cache.k.clone(), cache.v.clone()))
        finally:
            c.close()
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    layer = H.gpu_layer(case, shape)
    x = wl.make_hidden(wl.Rng(2010 + rank), "x", 300, shape).cuda()
    rows = []
    for n in (40, 300):
        c = ab.Context(0)
        try:
            c.set_option("prep_split", 0)
            cache = ab.KVCache([n], shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda")
            ab.alora_prefill(c, layer, cache, x[:n].contiguous(), [0, n], [7], [2])
            torch.cuda.synchronize()
            rows.append(cache.rows(0, 0, 40))
        finally:
            c.close()
    for a, b in zip(*rows):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("linear", ["W_o", "W_down"])
def test_gemm_splits_cuts_the_same_segments_at_every_number_of_rows(ab, linear):
    """gemm_splits = 4: a row's sums are the same bits from a call of 256 rows (a workgroup per segment) and one of 300 (a workgroup
    adds the segments itself), and other ones than with a single running sum.  Sequences of one row, so attention hands on v; for
    W_down W_v = 0 and x is +-1, so both calls normalise exactly the same rows."""
    shape = dataclasses.replace(SMALL_BF16, intermediate=1280)
    rng = wl.Rng(2100)
    t = wl.make_layer(shape, rng)
    if linear == "W_o":
        t["W_down"].zero_()
        x = wl.make_hidden(rng, "x", 300, shape)
    else:
        t["W_qkv"][-shape.n_kv:].zero_()
        x = wl.make_hidden(rng, "x", 300, shape).sign()
    layer, x = H.gpu_layer(t, shape), x.cuda()
    got = {}
    for splits, n in ((4, 256), (4, 300), (1, 300)):
        c = ab.Context(0)
        try:
            c.set_option("gemm_splits", splits)
            cache = ab.KVCache([1] * n, shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda")
            out = ab.alora_stack_prefill(c, [layer], [cache], x[:n].contiguous(), list(range(n + 1)), [0] * n, [-1] * n)
            torch.cuda.synchronize()
            got[splits, n] = out[:256].clone().view(torch.int16)
        finally:
            c.close()
    assert torch.equal(got[4, 256], got[4, 300])
    assert not torch.equal(got[4, 300], got[1, 300])


def _appended(ab, layer, shape, x, opts=(), profile=False, decode=False):
    """The rows that a base-only call on the hidden states x appends: one sequence, or (decode) a sequence per row"""
    c = ab.Context(0)
    try:
        for k, v in opts:
            c.set_option(k, v)
        if profile:
            c.set_option("profile", 1)
        n = x.shape[0]
        cache = ab.KVCache([1] * n if decode else [n], shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda")
        if decode:
            ab.alora_decode(c, layer, cache, x, [0] * n, [-1] * n)
        else:
            ab.alora_prefill(c, layer, cache, x, [0, n], [0], [-1])
        torch.cuda.synchronize()
        return torch.cat([cache.k, cache.v], dim=2).view(torch.int16), c.profile_read() if profile else None
    finally:
        c.close()


# hidden sizes of the plain row preparation, reductions that end in half a stage (384, 640, 896), heads of 48, 64 and 256 columns, query
# groups that the matrix attention kernels do not take (5, and any other head size: queries as fp32); 320 is not streamed
OTHER_SHAPES = [(640, 8, 2, 128), (384, 4, 2, 64), (1280, 10, 2, 128), (768, 4, 1, 256), (896, 16, 2, 48), (320, 8, 2, 128)]


@pytest.mark.parametrize("d,hq,hkv,h", OTHER_SHAPES)
@pytest.mark.parametrize("T", [1, 70, 200])
def test_few_rows_of_other_shapes(ab, ctx, d, hq, hkv, h, T):
    shape = wl.LayerShape(d=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, rank=24, n_adapters=4)
    n = min(T, 4)
    S = _split(T, n)
    P = [40, 0, 17, 90][:n]
    case = H.make_case(shape, P, S, [P[b] + (S[b] // 2 if b % 2 else 0) for b in range(n)], [3, 1, -1, 2][:n], seed=2200 + T + d,
                       prefix="random")
    check_case(ab, ctx, case)
    if T > 1:
        case = H.make_case(shape, [40] * T, [1] * T, [20] * T, [b % 5 - 1 for b in range(T)], seed=2210 + T + d, prefix="random")
        check_case(ab, ctx, case, decode=True)
        _both(ab, ctx, case)


@pytest.mark.parametrize("d,hq,hkv,h", OTHER_SHAPES)
def test_rows_of_other_shapes_do_not_depend_on_the_call(ab, d, hq, hkv, h):
    """One row, 40, 200 and 300, a decode step: the same bits; few rows are rotated in the projection except where it cannot."""
    shape = wl.LayerShape(d=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=h, rank=8, n_adapters=1)
    rng = wl.Rng(2300 + d)
    layer, x = H.gpu_layer(wl.make_layer(shape, rng), shape), wl.make_hidden(rng, "x", 300, shape).cuda()
    want, _ = _appended(ab, layer, shape, x)
    for n in (1, 40, 200):
        got, prof = _appended(ab, layer, shape, x[:n].contiguous(), profile=True)
        assert torch.equal(got, want[:n])
        assert ("rope_append" in prof) == (d == 320)
    step, _ = _appended(ab, layer, shape, x[:1].contiguous(), decode=True)
    assert torch.equal(step, want[:1])


def test_unaligned_weights_keep_the_segments_of_their_shape(ab):
    """2048 x 1536 a few bytes off: four segments, from one row to 300 (default = gemm_splits 4, bit for bit)."""
    shape = wl.LayerShape(d=2048, n_q_heads=8, n_kv_heads=2, head_dim=128, rank=8, n_adapters=1)
    rng = wl.Rng(2400)
    t = wl.make_layer(shape, rng)
    x = wl.make_hidden(rng, "x", 300, shape).cuda()
    flat = torch.empty(t["W_qkv"].numel() + 4, dtype=torch.bfloat16, device="cuda")
    flat[4:] = t["W_qkv"].reshape(-1).cuda()
    t["W_qkv"] = flat[4:].view(t["W_qkv"].shape)
    layer = H.gpu_layer(t, shape)
    assert layer.t["W_qkv"].data_ptr() % 16 == 8
    want, _ = _appended(ab, layer, shape, x, [("gemm_splits", 4)])
    for n in (1, 40, 200, 300):
        got, prof = _appended(ab, layer, shape, x[:n].contiguous(), profile=True)
        assert torch.equal(got, want[:n])
        assert ("rope_append" in prof) == (n <= 256)
    got, _ = _appended(ab, layer, shape, x, [("rope_fuse", 0)])
    assert torch.equal(got, want)
    one, _ = _appended(ab, layer, shape, x, [("gemm_splits", 1)])
    assert not torch.equal(one, want)


def test_static_decode_with_segments_that_do_not_fit_the_scratch(ab, ctx):
    """240 rows of unaligned 4096 x 6144 weights: four partial sums of the projection alone are 24 MB of the 32; both entry points add the
    segments inside the workgroups, with the bits that one row gets from partial sums."""
    shape = wl.SHAPE_8B_4AD
    rng = wl.Rng(2450, "cuda")
    t = wl.make_layer(shape, rng)
    flat = torch.empty(t["W_qkv"].numel() + 4, dtype=torch.bfloat16, device="cuda")
    flat[4:] = t["W_qkv"].reshape(-1)
    t["W_qkv"] = flat[4:].view(t["W_qkv"].shape)
    layer = ab.Layer(t, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rms_eps, shape.rope_theta)
    n = 240
    x = wl.make_hidden(rng, "x", n, shape)
    got = []
    for call in (ab.alora_decode, ab.alora_decode_static):
        cache = ab.KVCache([6] * n, shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda", fill=0.5)
        cache.seq_len[:] = 5
        out = torch.empty((n, shape.n_q), dtype=shape.torch_dtype, device="cuda")
        call(ctx, layer, cache, x, [0] * n, [b % 5 - 1 for b in range(n)], out)
        torch.cuda.synchronize()
        got.append([v.view(torch.int16) for v in (out, cache.k, cache.v)])
    assert all(torch.equal(a, b) for a, b in zip(*got))
    cache = ab.KVCache([6], shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda", fill=0.5)
    cache.seq_len[:] = 5
    ab.alora_decode(ctx, layer, cache, x[:1].contiguous(), [0], [-1])
    torch.cuda.synchronize()
    assert torch.equal(cache.k[5].view(torch.int16), got[0][1][5]) and torch.equal(cache.v[5].view(torch.int16), got[0][2][5])


@pytest.mark.parametrize("T", [128, 129, 256])
def test_rows_of_wide_weights_do_not_depend_on_the_call(ab, ctx, T):
    """More than 4096 rotation pairs: the streaming kernel up to 128 rows, the tiles beyond, the same bits."""
    shape = wl.LayerShape(d=512, n_q_heads=64, n_kv_heads=8, head_dim=128, rank=8, n_adapters=2)
    S = _split(T, 3)
    case = H.make_case(shape, [30, 0, 64], S, [30, S[1] // 2, 64], [1, 0, -1], seed=2500 + T, prefix="random")
    check_case(ab, ctx, case)
    layer, x = H.gpu_layer(case, shape), wl.make_hidden(wl.Rng(2510), "x", 300, shape).cuda()
    want, _ = _appended(ab, layer, shape, x)
    got, _ = _appended(ab, layer, shape, x[:T].contiguous())
    assert torch.equal(got, want[:T])


# one range per row and eight heads side by side; heads that are no multiple of eight; a long row among more rows than two rounds of
# workgroups; four heads, ranges of one round; one row with as many records as it may have
@pytest.mark.parametrize("hq,hkv,P", [(16, 16, [64] * 130), (20, 10, [300] * 70 + [31, 0]), (8, 8, [5000] + [20] * 600), (8, 4, [900] * 33),
                                      (16, 16, [63, 1, 200] * 50), (8, 8, [20000])])
def test_decode_cuts_of_many_and_few_rows(ab, ctx, hq, hkv, P):
    shape = wl.LayerShape(d=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=16, n_adapters=3)
    n = len(P)
    case = H.make_case(shape, P, [1] * n, [max(0, p - 10) for p in P], [b % 4 - 1 for b in range(n)], seed=2600 + n + hkv, prefix="random")
    check_case(ab, ctx, case, decode=True)
    if n < 200:
        _both(ab, ctx, case)


@pytest.mark.parametrize("P", [[5, 200], [0], [31, 700, 64, 1, 90]])
def test_long_run_of_decode_steps(ab, ctx, P):
    """300 steps: the keys are cut as the last step has them, so the first steps meet ranges that hold nothing yet."""
    shape = wl.LayerShape(d=512, n_q_heads=8, n_kv_heads=4, head_dim=128, rank=16, n_adapters=3)
    n, steps = len(P), 300
    case = H.make_case(shape, P, [steps] * n, [p + 40 * b for b, p in enumerate(P)], [b % 4 - 1 for b in range(n)], seed=2700 + n, prefix="random")
    x = torch.stack([torch.stack([case.x_new[b][t] for b in range(n)]) for t in range(steps)]).cuda().contiguous()
    cache = H.gpu_cache(case)
    before_k, before_v = cache.k.cpu(), cache.v.cpu()
    out = ab.alora_decode_steps(ctx, H.gpu_layer(case, shape), cache, x, case.k, case.adapter)
    torch.cuda.synchronize()
    ref, rows = H.oracle_prefill(case)
    H.check_cache_after(case, cache, before_k, before_v, rows, H.TOL["bf16"])
    got = H.f64(out).transpose(1, 0, 2).reshape(n * steps, -1)
    assert H.rel_err(got, ref) <= H.TOL["bf16"]


@pytest.mark.parametrize("T", [40, 300])
def test_lora_split_gives_the_low_rank_term_a_partial_sum(ab, T):
    """Always (1): few rows and many leave the fused kernels, which have no partial sums; rows without an adapter keep their bits."""
    S = _split(T, 3)
    case = H.make_case(SMALL_BF16, [30, 0, 64], S, [30, S[1], 64], [1, 0, -1], seed=2800 + T, prefix="random")
    got = {}
    for split in (0, 1, 2):
        c = ab.Context(0)
        try:
            c.set_option("lora_split", split)
            c.set_option("profile", 1)
            _, cache = check_case(ab, c, case)
            assert ("rope_append" in c.profile_read()) == (split == 1)
            got[split] = [torch.cat([t[int(o) + p:int(o) + p + s] for o, p, s in zip(cache.seq_offset[1:], case.P[1:], S[1:])]).clone().view(torch.int16)
                          for t in (cache.k, cache.v)]
        finally:
            c.close()
    for split in (1, 2):
        assert all(torch.equal(a, b) for a, b in zip(got[0], got[split]))


# one to five tiles of 64 keys, whole, one short and one over; padding rows; a causal edge in every place of a tile
@pytest.mark.parametrize("splits", [0, 1, 3])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_prefill_attention_around_tiles_of_keys(ab, ctx, G, splits):
    ctx.set_option("kv_splits", splits)
    shape = wl.LayerShape(d=256, n_q_heads=8, n_kv_heads=8 // G, head_dim=128, rank=8, n_adapters=2)
    P = [0, 0, 0, 31, 32, 62, 63, 64, 127, 128, 190, 191, 192, 193, 255, 256, 257, 320]
    S = [1, 33, 64, 1, 1, 1, 2, 65, 1, 1, 2, 1, 130, 1, 1, 1, 63, 257]
    n = len(P)
    case = H.make_case(shape, P, S, [P[b] + b % 2 for b in range(n)], [b % 3 - 1 for b in range(n)], seed=1500 + G, prefix="random")
    check_case(ab, ctx, case)


# gate/up tiles of 16, 32, 48, 56 and 64 pairs, one round or several, a partial last one; W_down streamed (whole kilobytes, up to 32 rows) or not;
# rows around the row blocks; adapters on every linear with ranks that are no multiple of 16
@pytest.mark.parametrize("T,inter,d,rest,rank", [(1, 1280, 512, False, 16), (32, 8192, 512, True, 8), (33, 12224, 256, False, 16), (31, 14336, 512, True, 24),
                                                 (64, 14336, 256, False, 8), (65, 16320, 256, True, 40), (128, 14336, 256, False, 16), (129, 8192, 256, True, 8),
                                                 (200, 14336, 256, True, 16), (256, 20032, 256, False, 16), (7, 20032, 640, True, 16), (3, 7168, 1152, True, 16),
                                                 # more than 192 rows: streamed in one round of tiles wider than the smallest, else in tiles of 128 rows
                                                 (192, 4096, 256, False, 16), (193, 4096, 256, True, 8), (193, 4160, 256, True, 24), (256, 16384, 256, False, 8),
                                                 (192, 16448, 256, True, 16), (193, 16448, 256, False, 16)])
def test_few_rows_through_the_streaming_linears(ab, ctx, T, inter, d, rest, rank):
    shape = wl.LayerShape(d=d, n_q_heads=4, n_kv_heads=1, head_dim=128, rank=rank, n_adapters=3, intermediate=inter, adapt_rest=rest)
    _one_stack_layer(ab, ctx, shape, T, 1700 + T + inter)


@pytest.mark.parametrize("B,V,d", [(1, 1000, 512), (32, 40004, 256), (33, 1024, 1024), (200, 2052, 256)])
def test_output_head_of_few_rows(ab, ctx, B, V, d):
    g = torch.Generator(device="cuda").manual_seed(V + B)
    x = torch.randn(B, d, device="cuda", generator=g).to(torch.bfloat16)
    gain = (1 + 0.1 * torch.randn(d, device="cuda", generator=g)).to(torch.bfloat16)
    W = (torch.randn(V, d, device="cuda", generator=g) * d ** -0.5).to(torch.bfloat16)
    token, logits = ab.alora_lm_head(ctx, x, gain, 1e-5, W, want_logits=True)
    torch.cuda.synchronize()
    x64 = x.double().cpu()
    xh = (x64 * gain.double().cpu() / torch.sqrt((x64 * x64).mean(1, keepdim=True) + 1e-5)).to(torch.bfloat16).double()
    ref = xh @ W.double().cpu().T
    # a row's d products of bf16 values summed in fp32, and elements of x_hat that round the other way (2^-9 of one of d terms)
    assert H.rel_err(H.f64(logits), ref.numpy()) <= 1e-2
    assert torch.equal(token.cpu().long(), logits.float().cpu().argmax(1))


# 96 columns per workgroup (many adapted rows) or 32; 3 * rank columns that end inside a tile of either
@pytest.mark.parametrize("rank,T", [(64, 3000), (40, 5200), (24, 700), (64, 2800)])
def test_down_projection_of_many_adapted_rows(ab, ctx, rank, T):
    ctx.set_option("prep_split", 0)
    shape = wl.LayerShape(d=512, n_q_heads=2, n_kv_heads=1, head_dim=128, rank=rank, n_adapters=3)
    S = _split(T, 3)
    case = H.make_case(shape, [5] * 3, S, [5, 5 + S[1] // 2, 5], [0, 2, 1], seed=1900 + rank + T, prefix="random")
    check_case(ab, ctx, case)


@pytest.mark.parametrize("shape", [wl.LayerShape(d=512, n_q_heads=4, n_kv_heads=2, head_dim=128, rank=16, n_adapters=2),
                                   wl.LayerShape(d=256, n_q_heads=4, n_kv_heads=4, head_dim=64, rank=8, n_adapters=2, dtype="f32", rmsnorm=False)],
                         ids=["bf16", "fp32"])
def test_decode_steps_whose_outputs_are_the_next_inputs(ab, ctx, shape):
    """attn_out one step into x_steps: every step reads what the step before wrote."""
    n, P = 5, [40, 7, 129]
    case = H.make_case(shape, P, [n] * 3, [30, 9, 400], [0, 1, -1], seed=2950, prefix="random")
    layer = H.gpu_layer(case, shape)
    x = torch.zeros(n + 1, 3, shape.d, dtype=shape.torch_dtype, device="cuda")
    x[0] = torch.stack([case.x_new[b][0] for b in range(3)]).cuda()
    chain, cache = H.gpu_cache(case), H.gpu_cache(case)
    want = [x[0].clone()]
    for t in range(n):
        want.append(ab.alora_decode(ctx, layer, chain, want[-1], case.k, case.adapter).clone())
    ab.alora_decode_steps(ctx, layer, cache, x[:n], case.k, case.adapter, x[1:])
    torch.cuda.synchronize()
    assert torch.equal(cache.k, chain.k) and torch.equal(cache.v, chain.v)
    # (the keys may be cut in other ranges: a run's as its last step has them)
    assert H.rel_err(H.f64(x[1:].reshape(3 * n, -1)), H.f64(torch.stack(want[1:]).reshape(3 * n, -1))) <= H.TOL[shape.dtype]


# 1024 rows at a time: steps that do and do not divide, more rows than that in one step, a plain shape
@pytest.mark.parametrize("P,steps,dtype", [([3, 90, 31], 350, "bf16"), ([20] * 300, 4, "bf16"), ([5] * 1100, 2, "bf16"), ([10, 2, 30], 400, "f32")])
def test_decode_steps_projected_together(ab, ctx, P, steps, dtype):
    shape = (wl.LayerShape(d=512, n_q_heads=4, n_kv_heads=2, head_dim=128, rank=16, n_adapters=3) if dtype == "bf16" else
             wl.LayerShape(d=128, n_q_heads=2, n_kv_heads=2, head_dim=32, rank=8, n_adapters=3, dtype="f32", rmsnorm=False))
    n = len(P)
    case = H.make_case(shape, P, [steps] * n, [p + b % 3 for b, p in enumerate(P)], [b % 4 - 1 for b in range(n)], seed=2970 + n, prefix="random")
    x = torch.stack([torch.stack([case.x_new[b][t] for b in range(n)]) for t in range(steps)]).cuda().contiguous()
    cache = H.gpu_cache(case)
    before_k, before_v = cache.k.cpu(), cache.v.cpu()
    out = ab.alora_decode_steps(ctx, H.gpu_layer(case, shape), cache, x, case.k, case.adapter)
    torch.cuda.synchronize()
    ref, rows = H.oracle_prefill(case)
    H.check_cache_after(case, cache, before_k, before_v, rows, H.TOL[dtype])
    assert H.rel_err(H.f64(out).transpose(1, 0, 2).reshape(n * steps, -1), ref) <= H.TOL[dtype]


# one prefill of all steps (rows step after step), or -- options that choose another prefill kernel -- a step at a time
@pytest.mark.parametrize("G,steps,opts", [(1, 2, {}), (2, 70, {}), (4, 65, {}), (8, 33, {}), (4, 3, {"kv_splits": 3}), (4, 5, {"attn_partials16": 0}),
                                          (4, 5, {"attn_fold": 0}), (4, 5, {"attn_waves": 4}), (4, 5, {"kernels": 1}), (16, 5, {})])
def test_runs_of_decode_steps(ab, ctx, G, steps, opts):
    for k, v in opts.items():
        ctx.set_option(k, v)
    shape = wl.LayerShape(d=256, n_q_heads=16, n_kv_heads=16 // G, head_dim=128, rank=8, n_adapters=2)
    P = [0, 63, 64, 1, 500]
    n = len(P)
    case = H.make_case(shape, P, [steps] * n, [p + b for b, p in enumerate(P)], [b % 3 - 1 for b in range(n)], seed=3000 + G + steps, prefix="random")
    x = torch.stack([torch.stack([case.x_new[b][t] for b in range(n)]) for t in range(steps)]).cuda().contiguous()
    cache = H.gpu_cache(case)
    before_k, before_v = cache.k.cpu(), cache.v.cpu()
    out = ab.alora_decode_steps(ctx, H.gpu_layer(case, shape), cache, x, case.k, case.adapter)
    torch.cuda.synchronize()
    ref, rows = H.oracle_prefill(case)
    H.check_cache_after(case, cache, before_k, before_v, rows, H.TOL["bf16"])
    assert H.rel_err(H.f64(out).transpose(1, 0, 2).reshape(n * steps, -1), ref) <= H.TOL["bf16"]


# beyond the 1024 rows that are projected together: parts of about equal length, each in one pass over what is cached before it
@pytest.mark.parametrize("n,steps,parts", [(64, 16, 1), (64, 17, 2), (64, 33, 3), (3, 341, 1), (3, 342, 2), (1, 2049, 3)])
def test_runs_of_decode_steps_in_parts(ab, ctx, n, steps, parts):
    ctx.set_option("profile", 1)
    shape = wl.LayerShape(d=256, n_q_heads=4, n_kv_heads=2, head_dim=128, rank=8, n_adapters=2)
    P = [(37 * b) % 90 for b in range(n)]
    case = H.make_case(shape, P, [steps] * n, [p + b % 5 for b, p in enumerate(P)], [b % 3 - 1 for b in range(n)], seed=3050 + n, prefix="random")
    x = torch.stack([torch.stack([case.x_new[b][t] for b in range(n)]) for t in range(steps)]).cuda().contiguous()
    cache = H.gpu_cache(case)
    before_k, before_v = cache.k.cpu(), cache.v.cpu()
    out = ab.alora_decode_steps(ctx, H.gpu_layer(case, shape), cache, x, case.k, case.adapter)
    torch.cuda.synchronize()
    assert {f: ctx.profile_read()[f]["launches"] for f in ("qkv_gemm", "attn_prefill", "attn_decode")} == {"qkv_gemm": parts, "attn_prefill": parts, "attn_decode": parts}
    ref, rows = H.oracle_prefill(case)
    H.check_cache_after(case, cache, before_k, before_v, rows, H.TOL["bf16"])
    assert H.rel_err(H.f64(out).transpose(1, 0, 2).reshape(n * steps, -1), ref) <= H.TOL["bf16"]


# one pass over the cache or a step at a time, whichever takes less: many workgroups on short caches, a long row of one kv head, contexts between
@pytest.mark.parametrize("n,kv,G,P,steps,one_pass", [(64, 32, 1, 16, 2, False), (500, 8, 2, 40, 2, False), (64, 32, 1, 16, 16, None), (1, 1, 8, 40000, 2, None),
                                                     (1, 1, 8, 40000, 3, True), (4, 8, 4, 3000, 4, True), (16, 2, 4, 300, 9, True)])
def test_runs_of_decode_steps_one_way_or_the_other(ab, ctx, n, kv, G, P, steps, one_pass):
    ctx.set_option("profile", 1)
    shape = wl.LayerShape(d=256, n_q_heads=kv * G, n_kv_heads=kv, head_dim=128, rank=8, n_adapters=2)
    P = [P - b % 3 for b in range(n)]
    case = H.make_case(shape, P, [steps] * n, [p + b % 2 for b, p in enumerate(P)], [b % 3 - 1 for b in range(n)], seed=3080 + n + steps, prefix="random")
    x = torch.stack([torch.stack([case.x_new[b][t] for b in range(n)]) for t in range(steps)]).cuda().contiguous()
    cache = H.gpu_cache(case)
    before_k, before_v = cache.k.cpu(), cache.v.cpu()
    out = ab.alora_decode_steps(ctx, H.gpu_layer(case, shape), cache, x, case.k, case.adapter)
    torch.cuda.synchronize()
    if one_pass is not None:
        launches = {f: r["launches"] for f, r in ctx.profile_read().items()}
        assert (launches.get("attn_prefill", 0), launches["attn_decode"]) == ((1, 1) if one_pass else (0, steps))
    ref, rows = H.oracle_prefill(case)
    H.check_cache_after(case, cache, before_k, before_v, rows, H.TOL["bf16"])
    assert H.rel_err(H.f64(out).transpose(1, 0, 2).reshape(n * steps, -1), ref) <= H.TOL["bf16"]


# row tiles of 32 that hold one adapter, two and many; few columns of the down-projection per workgroup, and many of them where most have nothing to do
@pytest.mark.parametrize("n,rows,rank,n_adapters", [(8, 125, 64, 8), (1, 1000, 64, 1), (40, 20, 16, 5), (3, 400, 24, 3), (16, 125, 32, 16)])
def test_down_projection_of_row_tiles_with_several_adapters(ab, ctx, n, rows, rank, n_adapters):
    shape = wl.LayerShape(d=512, n_q_heads=2, n_kv_heads=1, head_dim=128, rank=rank, n_adapters=n_adapters)
    P, S = [b % 3 for b in range(n)], [rows - b % 2 for b in range(n)]
    case = H.make_case(shape, P, S, [P[b] + (S[b] // 2 if b % 3 == 2 else 0) for b in range(n)], [b % n_adapters for b in range(n)], seed=3150 + n,
                       prefix="random")
    check_case(ab, ctx, case)


# one range of keys where the row tiles fill the chip by themselves and a merge would cost more than it evens out, several where they do not
@pytest.mark.parametrize("T,P,merged", [(2500, 64, False), (1000, 64, False), (128, 4000, True), (1024, 4096, True)])
def test_ranges_of_prefill_attention(ab, ctx, T, P, merged):
    ctx.set_option("profile", 1)
    shape = wl.LayerShape(d=256, n_q_heads=32, n_kv_heads=8, head_dim=128, rank=8, n_adapters=1)
    case = H.make_case(shape, [P], [T], [P], [0], seed=3170, prefix="random")
    cache = H.gpu_cache(case)
    out = ab.alora_prefill(ctx, H.gpu_layer(case, shape), cache, case.x_packed.cuda().contiguous(), case.cu, case.k, case.adapter)
    torch.cuda.synchronize()
    assert ("attn_merge" in ctx.profile_read()) == merged
    ref, _ = H.oracle_prefill(case)
    assert H.rel_err(H.f64(out), ref) <= H.TOL["bf16"]


# records from the kernel arguments (up to 16 sequences), one per thread, and more than a workgroup has threads; 3 * rank columns in tiles of 8 and of 16
@pytest.mark.parametrize("n,rank,n_adapters", [(16, 8, 2), (17, 24, 3), (512, 8, 1), (513, 8, 2), (700, 16, 2)])
def test_row_preparation_of_many_short_sequences(ab, ctx, n, rank, n_adapters):
    ctx.set_option("prep_split", 2)
    shape = wl.LayerShape(d=512, n_q_heads=2, n_kv_heads=1, head_dim=128, rank=rank, n_adapters=n_adapters)
    P, S = [b % 5 for b in range(n)], [1 + (b % 7 == 3) for b in range(n)]
    case = H.make_case(shape, P, S, [P[b] + (b % 7 == 3) for b in range(n)], [b % (n_adapters + 1) - 1 for b in range(n)], seed=3100 + n,
                       prefix="random")
    check_case(ab, ctx, case)


@pytest.mark.parametrize("records", [2, 3, 4, 5, 6, 7, 8, 9, 11, 16, 17])
@pytest.mark.parametrize("compact", [1, 0])
def test_merge_of_every_number_of_records(ab, records, compact):
    """Ranges that hold keys and, of the short sequence, ranges that hold none (their records have no weight)."""
    shape = wl.LayerShape(d=512, n_q_heads=6, n_kv_heads=3, head_dim=128, rank=16, n_adapters=2)
    case = H.make_case(shape, [1500, 3], [9, 2], [1500, 3], [1, 0], seed=2400 + records, prefix="random")
    c = ab.Context(0)
    c.set_option("kv_splits", records)
    c.set_option("attn_partials16", compact)
    check_case(ab, c, case)
    c.close()


@pytest.mark.parametrize("d,rank", [(4096, 8), (2048, 24)])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 8, 9])
def test_row_preparation_of_up_to_eight_rows(ab, d, rank, T):
    """Normalised rows and t of few rows: outputs against the oracle, base rows' keys and values bit for bit those of a call of many rows."""
    shape = wl.LayerShape(d=d, n_q_heads=4, n_kv_heads=2, head_dim=128, rank=rank, n_adapters=3)
    S = _split(T, min(T, 3))
    n = len(S)
    case = H.make_case(shape, [64, 3, 40][:n], S, [64, 3, 40 + S[-1] // 2][:n], [1, 2, 0][:n], seed=2500 + T + d, prefix="random")
    c = ab.Context(0)
    check_case(ab, c, case)
    x = wl.make_hidden(wl.Rng(2510 + T), "x", 40, shape).cuda()
    layer, rows = H.gpu_layer(case, shape), []
    for m in (T, 40):
        cache = ab.KVCache([40], shape.n_kv_heads, shape.head_dim, shape.torch_dtype, "cuda")
        ab.alora_prefill(c, layer, cache, x[:m].contiguous(), [0, m], [T - 1], [1])      # (the last row of the short call is an adapted one)
        torch.cuda.synchronize()
        rows.append([t.clone() for t in cache.rows(0, 0, T)])
    for a, b in zip(*rows):
        assert torch.equal(a[:T - 1].view(torch.int16), b[:T - 1].view(torch.int16))
    c.close()


@pytest.mark.parametrize("hq,hkv", [(8, 4), (6, 3), (16, 1), (24, 8)])
@pytest.mark.parametrize("P", [[0, 1, 14], [15, 16, 17], [30, 31, 31, 7]])
def test_decode_of_at_most_32_keys(ab, ctx, hq, hkv, P):
    """Steps of 1 to 32 keys an item: the kernel without loads ahead, one block of 16 keys or two."""
    shape = wl.LayerShape(d=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=16, n_adapters=3)
    n = len(P)
    case = H.make_case(shape, P, [1] * n, [max(0, p - 3) for p in P], [b % 4 - 1 for b in range(n)], seed=2600 + n + hq + P[0], prefix="random")
    check_case(ab, ctx, case, decode=True)


@pytest.mark.parametrize("n,rank", [(129, 16), (200, 24)])
def test_static_decode_of_more_rows_than_stream(ab, ctx, n, rank):
    """The step that may allocate projects its rows in tiles, the static one streams the weights past them: the same bits."""
    shape = wl.LayerShape(d=512, n_q_heads=16, n_kv_heads=8, head_dim=128, rank=rank, n_adapters=3)      # (4096 columns: fewer than 3201 are always streamed)
    P = [(7 * b) % 90 for b in range(n)]
    case = H.make_case(shape, P, [1] * n, [max(0, p - 5) for p in P], [b % 4 - 1 for b in range(n)], seed=2700 + n, prefix="random")
    _both(ab, ctx, case)


def _segments_of_a_linear(ab, which, T, d, heads, inter):
    """In how many segments W_o or W_down sums its K products, read off the result: every product is 0 but for 2^32 at k = 0 and, in output column
    j, -2^32 at k = j K / 8 and 64 behind that.  Summed in one segment they leave 64; where the second lies in another segment the 64 is
    less than half a unit of its -2^32 and lost.  (All of it exact in bf16; x, its norm, the attention output and silu(gate) * up are ones.)"""
    kv, h = heads // 4, 128
    K = heads * h if which == "o" else inter
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    t = {"W_qkv": z((heads + 2 * kv) * h, d), "W_o": z(d, heads * h), "W_gate": z(inter, d), "W_up": z(inter, d), "W_down": z(d, inter),
         "rms_gain": torch.ones(d, dtype=torch.bfloat16, device="cuda"), "rms2_gain": torch.ones(d, dtype=torch.bfloat16, device="cuda")}
    W = t["W_o"] if which == "o" else t["W_down"]
    W[:, 0] = 2.0 ** 32
    for n in range(d):
        at = K * (n % 7 + 1) // 8
        W[n, at], W[n, at + 32] = -(2.0 ** 32), 64.0
    if which == "o":
        t["W_qkv"][(heads + kv) * h:, 0] = 1.0      # values of one: so is every average of them
    else:
        t["W_gate"][:, 0], t["W_up"][:, 0] = 32.0, 1 / 32      # silu(32) = 32 in fp32
    layer = ab.Layer(t, heads, kv, h, 1e-5, 10000.0, inter)
    x = torch.ones((T, d), dtype=torch.bfloat16, device="cuda")
    c = ab.Context(0)
    out = ab.alora_stack_prefill(c, [layer], [ab.KVCache([T], kv, h, torch.bfloat16, "cuda")], x, [0, T], [T], [-1])
    torch.cuda.synchronize()
    c.close()
    out = out.float().cpu()
    kept = out[0, :7] == 65.0
    assert torch.equal(out, torch.where(kept.repeat(d // 7 + 1)[:d], 65.0, 1.0).expand(T, d)), out
    segments = {7: 1, 3: 2, 1: 4, 0: 8}[int(kept.sum())]
    assert all(bool(kept[j - 1]) == (j * segments < 8) for j in range(1, 8)), kept
    return segments


# d x K: tiles that fill a round, short ones, a segment of an odd number of k-tiles
@pytest.mark.parametrize("which,d,heads,inter,segments", [("o", 1536, 32, 128, 8), ("down", 1536, 4, 4096, 8), ("down", 1280, 4, 6912, 4),
                                                          ("o", 1024, 8, 128, 2), ("down", 512, 4, 512, 1)])
def test_segments_of_up_to_256_rows_are_those_of_the_weights(ab, which, d, heads, inter, segments):
    """W_o of 1 to 256 rows and W_down of 33 to 256 (fewer are streamed) are cut by the shape of the weights alone: a row's sum does not
    depend on how many rows the call has."""
    for T in ([1, 8, 32] if which == "o" else []) + [33, 64, 65, 128, 129, 200, 256]:
        assert _segments_of_a_linear(ab, which, T, d, heads, inter) == segments, T


# rows -> segments of a W_down of 1024 x 4096 and of 512 x 2048
@pytest.mark.parametrize("d,inter,segments", [(1024, 4096, {257: 4, 640: 4, 1024: 4, 1281: 2, 2049: 1}), (512, 2048, {257: 4, 1024: 4, 2049: 2, 5000: 1})])
def test_segments_of_more_than_256_rows(ab, d, inter, segments):
    """The cut of the reduction is part of the result: it stays when tiles get quicker."""
    assert {T: _segments_of_a_linear(ab, "down", T, d, 4, inter) for T in segments} == segments


# packed rows of an item: one wave's 32 or less (results straight from registers), 33 and more (through LDS), a last wave with one row
@pytest.mark.parametrize("hq,hkv,S", [(4, 4, [1, 32, 33]), (6, 3, [1, 16, 17]), (8, 2, [3, 8, 9]), (16, 2, [1, 4, 5]), (3, 3, [31, 64, 65])])
@pytest.mark.parametrize("splits,compact", [(1, 1), (3, 1), (3, 0)])
def test_prefill_items_of_one_wave_and_of_more(ab, hq, hkv, S, splits, compact):
    shape = wl.LayerShape(d=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=16, n_adapters=2)
    case = H.make_case(shape, [700, 0, 200], S, [700, S[1] // 2, 200], [1, 0, -1], seed=2900 + hq + S[0], prefix="random")
    c = ab.Context(0)
    c.set_option("kv_splits", splits)
    c.set_option("attn_partials16", compact)
    check_case(ab, c, case)
    c.close()


@pytest.mark.parametrize("n,cached", [(1, 20), (3, 2000), (16, 900), (17, 40)])
def test_metadata_carried_beside_base_rows(ab, ctx, n, cached):
    """Calls without adapters, whose first workgroup carries the staged metadata (few sequences) or does not (17)."""
    shape = wl.LayerShape(d=512, n_q_heads=8, n_kv_heads=2, head_dim=128, rank=16, n_adapters=2)
    for S in (1, 5):
        case = H.make_case(shape, [cached + 3 * b for b in range(n)], [S] * n, [0] * n, [-1] * n, seed=2950 + n + S, prefix="random")
        check_case(ab, ctx, case)
