"""Launch forms of the fused kernel: every one gives a (sequence, KV head) the bits it has alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2605_23081_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()
    return binding


def _qkv(B, Hq, Hkv, N, dtype, seed=7):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    mk = lambda H: torch.randn(B, H, N, 128, generator=g, device="cuda")
    q, k, v = mk(Hq), mk(Hkv), mk(Hkv)
    k[:, :, :4] *= 6.0                                                       # sinks, and a direction the queries share
    q += 2.0 * k.mean(2, keepdim=True).repeat_interleave(Hq // Hkv, 1) / 0.1
    return q.to(dtype), k.to(dtype), v.to(dtype)


@pytest.mark.parametrize("B,Hq,Hkv,N,Bq,causal", [
    (2, 16, 16, 1000, 128, True),        # four units on every XCD, interleaved
    (3, 8, 1, 333, 64, True),            # three units, not a multiple of the XCDs
    (1, 8, 2, 65, 128, True),
    (2, 6, 2, 700, 64, False),           # no causal mask: one unit after the other
    (4, 64, 8, 1536, 64, True),          # 3072 workgroups of two query blocks each
    (4, 64, 8, 1537, 64, True),          # 3328, the last of them with one row
])
def test_order_of_the_workgroups(T, B, Hq, Hkv, N, Bq, causal):
    print(f"order of the workgroups B={B} {Hq}/{Hkv} N={N} Bq={Bq} causal={causal}", flush=True)
    q, k, v = _qkv(B, Hq, Hkv, N, torch.bfloat16)
    G = Hq // Hkv
    for order in (0, 1):
        out = T.thrift_attention(q, k, v, causal, Bq, 64, 0.1, tile_order=order)
        for b, h in {(0, 0), (B - 1, Hkv - 1), (B // 2, Hkv // 2)}:
            alone = T.thrift_attention(q[b:b + 1, h * G:(h + 1) * G].contiguous(), k[b:b + 1, h:h + 1].contiguous(),
                                       v[b:b + 1, h:h + 1].contiguous(), causal, Bq, 64, 0.1, tile_order=order)
            assert torch.equal(out[b, h * G:(h + 1) * G], alone[0])


@pytest.mark.parametrize("B,Hq,Hkv,N,Bq,budget", [
    (1, 32, 8, 1025, 128, 0.05),         # 288 workgroups, 17 key blocks: one turn and one block
    (2, 16, 16, 2048, 128, 0.05),        # 512
    (3, 8, 1, 3999, 128, 0.05),          # 768
    (1, 32, 8, 2048, 128, 0.25),         # 512, the wide schedule in ascending order
    (1, 32, 8, 2000, 64, 0.05),          # two query blocks per workgroup
    (1, 32, 8, 1100, 64, 0.05),          # 576 workgroups of one
])
def test_turns_between_workgroups(T, B, Hq, Hkv, N, Bq, budget):
    """Rows of one length in a grid of one round: the workgroups' priorities change nothing but the time."""
    print(f"turns B={B} {Hq}/{Hkv} N={N} Bq={Bq} f={budget}", flush=True)
    q, k, v = _qkv(B, Hq, Hkv, N, torch.float16)
    G = Hq // Hkv
    for order in (0, 1):
        out = T.thrift_attention(q, k, v, False, Bq, 64, budget, tile_order=order, out_dtype=torch.float32)
        for b in range(B):
            for h in range(Hkv):
                heads = slice(h * G, (h + 1) * G)
                alone = T.thrift_attention(*(x[b:b + 1, s].contiguous() for x, s in ((q, heads), (k, slice(h, h + 1)), (v, slice(h, h + 1)))),
                                           False, Bq, 64, budget, tile_order=order, out_dtype=torch.float32)
                assert torch.equal(out[b, heads], alone[0])


@pytest.mark.parametrize("Hq,Hkv,Nq,N,Bq,budget", [
    (32, 8, 1100, 2380, 128, 0.05),      # 288 workgroups; rows of 21 to 38 key blocks, the last of them short
    (16, 16, 2048, 4096, 128, 0.1),      # 256: one per CU, no turns
    (32, 8, 2000, 4048, 128, 0.05),      # 512
    (32, 8, 2000, 4048, 128, 0.25),      # the wide schedule in ascending order
    (32, 8, 3072, 5120, 128, 0.0),       # 768, no block promoted
    (32, 8, 2000, 4048, 64, 0.05),       # two query blocks per workgroup
    (32, 8, 1100, 2380, 64, 0.25),       # 576 workgroups of one
])
def test_turns_between_workgroups_of_a_chunk(T, Hq, Hkv, Nq, N, Bq, budget):
    """Behind cached tokens the rows are nearly equal in length and take turns as well; every KV head has the bits of a call of its own."""
    print(f"turns in a chunk of {Nq} of {N} {Hq}/{Hkv} Bq={Bq} f={budget}", flush=True)
    q, k, v = _qkv(1, Hq, Hkv, N, torch.bfloat16)
    q = q[:, :, :Nq].contiguous()
    G, off = Hq // Hkv, (N - Nq) // Bq
    assert N - Nq == off * Bq

    def run(q, k, v, order):
        idx, cnt = T.thrift_select_topk(T.thrift_block_means(q, Bq), T.thrift_block_means(k, 64), Bq, 64, True, budget, q_block_offset=off)
        codes = [*T.thrift_quantize_mxfp4(q, 0), *T.thrift_quantize_mxfp4(k, 0), *T.thrift_quantize_mxfp4(v, 1)]
        return T.thrift_attn_prefill_chunk(q, k, v, *codes, idx, cnt, Bq, 64, True, off, out_dtype=torch.float32, tile_order=order)

    for order in (0, 1):
        out = run(q, k, v, order)
        assert bool(torch.isfinite(out).all())
        for h in {0, Hkv // 2, Hkv - 1}:
            heads = slice(h * G, (h + 1) * G)
            alone = run(*(x.contiguous() for x in (q[:, heads], k[:, h:h + 1], v[:, h:h + 1])), order)
            assert torch.equal(out[0, heads], alone[0])


def _form(B, Hq, Nq, N, kmax):
    """Row groups per workgroup of the four-wavefront kernel, 0: the plain one (launch_prefill_split's rule)."""
    groups, Tk = B * Hq * -(-Nq // 32), -(-N // 64)
    if kmax * 100 >= Tk * 15:
        return 0
    return 1 if groups <= 256 else 2 if groups <= 512 and Tk >= 10 else 0


@pytest.mark.parametrize("B,Hq,Hkv,N,Bq", [
    (1, 32, 8, 1024, 128),               # 256 workgroups: one third, as it comes
    (1, 32, 8, 1025, 128),               # 288: a second third of 32
    (3, 11, 11, 1153, 128),              # 330, units not a multiple of the XCDs
    (2, 16, 16, 2048, 128),              # 512
    (1, 32, 8, 3072, 128),               # 768
    (1, 32, 8, 3073, 128),               # 800: more than the chip holds, as it comes
    (1, 32, 8, 1500, 64),                # 768 of two wavefronts, one query block of 64 rows each
    (1, 32, 8, 2700, 64),                # 704 of two query blocks each, the last of them with one
])
def test_folded_order_of_the_workgroups(T, B, Hq, Hkv, N, Bq, budget=0.1):
    """Grids of one round, whose second third runs the other way: every head has the bits it has in a call of its own."""
    print(f"folded order B={B} {Hq}/{Hkv} N={N} Bq={Bq} f={budget}", flush=True)
    q, k, v = _qkv(B, Hq, Hkv, N, torch.bfloat16)
    G = Hq // Hkv
    for order in (0, 1, 2):
        out = torch.full((B, Hq, N, 128), float("nan"), device="cuda")
        T.thrift_attention(q, k, v, True, Bq, 64, budget, tile_order=order, out=out)
        for b in range(B):
            for h in range(Hkv):
                heads = slice(h * G, (h + 1) * G)
                alone = T.thrift_attention(*(x[b:b + 1, s].contiguous() for x, s in ((q, heads), (k, slice(h, h + 1)), (v, slice(h, h + 1)))),
                                           True, Bq, 64, budget, tile_order=order, out_dtype=torch.float32)
                assert torch.equal(out[b, heads], alone[0])


@pytest.mark.parametrize("N", [2048, 2100, 3072])                            # 512, 544 and 768 workgroups, of which a CU holds two
def test_folded_order_of_the_wide_schedule(T, N):
    test_folded_order_of_the_workgroups(T, 1, 32, 8, N, 128, 0.25)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("Hq,Hkv,N,Bq,causal,copies,form", [
    (1, 1, 385, 64, True, 50, 1),         # seven key blocks, the fewest: groups of four and three; one key and one row in the last
    (2, 1, 448, 128, False, 30, 1),       # the same, all whole; every row sees every block
    (1, 1, 513, 64, True, 40, 1),         # nine: the last group of key blocks is one block
    (2, 1, 700, 128, True, 20, 1),        # four row groups per query block, of which the last has none
    (3, 1, 1100, 64, False, 8, 1),        # every row sees every block
    (8, 2, 1024, 128, True, 4, 1),        # 256 row groups, the most with one per workgroup
    (8, 8, 1025, 128, True, 2, 2),        # 264: two row groups per workgroup
    (16, 16, 577, 64, False, 2, 2),       # ten key blocks, the fewest with two; a last workgroup of one row group of one row
    (16, 4, 640, 128, True, 2, 2),        # ten whole ones
    (16, 4, 609, 64, True, 2, 2),         # both row groups of the last workgroup, one of them with one row
    (4, 1, 4095, 64, True, 2, 2),         # 512 row groups, the most
    (16, 16, 576, 64, True, 2, 0),        # nine key blocks: the plain kernel
])
def test_four_wavefronts_per_row_group(T, Hq, Hkv, N, Bq, causal, copies, form, dtype):
    """The same sequence alone and in a batch that is large enough for the plain kernel: equal bits, LSE included, for lists up
    to 15 % of the key blocks (none, some, neighbouring blocks)."""
    print(f"four wavefronts per row group {Hq}/{Hkv} N={N} Bq={Bq} causal={causal} {dtype}", flush=True)
    q, k, v = _qkv(1, Hq, Hkv, N, dtype)
    Tk = -(-N // 64)
    ks = sorted({0, max(1, Tk // 20), max(0, (15 * Tk - 1) // 100)})
    many = [t.expand(copies, -1, -1, -1).contiguous() for t in (q, k, v)]
    for fixed_k in ks:
        assert _form(1, Hq, N, N, max(1, fixed_k)) == form and _form(copies, Hq, N, N, max(1, fixed_k)) == 0
        for order in (0, 1):
            lse, lse_n = torch.full((1, Hq, N), 7.0, device="cuda"), torch.full((copies, Hq, N), 7.0, device="cuda")
            a = T.thrift_attention(q, k, v, causal, Bq, 64, fixed_k=fixed_k, tile_order=order, lse=lse)
            b = T.thrift_attention(*many, causal, Bq, 64, fixed_k=fixed_k, tile_order=order, lse=lse_n)
            assert bool(torch.isfinite(a).all())
            for c in {0, copies - 1}:
                assert torch.equal(a[0], b[c]) and torch.equal(lse[0], lse_n[c])


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("Nq,off,N,ids,form", [
    (128, 30, 4000, [0, 1, 2, 3, 7, 8], 1),                                  # promoted blocks that follow each other
    (100, 15, 2050, [31, 32], 1),                                            # the last blocks, of which one is short
    (64, 31, 4096, [0, 62, 63], 1),                                          # some blocks after the rows' own
    (2113, 15, 4090, [0, 1, 2, 3, 7, 8, 62, 63], 2),                         # two row groups per workgroup; all of it
])
def test_four_wavefronts_per_row_group_in_a_chunk(T, Nq, off, N, ids, form, order):
    print(f"four wavefronts, chunk of {Nq} at {off} in {N}, ids {ids}, order {order}", flush=True)
    q, k, v = _qkv(1, 4, 2, N, torch.bfloat16)
    q = q[:, :, :Nq].contiguous()
    idx = torch.tensor(ids, dtype=torch.int32, device="cuda").expand(1, 4, -(-Nq // 128), -1).contiguous()
    cnt = torch.full(idx.shape[:3], len(ids), dtype=torch.int32, device="cuda")

    def run(n):
        a, b, c = (t.expand(n, -1, -1, -1).contiguous() for t in (q, k, v))
        codes = [*T.thrift_quantize_mxfp4(a, 0), *T.thrift_quantize_mxfp4(b, 0), *T.thrift_quantize_mxfp4(c, 1)]
        return T.thrift_attn_prefill_chunk(a, b, c, *codes, idx.expand(n, -1, -1, -1).contiguous(), cnt.expand(n, -1, -1).contiguous(),
                                           128, 64, True, off, tile_order=order)

    copies = 80 if form == 1 else 2
    assert _form(1, 4, Nq, N, len(ids)) == form and _form(copies, 4, Nq, N, len(ids)) == 0
    alone, many = run(1), run(copies)
    assert bool(torch.isfinite(alone).all()) and torch.equal(alone[0], many[0]) and torch.equal(alone[0], many[copies - 1])


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("Nq,off,N,even,odd", [
    (64, 0, 64, [0], []),                                                     # one query block: the other list does not exist
    (65, 0, 65, [0], [0, 1]),                                                 # one row in the second
    (128, 0, 1000, [1, 3, 5, 7], [2, 4, 6, 8]),                               # neighbours in turn: a promoted block behind every one
    (192, 5, 1000, [], [0, 1, 2, 3]),                                         # a run of one list alone; an odd offset and number of blocks
    (577, 3, 1024, [0, 1, 2, 9, 15], [1, 2, 3, 4, 10, 15]),                   # overlapping runs
    (640, 6, 1024, list(range(16)), [0, 4, 8, 12, 13]),                       # one list has everything
    (640, 0, 640, list(range(10)), list(range(10))),                          # no 4-bit block at all
    (333, 4, 700, [9, 10], []),                                               # the last blocks, of which one is short
])
def test_two_query_blocks_per_workgroup(T, Nq, off, N, even, odd, causal, order):
    """Query blocks of 64 rows go in pairs, each with its own list, where the grid is large: every row has the bits it has in a
    query block of 128 rows with its list."""
    print(f"two query blocks per workgroup: {Nq} at {off} in {N}, {even} / {odd}, causal {causal}, order {order}", flush=True)
    dtype = torch.bfloat16 if N % 2 else torch.float16
    q, k, v = _qkv(1, 4, 2, N, dtype)
    q = q[:, :, :Nq].contiguous()
    Tq, Tk = -(-Nq // 64), -(-N // 64)
    lists = torch.full((2, Tk), -1, dtype=torch.int32, device="cuda")         # as wide as the row: the plain kernel at any size
    for i, ids in enumerate((even, odd)):
        lists[i, :len(ids)] = torch.tensor(ids, dtype=torch.int32)
    count = torch.tensor([len(even), len(odd)], dtype=torch.int32, device="cuda")
    codes = [*T.thrift_quantize_mxfp4(q, 0), *T.thrift_quantize_mxfp4(k, 0), *T.thrift_quantize_mxfp4(v, 1)]

    def run(which, Bq, off, n=1):
        lse = torch.zeros(n, 4, Nq, device="cuda")
        many = [t.expand(n, *t.shape[1:]).contiguous() for t in (q, k, v, *codes)]
        out = T.thrift_attn_prefill_chunk(*many, lists[which].expand(n, 4, -1, -1).contiguous(),
                                          count[which].expand(n, 4, -1).contiguous(), Bq, 64, causal, off,
                                          out_dtype=torch.float32, lse=lse, tile_order=order)
        assert torch.equal(out[0], out[n - 1]) and torch.equal(lse[0], lse[n - 1])
        return out[:1], lse[:1]

    copies = 6 * 256 // (4 * Tq) + 1                                          # past the grids that take one block to a workgroup
    both, lse = run(torch.arange(Tq, device="cuda") % 2, 64, off, copies)
    one, lse_one = run(torch.arange(Tq, device="cuda") % 2, 64, off)          # one of those
    assert torch.equal(both, one) and torch.equal(lse, lse_one)
    assert bool(torch.isfinite(both).all())
    if off % 2:                                                               # 128-row blocks start at even offsets only
        pad = torch.cat([torch.zeros_like(q[:, :, :64]), q], 2)
        q, Nq, off = pad.contiguous(), Nq + 64, off - 1
        codes[:2] = T.thrift_quantize_mxfp4(q, 0)
        both, lse = torch.nn.functional.pad(both, (0, 0, 64, 0)), torch.nn.functional.pad(lse, (64, 0))
        skip = 64
    else:
        skip = 0
    zero = torch.zeros(-(-Nq // 128), dtype=torch.long, device="cuda")
    for which in (0, 1):
        alone, lse_1 = run(zero + which, 128, off // 2)
        mine = (torch.arange(skip, Nq, device="cuda") - skip) // 64 % 2 == which
        assert torch.equal(both[:, :, skip:][:, :, mine], alone[:, :, skip:][:, :, mine])
        assert torch.equal(lse[:, :, skip:][:, :, mine], lse_1[:, :, skip:][:, :, mine])


def test_order_of_the_largest_interleaved_grid(T):
    test_order_of_the_workgroups(T, 4, 64, 8, 3072, 64, True)                 # 6144 workgroups of two query blocks each
    test_order_of_the_workgroups(T, 4, 64, 8, 3073, 64, True)                 # and the next, one unit after the other
