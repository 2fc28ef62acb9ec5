"""The decode in finer pieces (two passes over chunks, in two launches or one; short caches, few sequences) against the oracle and
against the walk over whole partitions, here the one-pass form.

Both forms give every block the running maximum of its partition and the same selection.  Their raw scores come from matrix
instructions of different shapes.  16-bit scores had equal bits in every comparison; 4-bit scores are sums of 128 products
that fp32 holds exactly where a row's products of group scales lie within 2^9 of each other, and none of two million with
these inputs' outlier channels differed.  The codes of P are then the same, and the fp32 results differ by the order of the
sums and of the rescaling factors alone, a few 2^-24 per addition over at most some hundred partials, whatever the input type.  A workspace that is too small for the two-pass form selects the one-pass
form.
"""
import numpy as np
import pytest
import torch

from paper_2605_23081_amd import workloads as W
from tests.test_gpu_parity import TOLMIX, _decode_case

pytestmark = pytest.mark.gpu

REL = 4e-6          # 2-norm: 64 x 2^-24, for sums of about 128 partials and blocks and the last bits of the exponentials


@pytest.fixture(scope="module")
def T():
    from paper_2605_23081_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()
    return binding


def _cache(T, wl):
    q, k, v = W.make_decode(wl, device="cuda")
    k4, ks = T.thrift_quantize_mxfp4(k, 0)
    v4, vs = T.thrift_quantize_mxfp4(v, 1)
    return q, k, v, k4, ks, v4, vs, T.thrift_block_means(k, wl.Bk)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("Hq,Hkv,B,N,split,lens,budget", [
    (1, 1, 1, 64, 256, None, 0.05),                                          # one key block
    (4, 2, 3, 1152, 256, [1152, 1, 0], 0.05),                                # a full cache, one token, none
    (6, 2, 2, 2048, 23, [2047, 1024], 0.25),                                 # partitions that end inside a workgroup's blocks
    (10, 2, 2, 1600, 17, [1537, 63], 1.0),                                   # five heads of eight columns, every block promoted
    (16, 2, 2, 4096, 256, [4095, 2049], 0.0),                                # eight heads, no block promoted
    (7, 1, 1, 4096, 40, None, 0.1),
    (32, 8, 2, 5376, 256, [5376, 4000], 1.0),                                # one launch, 2 key blocks per wavefront; 1 in shorter rows
    (32, 8, 16, 640, 256, [640 - 37 * b for b in range(16)], 0.1),
    (32, 8, 2, 16384, 100, [16384, 9000], 0.05),                             # 2 key blocks per wavefront
    (8, 8, 2, 65536, 256, [65535, 40001], 0.05),                             # 4
    (16, 8, 2, 131072, 250, [131072, 70000], 0.25),                          # 8
    (32, 8, 4, 16896, 256, [16896 - 1500 * b for b in range(4)], 0.25),      # 4 in two launches, above 8192 key blocks; a partition of 8
    (16, 8, 2, 36864, 256, None, 0.05),                                      # 9216, the most in two launches
    (64, 8, 2, 40960, 250, [40959, 33000], 0.1),                             # 10240, the most with eight heads
    (16, 16, 11, 2176, 17, [2176 - 197 * b for b in range(11)], 0.25),       # one head per KV head: 352 partitions
    (16, 16, 16, 2176, 17, [2175] * 16, 0.05),                               # 512, the most
])
def test_two_pass_decode_equals_one_pass(T, Hq, Hkv, B, N, split, lens, budget, dtype):
    print(f"decode split Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} lens={lens} budget={budget} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv, dtype=dtype)
    args = _cache(T, wl)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    need = T.decode_workspace_bytes(B, Hq, Hkv, N, wl.D, 64, split)
    big, small = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda"), torch.full((need - 256,), 0xFF, dtype=torch.uint8, device="cuda")
    kw = dict(split_blocks=split, seqlens=sl, out_dtype=torch.float32, return_selection=True)
    two, idx2, cnt2 = T.thrift_attn_decode(*args, 64, budget, workspace=big, **kw)
    one, idx1, cnt1 = T.thrift_attn_decode(*args, 64, budget, workspace=small, **kw)
    assert torch.equal(idx1, idx2) and torch.equal(cnt1, cnt2)
    assert bool(torch.isfinite(two).all())
    err = float((two - one).norm() / one.norm().clamp_min(1e-30))
    print(f"  rel {err:.2e}", flush=True)
    assert err <= REL
    again, _, _ = T.thrift_attn_decode(*args, 64, budget, workspace=big, **kw)
    assert torch.equal(two, again)


@pytest.mark.parametrize("Hq,Hkv,B,N,split,lens,budget", [
    (32, 8, 1, 32768, 256, [31937], 0.05),                                   # places whose last wavefronts have no block
    (4, 4, 3, 16448, 256, [16448, 8321, 577], 0.25),                         # one head
    (16, 2, 2, 32768, 509, [32767, 16385], 0.1),                             # more maxima in front than are asked for at once
    (64, 8, 2, 40960, 250, [40959, 33000], 0.1),                             # a selection of its own launch
    (8, 4, 2, 5376, 37, [5375, 2368], 0.0),                                  # no block promoted
])
def test_two_launches_in_any_workspace(T, Hq, Hkv, B, N, split, lens, budget):
    """What is asked for before the length is known may never have been written: the results do not depend on what lies there."""
    print(f"decode in any workspace Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} budget={budget}", flush=True)
    args = _cache(T, W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv))
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.empty(T.decode_workspace_bytes(B, Hq, Hkv, N, 128, 64, split), dtype=torch.uint8, device="cuda")
    outs = []
    for fill in (0, 0xFF, 0x7F, 0x55):                                       # 0x7F7F7F7F: a larger maximum than any
        ws.fill_(fill)
        outs.append(T.thrift_attn_decode(*args, 64, budget, split_blocks=split, seqlens=sl, workspace=ws,
                                         out=torch.empty(B, Hq, 128, dtype=torch.float32, device="cuda")))
        assert bool(torch.isfinite(outs[-1]).all()) and torch.equal(outs[-1], outs[0])


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("Hq,Hkv,B,N,split,lens,budget,shared", [
    (8, 8, 9, 8192, 256, [8192 - 517 * b for b in range(9)], 0.05, False),   # 9216 key blocks: one launch; it selects for itself
    (12, 4, 17, 8192, 31, [8191 - 481 * b for b in range(17)], 0.25, False),             # rows of two registers, partitions of 31 blocks
    (40, 8, 9, 8192, 256, None, 0.1, True),                                  # five heads, one set for them; no lengths
    (16, 16, 5, 8256, 129, [8256, 8255, 64, 1, 0], 0.05, False),             # 129 key blocks: one more than it selects itself
    (14, 2, 5, 65536, 256, [65535 - 13000 * b for b in range(5)], 0.1, False),           # seven heads
    (16, 8, 6, 16384, 100, [16384, 9000, 0, 6463, 6400, 6401], 0.0, False),  # no block promoted: no selection clears the tickets
    (32, 4, 9, 16384, 256, [16384] * 9, 1.0, False),                         # every block
    (8, 2, 56, 32768, 512, [32768 - 577 * b for b in range(56)], 0.05, False),           # longer partitions; 112
    (16, 8, 28, 32768, 256, None, 0.05, False),                              # 448 partitions, the most
    (32, 8, 16, 8192, 256, [8192 - 333 * b for b in range(16)], 0.05, False),            # four heads, eight blocks per wavefront
    (32, 8, 3, 32768, 256, [32767, 20000, 16384], 0.1, False),               # the same, selected by a launch of its own
])
def test_both_passes_in_one_launch_equal_the_walk(T, Hq, Hkv, B, N, split, lens, budget, shared, dtype):
    """Many key blocks, or short rows.  The workspace starts from bytes that look like published maxima and tickets (zeros), like
    maxima still to come (ones) and from what the call before has left."""
    print(f"decode in one launch Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} budget={budget} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv, dtype=dtype)
    assert B * Hkv * (N // 64) > 8192
    args = _cache(T, wl)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    size = B, Hq, Hkv, N, wl.D, 64, split
    need, least = T.decode_workspace_bytes(*size), T.decode_least_workspace_bytes(*size)
    assert need > least
    kw = dict(split_blocks=split, seqlens=sl, group_shared=shared)
    run = lambda ws: T.thrift_attn_decode(*args, 64, budget, out=torch.empty(B, Hq, 128, dtype=torch.float32, device="cuda"), workspace=ws, **kw)
    one = run(torch.empty(least, dtype=torch.uint8, device="cuda"))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    got = []
    for fill in (0, 0xFF, None, 0x55):
        if fill is not None:
            ws.fill_(fill)
        got.append(run(ws))
    assert bool(torch.isfinite(got[0]).all()) and all(torch.equal(x, got[0]) for x in got)
    err = float((got[0] - one).norm() / one.norm())
    print(f"  rel {err:.2e}", flush=True)
    assert err <= REL
    listed, _, _ = T.thrift_attn_decode(*args, 64, budget, out_dtype=torch.float32, return_selection=True, workspace=ws, **kw)
    assert torch.equal(listed, got[0])                                       # selected by a launch of its own


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("Hq,Hkv,B,N,split,lens", [
    (32, 8, 2, 6144, 256, [6143, 5000]),                                     # 1536 key blocks: the most in two launches of short rows, ..
    (24, 8, 2, 6208, 23, [6208, 77]),                                        # .. and one launch above
    (16, 16, 16, 8192, 256, [8192 - 300 * b for b in range(16)]),            # one head, 32768, the most in two; 8 per wavefront
    (16, 16, 17, 8192, 256, None),
    (16, 8, 2, 40960, 256, [40959, 20000]),                                  # two heads, 10240, the most in two
    (16, 8, 3, 28672, 100, None),
    (64, 8, 2, 51200, 256, [51200, 44444]),                                  # eight heads, 12800, the most in two of long rows
    (40, 8, 3, 34816, 250, [34815, 1, 30000]),
])
def test_no_promoted_block(T, Hq, Hkv, B, N, split, lens, dtype):
    """The form without promoted blocks, on both sides of its rules, against the walk; with and without the (empty) lists, over any
    bytes in the workspace."""
    print(f"decode without promoted blocks Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} lens={lens} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv, dtype=dtype)
    args = _cache(T, wl)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    size = B, Hq, Hkv, N, wl.D, 64, split
    need, least = T.decode_workspace_bytes(*size), T.decode_least_workspace_bytes(*size)
    kw = dict(split_blocks=split, seqlens=sl, out_dtype=torch.float32, return_selection=True)
    one, idx, cnt = T.thrift_attn_decode(*args, 64, 0.0, workspace=torch.full((least,), 0xFF, dtype=torch.uint8, device="cuda"), **kw)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    got, idx2, cnt2 = T.thrift_attn_decode(*args, 64, 0.0, workspace=ws, **kw)
    assert int(cnt.sum()) == 0 and torch.equal(cnt, cnt2) and torch.equal(idx, idx2)
    assert bool(torch.isfinite(got).all()) and float((got - one).norm() / one.norm()) <= REL
    for fill in (0, None, 0xFF):
        if fill is not None:
            ws.fill_(fill)
        out = torch.full_like(got, float("nan"))
        T.thrift_attn_decode(*args, 64, 0.0, split_blocks=split, seqlens=sl, out=out, workspace=ws)
        assert torch.equal(out, got)


@pytest.mark.parametrize("Hq,Hkv,B,N,split,lens", [
    (1, 1, 2, 4096, 256, [4095, 4096 - 64]),                                 # one head, 16 workgroups or more per partition
    (12, 4, 3, 8192, 31, [8191, 2000, 64]),                                  # three heads; partitions of one workgroup and of several
    (16, 2, 9, 8192, 256, None),                                             # eight
])
def test_a_wait_without_an_answer_gives_nan(T, Hq, Hkv, B, N, split, lens):
    """One launch, whose workgroups may not ask once for the largest scores in front of them: NaN wherever a partition has more
    than one workgroup, never numbers that lack what was not waited for; then, asking, the results again."""
    print(f"decode without answers Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} lens={lens}", flush=True)
    import ctypes as C
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv)
    assert N // 64 <= 128                                                    # short rows: one launch whatever the grid
    args = _cache(T, wl)
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.empty(T.decode_workspace_bytes(B, Hq, Hkv, N, 128, 64, split), dtype=torch.uint8, device="cuda")
    call = T.lib().thrift_test_attn_decode_polls
    call.argtypes = [*T.lib().thrift_attn_decode.argtypes, C.c_int]

    def run(polls):
        out = torch.full((B, Hq, 128), 7.0, dtype=torch.float32, device="cuda")
        code = call(args[0].data_ptr(), T.F16 if args[0].dtype == torch.float16 else T.BF16, *(t.data_ptr() for t in args[1:]),
                    None if sl is None else sl.data_ptr(), B, Hq, Hkv, N, 128, 64, 0.1, -1, split, 0.0, out.data_ptr(), T.F32, None, None, 0,
                    ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream, polls)
        assert code == 0
        return out

    want = torch.empty(B, Hq, 128, dtype=torch.float32, device="cuda")
    T.thrift_attn_decode(*args, 64, 0.1, split_blocks=split, seqlens=sl, out=want, workspace=ws)
    assert bool(torch.isfinite(want).all())
    got = run(0)
    nan = torch.isnan(got)
    for b in range(B):
        blocks = (N if lens is None else lens[b]) // 64
        assert bool(nan[b].all()) if min(blocks, split) > 32 else torch.equal(got[b], want[b]) or bool(nan[b].all())     # 4 x 8 blocks at most per workgroup
    assert torch.equal(run(1 << 19), want)


def test_calls_in_one_launch_on_two_streams(T):
    """Workgroups that wait for each other, of two calls at a time with a workspace each, more than the chip holds: every call gives
    what it gives alone."""
    print("decode in one launch on two streams", flush=True)
    calls = []
    for Hq, Hkv, B, N, budget in ((32, 8, 16, 16384, 0.05), (16, 16, 12, 8192, 0.25)):
        args = _cache(T, W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv))
        sl = torch.tensor([N - 731 * b for b in range(B)], dtype=torch.int32, device="cuda")
        ws = torch.empty(T.decode_workspace_bytes(B, Hq, Hkv, N, 128, 64, 256), dtype=torch.uint8, device="cuda")
        outs = [torch.full((B, Hq, 128), float("nan"), dtype=torch.float32, device="cuda") for _ in range(21)]
        run = lambda out, args=args, budget=budget, sl=sl, ws=ws: T.thrift_attn_decode(*args, 64, budget, seqlens=sl, out=out, workspace=ws)
        run(outs[0])
        calls.append((run, outs, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for n in range(1, 21):
        for run, outs, stream in calls:
            with torch.cuda.stream(stream):
                run(outs[n])
    torch.cuda.synchronize()
    for _, outs, _ in calls:
        assert bool(torch.isfinite(outs[0]).all()) and all(torch.equal(x, outs[0]) for x in outs)


@pytest.mark.parametrize("Hq,Hkv,B,N", [(32, 8, 9, 8192), (8, 2, 2, 4096)])
def test_decode_in_a_graph(T, Hq, Hkv, B, N):
    """Tickets and maxima are cleared inside the call: every replay gives what the eager call gives, on new values too."""
    print(f"decode in a graph Hq={Hq} Hkv={Hkv} B={B} N={N}", flush=True)
    args = list(_cache(T, W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv)))
    ws = torch.empty(T.decode_workspace_bytes(B, Hq, Hkv, N, 128, 64, 256), dtype=torch.uint8, device="cuda")
    sl = torch.full((B,), N - 5, dtype=torch.int32, device="cuda")
    for budget in (0.05, 0.0):
        out, kw = torch.empty_like(args[0]), dict(seqlens=sl, workspace=ws)
        T.thrift_attn_decode(*args, 64, budget, out=out, **kw)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            T.thrift_attn_decode(*args, 64, budget, out=out, **kw)
        for n in range(3):
            args[0].mul_(0.75)
            sl.sub_(61)
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            want = T.thrift_attn_decode(*args, 64, budget, seqlens=sl)
            assert torch.equal(out, want)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("Hq,Hkv,B,N,split,lens,budget", [
    (8, 2, 2, 1536, 256, None, 0.1), (5, 1, 1, 1024, 256, [833], 0.25), (8, 1, 2, 2048, 24, [2048, 1300], 0.05), (3, 3, 1, 704, 256, None, 1.0),
    (4, 2, 1, 1344, 256, None, 0.1), (6, 2, 2, 1024, 256, [1024, 300], 0.25),
])
def test_two_pass_decode_matches_the_oracle(T, Hq, Hkv, B, N, split, lens, budget, dtype):
    from oracle import thrift_oracle as oracle
    print(f"decode split vs oracle Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} lens={lens} budget={budget} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv, dtype=dtype)
    lens = None if lens is None else [n // 64 * 64 for n in lens]            # the helper's selection takes whole blocks
    got, want, swaps = _decode_case(T, oracle, wl, budget, split, lens)
    assert swaps == 0 and np.abs(got - want).max() <= TOLMIX


@pytest.mark.parametrize("Hq,Hkv,B,N,split,dtype", [
    (8, 2, 1, 69632, 1088, "f16"), (8, 2, 1, 36864, 576, "bf16"),             # one head per wavefront
    (16, 2, 1, 40960, 640, "f16"), (16, 2, 1, 36864, 576, "bf16"),            # two
])
def test_walk_reloads_its_window(T, Hq, Hkv, B, N, split, dtype):
    """The one-pass form over partitions longer than its window of cached selection words (512 key blocks)."""
    from oracle import thrift_oracle as oracle
    print(f"decode walk Hq={Hq} Hkv={Hkv} B={B} N={N} split={split} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv, dtype=dtype)
    got, want, swaps = _decode_case(T, oracle, wl, 0.1, split, one_pass=True)
    assert swaps == 0 and np.abs(got - want).max() <= TOLMIX


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8])
def test_what_lies_past_the_tokens_is_not_read(T, G, dtype):
    """Lengths that leave the last key block partly filled, in a cache whose unwritten bytes are all ones (NaN in every type,
    an E8M0 scale of NaN) or zeros: the same bits, in both forms, which agree with each other."""
    lens, Hkv, cap = [4095, 2049 + 31, 1985, 161, 64, 33, 1], 2, 4096
    B, Hq = len(lens), G * Hkv
    print(f"decode past the tokens G={G} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=cap, Hq=Hq, Hkv=Hkv, dtype="f16" if dtype == torch.float16 else "bf16")
    q, k, v = W.make_decode(wl, device="cuda")
    need = T.decode_workspace_bytes(B, Hq, Hkv, cap, 128, 64, 256)
    caches = [T.KVCache(B, Hkv, cap, 128, 64, dtype, "cuda", fill=fill) for fill in (0xFF, 0)]
    for c in caches:
        c.append(k, v, torch.tensor(lens, dtype=torch.int32, device="cuda"))
    for budget in (0.0, 0.25, 1.0):
        one, two = ([T.thrift_attn_decode(q, c.k16, c.v16, c.k4, c.ks, c.v4, c.vs, c.kmean, 64, budget, seqlens=c.seqlens,
                                          out_dtype=torch.float32, return_selection=True,
                                          workspace=torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda"))[0] for c in caches]
                    for n in (need - 256, need))
        assert bool(torch.isfinite(two[0]).all()) and torch.equal(two[0], two[1]) and torch.equal(one[0], one[1])
        assert float((two[0] - one[0]).norm() / one[0].norm()) <= REL


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("Hq,Hkv,B,N,lens,budget,fixed_k,shared,ties", [
    (4, 1, 1, 64, None, 0.05, -1, False, False),                              # one key block
    (8, 2, 3, 4096, [4096, 1, 0], 0.05, -1, False, False),                    # a full row, one token, none
    (6, 2, 2, 4160, [4159, 4097], 0.25, -1, False, False),                    # three rows; one block past the first word
    (2, 2, 2, 32768, [32768, 32705], 0.1, -1, False, False),                  # all eight words; a partly filled last block
    (8, 2, 1, 8192, [8191], 1.0, -1, False, False),                           # every block
    (8, 2, 2, 8192, [8000, 130], 0.0, 7, False, False),                       # a fixed count, more than the second row has
    (8, 2, 2, 16384, [16384, 9001], 0.05, -1, True, False),                   # one set per KV head
    (4, 1, 1, 8192, None, 0.1, -1, False, True),                              # equal keys: the smaller ids
])
def test_selection_inside_the_scores_pass(T, Hq, Hkv, B, N, lens, budget, fixed_k, shared, ties, dtype):
    """Without lists to write, the scores pass selects for itself; the kernel that writes the lists selects the same blocks:
    equal bits of the results."""
    print(f"decode selection in the pass Hq={Hq} Hkv={Hkv} B={B} N={N} lens={lens} f={budget} k={fixed_k} {shared} {ties} {dtype}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=B, N=N, Hq=Hq, Hkv=Hkv, dtype=dtype)
    args = list(_cache(T, wl))
    if ties:
        args[7] = args[7][:, :, :1].expand_as(args[7]).contiguous()
    sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.full((T.decode_workspace_bytes(B, Hq, Hkv, N, wl.D, 64, 256),), 0xFF, dtype=torch.uint8, device="cuda")
    kw = dict(fixed_k=fixed_k, seqlens=sl, workspace=ws, group_shared=shared)
    want, _, _ = T.thrift_attn_decode(*args, 64, budget, out_dtype=torch.float32, return_selection=True, **kw)
    for _ in range(2):
        ws.fill_(0xFF)
        out = torch.empty_like(want)
        T.thrift_attn_decode(*args, 64, budget, out=out, **kw)
        assert torch.equal(out, want)


@pytest.mark.parametrize("Tk", [1, 64, 65, 256, 257, 512, 513, 1025, 2048, 2049, 4096])
def test_listed_selection_is_the_k_largest(T, Tk):
    """The selection of a launch of its own against a stable sort: scores that its bins separate, that crowd one bin, that fp32 does
    not tell apart, that tie or are infinite.  The query's first two channels alone are not zero, so that the scores are exact."""
    print(f"decode listed selection Tk={Tk}", flush=True)
    gen = torch.Generator().manual_seed(Tk)
    normal = torch.randn(Tk, generator=gen, dtype=torch.float64)
    j = torch.randperm(Tk, generator=gen).double()
    rows = {                                                                 # (first, second channel of the key block means)
        "normal": (normal, None),
        "outlier": (torch.where(j == 0, 1e30, normal), None),
        "geometric": (torch.exp2(-(j % 120)) * torch.where(j % 2 == 0, 1., -1.), None),       # every round splits off a few
        "below fp32": (torch.ones(Tk).double(), j * 2.0 ** -20),
        "equal": (torch.full((Tk,), -3.0).double(), None),
        "two values": ((j % 2), None),
        "few values": ((j % 7) - 3, None),                                   # more ties than a wavefront ranks
        "infinite": (torch.where(j % 9 == 0, float("inf"), torch.where(j % 9 == 1, -float("inf"), normal)), None),
    }
    B, N = len(rows), Tk * 64
    kmean, score = torch.zeros(B, 1, Tk, 128), torch.empty(B, Tk, dtype=torch.float64)
    for b, (x, y) in enumerate(rows.values()):
        kmean[b, 0, :, 0] = x.float()
        score[b] = x.float().double()
        if y is not None:
            kmean[b, 0, :, 1] = y.float()
            score[b] += y.float().double() * 2.0 ** -10
    q = torch.zeros(B, 2, 128, dtype=torch.float16)
    q[..., 0], q[..., 1] = 1.0, 2.0 ** -10
    k = torch.zeros(B, 1, N, 128, dtype=torch.float16, device="cuda")
    k4, ks = T.thrift_quantize_mxfp4(k, 0)
    v4, vs = T.thrift_quantize_mxfp4(k, 1)
    args = (q.cuda(), k, k, k4, ks, v4, vs, kmean.cuda())
    for lens in (None, [max(1, N - 64 * 3 * b - 17) for b in range(B)]):
        sl = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
        for fixed_k in sorted({1, 2, max(1, Tk // 20), max(1, Tk // 2), max(1, Tk - 1), Tk}):
            _, idx, cnt = T.thrift_attn_decode(*args, 64, 0.0, fixed_k=fixed_k, seqlens=sl, return_selection=True)
            for b in range(B):
                vis = Tk if lens is None else (lens[b] + 63) // 64
                n = min(fixed_k, vis)
                want = torch.sort(score[b, :vis], descending=True, stable=True).indices[:n].sort().values
                for h in range(2):
                    assert int(cnt[b, h]) == n
                    assert torch.equal(idx[b, h, :n].cpu().long(), want), (list(rows)[b], fixed_k, vis)
                    assert bool((idx[b, h, n:] == -1).all())


@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (2, 2)])
def test_a_key_of_nan_reaches_the_results_it_reaches_in_one_pass(T, Hq, Hkv):
    """Its row sums are NaN, in whichever chunk it lies, and what they divide is not a result of the other chunks alone."""
    print(f"decode split NaN Hq={Hq} Hkv={Hkv}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=2, N=4096, Hq=Hq, Hkv=Hkv)
    q, k, v = W.make_decode(wl, device="cuda")
    k[0, 1, 1000] = float("nan")
    k4, ks = T.thrift_quantize_mxfp4(k, 0)
    v4, vs = T.thrift_quantize_mxfp4(v, 1)
    args = (q, k, v, k4, ks, v4, vs, T.thrift_block_means(k, 64))
    need = T.decode_workspace_bytes(2, Hq, Hkv, 4096, wl.D, 64, 256)
    for budget in (0.0, 0.25, 1.0):
        two, one = (T.thrift_attn_decode(*args, 64, budget, out_dtype=torch.float32, return_selection=True,
                                         workspace=torch.zeros(n, dtype=torch.uint8, device="cuda"))[0] for n in (need, need - 256))
        assert torch.equal(torch.isnan(two), torch.isnan(one))
        assert float(torch.nan_to_num(two - one).norm() / torch.nan_to_num(one).norm()) <= REL


@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (2, 2), (16, 2)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_an_infinite_value_stays_with_the_heads_that_read_it(T, Hq, Hkv, bad):
    """A value that is not finite reaches the heads that have promoted its block and no other head of their KV group (a
    4-bit code is always finite), in the channel it has."""
    print(f"decode split V={bad} Hq={Hq} Hkv={Hkv}", flush=True)
    wl = W.scaled(W.DECODE_131K, B=1, N=4096, Hq=Hq, Hkv=Hkv)
    q, k, v = W.make_decode(wl, device="cuda")
    v[0, 1, 1000, 5] = bad
    k4, ks = T.thrift_quantize_mxfp4(k, 0)
    v4, vs = T.thrift_quantize_mxfp4(v, 1)
    args = (q, k, v, k4, ks, v4, vs, T.thrift_block_means(k, 64))
    for budget in (0.0, 0.25, 0.5, 1.0):
        out, idx, _ = T.thrift_attn_decode(*args, 64, budget, out_dtype=torch.float32, return_selection=True)
        reads = (idx[0] == 1000 // 64).any(-1) & (torch.arange(Hq, device="cuda") >= Hq // Hkv)
        want = torch.zeros_like(out, dtype=torch.bool)
        want[0, :, 5] = reads
        assert torch.equal(~torch.isfinite(out), want)


@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (24, 2)])
def test_partition_sizes_beyond_the_row(T, Hq, Hkv):
    """The largest int as partition size is one partition, in the two passes (8 / 2 heads) and in the walk (24 / 2)."""
    print(f"decode partition size beyond the row Hq={Hq} Hkv={Hkv}", flush=True)
    args = _cache(T, W.scaled(W.DECODE_131K, B=1, N=2048, Hq=Hq, Hkv=Hkv))
    want = T.thrift_attn_decode(*args, 64, 0.1, split_blocks=2048 // 64)
    for split in (2048 // 64 + 1, 2 ** 31 - 1):
        assert torch.equal(T.thrift_attn_decode(*args, 64, 0.1, split_blocks=split), want)


def test_a_card_without_room_for_two_passes_runs_one(T, monkeypatch):
    """No workspace given and no memory for the two-pass form's: the call runs the one-pass form."""
    print("decode without room for the larger workspace", flush=True)
    Hq, Hkv, N = 64, 8, 65536
    args = _cache(T, W.scaled(W.DECODE_131K, B=1, N=N, Hq=Hq, Hkv=Hkv))
    need, least = (f(1, Hq, Hkv, N, 128, 64, 256) for f in (T.decode_workspace_bytes, T.decode_least_workspace_bytes))
    assert need > (16 << 20) and least < (1 << 20)
    want = T.thrift_attn_decode(*args, 64, 0.05, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    two = T.thrift_attn_decode(*args, 64, 0.05, workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []                                                # what the allocator holds has no room for it either
    while not held or torch.cuda.memory_reserved() == before:
        before = torch.cuda.memory_reserved()
        held.append(torch.empty(need, dtype=torch.uint8, device="cuda"))
    total = torch.cuda.get_device_properties(0).total_memory
    got = []
    try:                                                     # the allocator's own limit: 8 MiB more than it holds
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (8 << 20)) / total)
        for call in (T._call, T._General):                   # the native entry and the general path
            monkeypatch.setattr(T, "_call", call)
            got.append(T.thrift_attn_decode(*args, 64, 0.05))
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert all(torch.equal(x, want) for x in got)
    assert torch.equal(T.thrift_attn_decode(*args, 64, 0.05), two)
