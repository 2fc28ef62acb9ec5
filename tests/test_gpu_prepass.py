"""The one-launch pre-pass against the single calls it stands for (which are checked against the oracle): the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,N,Bq,dtype", [
    (1, 1, 1, 1, 64, torch.float16), (1, 2, 1, 63, 128, torch.bfloat16), (2, 3, 3, 65, 64, torch.float16),
    (1, 4, 2, 129, 128, torch.bfloat16), (2, 2, 1, 1000, 128, torch.float16), (1, 8, 2, 2048, 64, torch.bfloat16),
])
def test_prepass_equals_the_single_calls(B, Hq, Hkv, N, Bq, dtype):
    from paper_2605_23081_amd import binding as T
    print(f"prepass B={B} Hq={Hq} Hkv={Hkv} N={N} Bq={Bq} {dtype}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    mk = lambda H: torch.randn(B, H, N, 128, generator=g, device="cuda") * torch.exp2(torch.randint(-20, 5, (B, H, N, 1), generator=g, device="cuda").float())
    q, k, v = mk(Hq).to(dtype), mk(Hkv).to(dtype), mk(Hkv).to(dtype)
    k[0, 0, 0] = 0.0                                         # an all-zero group
    if dtype == torch.bfloat16:
        q[0, 0, 0, :32] = 2.0 ** -130                        # groups below the converter's range
    qm, km = T.thrift_block_means(q, Bq), T.thrift_block_means(k, 64)
    want = [qm, km, *T.thrift_quantize_mxfp4(q, 0), *T.thrift_quantize_mxfp4(k, 0), *T.thrift_quantize_mxfp4(v, 1)]
    got = [torch.full_like(t, 77) for t in want]
    T.thrift_prefill_prepass(q, k, v, Bq, 64, *got)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("rows,Tk", [(1, 1), (5, 64), (17, 65), (16, 128), (33, 129), (15, 300)])
def test_selection_chunks_and_row_counts(rows, Tk):
    """64-key chunks left out at the end of a row, ragged last workgroups; few rows, hence 4 per workgroup."""
    import numpy as np
    from oracle import thrift_oracle as oracle
    from paper_2605_23081_amd import binding as T
    from tests.gpu_util import check_selection, to_np
    print(f"select rows={rows} Tk={Tk}", flush=True)
    rng = np.random.default_rng(rows * 1000 + Tk)
    qm = rng.standard_normal((1, 2, rows, 128), dtype=np.float32)
    km = rng.standard_normal((1, 1, Tk, 128), dtype=np.float32)
    for causal in (False, True):
        if causal and rows > Tk:
            continue
        idx_o, cnt_o = oracle.select_topk(qm, km, 64, 64, causal, 0.3)
        idx, cnt = T.thrift_select_topk(torch.from_numpy(qm).cuda(), torch.from_numpy(km).cuda(), 64, 64, causal, 0.3)
        assert check_selection(to_np(idx), to_np(cnt), idx_o, cnt_o, oracle.block_scores(qm, km)) == 0


@pytest.mark.parametrize("B,Hq,Hkv,Tq,Tk,causal,off,shared", [
    (16, 8, 8, 17, 65, False, 0, False),               # 256 workgroups of 16 rows, the fewest; the last of a unit has one row
    (16, 8, 8, 16, 65, False, 0, False),               # 128 would be too few: 4 rows each
    (32, 8, 8, 5, 300, False, 0, False),               # one ragged workgroup of 16 rows per unit
    (32, 8, 8, 4, 300, False, 0, False),               # four rows are one workgroup of 4
    (32, 16, 8, 9, 300, True, 291 * 64, False),        # 18 rows in the order (query block, head), a causal frontier
    (32, 16, 8, 18, 600, True, 582 * 64, True),        # 16 chunks per lane, one set per KV head
    (16, 16, 8, 9, 2048, True, 2039 * 64, False),      # 32 chunks
    (16, 8, 8, 18, 2048, False, 0, False),
    (16, 8, 8, 18, 2049, False, 0, False),             # one key block more than 16 rows' registers hold
])
def test_selection_rows_per_workgroup(B, Hq, Hkv, Tq, Tk, causal, off, shared):
    """The selection kernel on both sides of the rule for its rows per workgroup."""
    from oracle import thrift_oracle as oracle
    from paper_2605_23081_amd import binding as T
    print(f"select B={B} Hq={Hq} Hkv={Hkv} Tq={Tq} Tk={Tk} causal={causal} off={off} shared={shared}", flush=True)
    g = torch.Generator().manual_seed(100 * Tq + Tk)
    qm, km = torch.randn(B, Hq, Tq, 128, generator=g), torch.randn(B, Hkv, Tk, 128, generator=g)
    idx_o, cnt_o = oracle.select_topk(qm.numpy(), km.numpy(), 64, 64, causal, 0.05, q_block_offset=off, group_shared=shared)
    idx, cnt = T.thrift_select_topk(qm.cuda(), km.cuda(), 64, 64, causal, 0.05, q_block_offset=off, group_shared=shared)
    assert torch.equal(cnt.cpu(), torch.from_numpy(cnt_o))
    assert torch.equal(idx.cpu()[..., :idx_o.shape[-1]], torch.from_numpy(idx_o)) and bool((idx[..., idx_o.shape[-1]:] == -1).all())


def test_plan_prepass_takes_each_tensor_in_its_own_type():
    """The pre-pass of a plan alone, with K in another 16-bit type than Q and V."""
    from paper_2605_23081_amd import binding as T
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    mk = lambda H, dt: torch.randn(1, H, 300, 128, generator=g, device="cuda").to(dt)
    q, k, v = mk(4, torch.float16), mk(2, torch.bfloat16), mk(2, torch.float16)
    plan = T.PrefillPlan(1, 4, 2, 300, 128, 128, 64, True, 0.3, torch.float16, "cuda")
    plan.run(q, k, v, attention=False)
    qm, km = T.thrift_block_means(q, 128), T.thrift_block_means(k, 64)
    want = [qm, km, *T.thrift_quantize_mxfp4(q, 0), *T.thrift_quantize_mxfp4(k, 0), *T.thrift_quantize_mxfp4(v, 1),
            *T.thrift_select_topk(qm, km, 128, 64, True, 0.3)]
    for a, b in zip((plan.qmean, plan.kmean, plan.q4, plan.qs, plan.k4, plan.ks, plan.v4, plan.vs, plan.idx, plan.cnt), want):
        assert torch.equal(a, b)
    with pytest.raises(AssertionError):
        plan.run(q, k, v)                                    # the attention itself takes one type
