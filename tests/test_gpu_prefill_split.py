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
    (4, 64, 8, 1536, 64, True),          # the last grid that is interleaved (6144 workgroups)
    (4, 64, 8, 1537, 64, True),          # the first that is not
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
