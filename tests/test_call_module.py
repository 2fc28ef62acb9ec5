"""The native entry of the serving calls: what it does not serve goes to the general path, which names the fault."""
import pytest
import torch

from paper_2605_23081_amd import binding as T


def _args(device):
    B, Hq, Hkv, N, D = 1, 4, 2, 128, 128
    z = lambda *s, dt=torch.uint8: torch.zeros(*s, dtype=dt, device=device)
    h = torch.float16
    return [z(B, Hq, D, dt=h), z(B, Hkv, N, D, dt=h), z(B, Hkv, N, D, dt=h), z(B, Hkv, N, D // 2), z(B, Hkv, N, D // 32),
            z(B, Hkv, N // 64, D, 32), z(B, Hkv, N // 32, D), z(B, Hkv, N // 64, D, dt=torch.float32)]


def test_other_devices_and_kinds_of_arguments_are_left_to_the_general_path():
    m = T._native()
    a = _args("cpu")
    rest = (64, 0.05, -1, 256, 0.0, None, None, None, 0, 0)
    assert m.decode(*a, *rest) is None                       # host tensors
    assert m.decode(*[None] * 8, *rest) is None and m.decode() is None
    assert m.append(*a[:2], None, None, *a[1:], 64, 0) is None and m.attention(*a[:3], 1, 128, 64, 0.05, -1, 0.0, None, None, None, 0, 0) is None
    with pytest.raises(AssertionError):
        T.thrift_attn_decode(*a, 64, 0.05)


def test_tensors_without_storage_are_left_to_the_general_path():
    """Under a transform a tensor has sizes but no data pointer; refusing it must not end the process."""
    from torch._subclasses.fake_tensor import FakeTensorMode
    m = T._native()
    with FakeTensorMode():
        a = _args("cuda")                                    # device tensors in a process without a device
        lens = torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    seen = []

    def served(q, k):
        seen.append(m.decode(q, *a[1:], 64, 0.05, -1, 256, 0.0, lens, a[0], ws, 0, 0))
        seen.append(m.append(k, a[1], lens, None, *a[1:], 64, 0))
        seen.append(m.attention(k, a[1], a[1], 1, 128, 64, 0.05, -1, 0.0, ws, a[1], None, 0, 0))
        return q

    torch.vmap(served)(a[0].unsqueeze(0), a[1].unsqueeze(0))
    assert seen == [None] * 3


def _without_module(monkeypatch):
    """binding as it is where the module cannot be loaded."""
    import sys
    import paper_2605_23081_amd as package
    monkeypatch.setattr(T, "_call", None)
    monkeypatch.delattr(package, "_call", raising=False)
    monkeypatch.setitem(sys.modules, package.__name__ + "._call", None)      # what an import that fails finds
    with pytest.warns(RuntimeWarning, match="_call"):
        return T._native()


def test_a_module_that_cannot_be_loaded_leaves_the_calls_to_the_general_path(monkeypatch):
    m = _without_module(monkeypatch)
    assert m.decode() is None and m.append() is None and m.attention() is None and T._native() is m
    with pytest.raises(AssertionError):
        T.thrift_attn_decode(*_args("cpu"), 64, 0.05)


@pytest.mark.gpu
def test_the_general_path_gives_the_same_results(monkeypatch):
    g = torch.Generator().manual_seed(1)
    q, k, v = (torch.randn(1, H, 200, 128, generator=g).half().cuda() for H in (4, 2, 2))

    def results():
        cache = T.KVCache(1, 2, 256, 128, 64, torch.float16, "cuda", fill=0)
        cache.append(k, v)
        cache.append(k[:, :, :1].contiguous(), v[:, :, :1].contiguous())
        c = (cache.k16, cache.v16, cache.k4, cache.ks, cache.v4, cache.vs, cache.kmean)
        return [T.thrift_attn_decode(q[:, :, 7].contiguous(), *c, 64, 0.5, seqlens=cache.seqlens), T.thrift_attention(q, k, v, budget=0.3),
                cache.seqlens, *c]

    want = results()
    _without_module(monkeypatch)
    for a, b in zip(results(), want):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_device_tensors_of_wrong_shape_or_type_raise_as_before():
    a = _args("cuda")
    assert torch.equal(T.thrift_attn_decode(*a, 64, 0.05), torch.zeros(1, 4, 128, dtype=torch.float16, device="cuda"))
    for i, bad in ((0, a[0].float()), (3, a[3][:, :, :64].contiguous()), (7, a[7].half()), (1, a[1].transpose(1, 2))):
        b = list(a)
        b[i] = bad
        with pytest.raises(AssertionError):
            T.thrift_attn_decode(*b, 64, 0.05)
    with pytest.raises(T.ThriftError):
        T.thrift_attn_decode(*a, 64, 1.5)                    # a status of the C call
    with pytest.raises(AssertionError):
        T.thrift_attn_decode(*a, 64, 0.05, seqlens=torch.zeros(2, dtype=torch.int32, device="cuda"))
    cache = T.KVCache(1, 2, 128, 128, 64, torch.float16, "cuda", fill=0)
    new = torch.zeros(1, 2, 100, 128, dtype=torch.float16, device="cuda")
    before = cache.seqlens
    cache.append(new, new)
    cache.append(new, new, torch.tensor([20], dtype=torch.int32, device="cuda"))
    assert before.tolist() == [0] and cache.seqlens.tolist() == [120]
    cache.append(new, new)
    assert cache.seqlens.tolist() == [128]                   # the capacity
    with pytest.raises(AssertionError):
        cache.append(new.float(), new.float())


@pytest.mark.gpu
@pytest.mark.parametrize("count", [64, 41, 33])
def test_the_mean_of_an_appended_block_adds_its_tokens_in_order(oracle, count):
    """Keys that lie further apart than a double reaches: the sum depends on its order, which is that of the tokens."""
    print(f"append mean count={count}", flush=True)
    g = torch.Generator().manual_seed(count)
    k = torch.randn(1, 2, count, 128, generator=g)
    k[:, 0, 0], k[:, 0, 40 if count > 40 else 20] = 2.0 ** 100, -2.0 ** 100
    k = k.to(torch.bfloat16)
    cache = T.KVCache(1, 2, 64, 128, 64, torch.bfloat16, "cuda", fill=0)
    kg = k.cuda()
    cache.append(kg[:, :, :7].contiguous(), kg[:, :, :7].contiguous())
    cache.append(kg[:, :, 7:].contiguous(), kg[:, :, 7:].contiguous())
    bits, dt = oracle.bits_of(k)
    assert torch.equal(cache.kmean.cpu(), torch.from_numpy(oracle.block_means(bits, dt, 64)))


@pytest.mark.gpu
def test_group_shared_is_taken_for_its_truth_value():
    a = _args("cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    for i in (0, 2):                                                         # V in 16 bits alone: which block is promoted shows
        a[i].copy_(torch.randn(a[i].shape, generator=g, device="cuda"))
    a[7].copy_(a[0].float().view(a[7].shape))                                # head i of a group prefers block i
    own, shared = (T.thrift_attn_decode(*a, 64, 0.5, group_shared=x) for x in (False, True))
    assert not torch.equal(own, shared)
    for x, want in ((None, own), (0, own), ("", own), (0.5, shared), (2 ** 40, shared), ([0], shared)):
        assert torch.equal(T.thrift_attn_decode(*a, 64, 0.5, group_shared=x), want)
