"""Buffers for which one launch of an elementwise kernel would pass the 2^32 threads that a dispatch
holds (the runtime cuts such a grid to 32 bits without an error, and the rest of the buffer was left
as it lay): every entry is written, on values known in advance."""
import pytest
import torch

import paper_2605_12070_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch.cuda.empty_cache()


def _say(*a):
    print("[case]", *a, flush=True)


@pytest.mark.parametrize("dtype,n,off", [(torch.float32, (1 << 34) + 4099, 0), (torch.bfloat16, (1 << 32) + 77, 1)])
@pytest.mark.parametrize("device", [False, True])
def test_ewma_update(dtype, n, off, device):
    """16-byte vectors (64 GB of them), and one entry per thread where the buffer is not aligned."""
    _say("ewma", dtype, n, off, device)
    x = torch.zeros(n + off, dtype=dtype, device=DEV)[off:]
    new = torch.empty(n + off, dtype=dtype, device=DEV)[off:]
    new.fill_(2.0)
    if device:
        proxy = P.EwmaProxyDevice(x[:16], beta=0.5, normalized=False)
        proxy.x = x                              # the wrapper's own copy of 64 GB is not needed
        proxy.step(new, torch.tensor([4, 4, 4, 4, 0], dtype=torch.int32, device=DEV))
    else:
        P.ewma_proxy_update(x, new, beta=0.5, normalized=False)
    low, high = torch.aminmax(x)
    assert low.item() == 1.0 and high.item() == 1.0


def test_shard_statistics():
    """One workgroup per row."""
    T, Vs = (1 << 24) + 5, 8
    _say("shard stats", T, Vs)
    z = torch.zeros(T, Vs, dtype=torch.bfloat16, device=DEV)
    ids = torch.zeros(T, dtype=torch.int64, device=DEV)
    for _ in range(2):                           # the second call's outputs reuse poisoned memory
        lse, zy = P.vocab_shard_stats(z, ids, 0, Vs)
        assert torch.all((lse - 2.0794415).abs() <= 2e-6) and torch.all(zy == 0)
        lse.fill_(-7.0)
        zy.fill_(-7.0)
        del lse, zy


def test_shard_gradient():
    """Two workgroups of 512 threads per row, in place."""
    T, Vs = 4194307, 4104
    _say("shard gradient", T, Vs)
    z = torch.zeros(T, Vs, dtype=torch.bfloat16, device=DEV)
    ids = torch.zeros(T, dtype=torch.int64, device=DEV)
    lse = torch.full((T,), float(torch.tensor(4104.0, dtype=torch.float64).log()), device=DEV)
    lp = -lse
    one = torch.ones(T, device=DEV)
    P.decoupled_ppo_loss_shard_fwd_bwd(z, 0, Vs, lse, torch.zeros(T, device=DEV), ids, lp, lp, one,
                                       dlogits=z, scale_mode="const")
    p = torch.tensor(1 / 4104).to(torch.bfloat16).item()
    low, high = torch.aminmax(z[:, 1:])
    assert low.item() == p and high.item() == p
    assert torch.all(z[:, 0] == torch.tensor(1 / 4104 - 1).to(torch.bfloat16).item())


def test_lm_head_gradient():
    """The one-pass LM head whose T V exponentials pass 2^35 (69 GB): dhidden of the last tokens is
    that of a call on them alone."""
    T, d, V = (1 << 18) + 64, 8, 131072 + 256
    _say("lm head", T, d, V)
    g = torch.Generator(device=DEV).manual_seed(3)
    h = torch.randn(T, d, generator=g, device=DEV).to(torch.bfloat16)
    w = torch.randn(V, d, generator=g, device=DEV).to(torch.bfloat16)
    ids = torch.randint(0, V, (T,), generator=g, device=DEV)
    lp = torch.full((T,), -13.0, device=DEV)
    adv = torch.randn(T, generator=g, device=DEV)
    kw = dict(scale_mode="const", clip_eps=(0.5, 1e9), band=(0.0, float("inf")))
    all_ = P.fused_lm_head_loss_fwd_bwd(h, w, ids, lp, lp, adv, **kw)
    tail = slice(T - 4096, T)
    part = P.fused_lm_head_loss_fwd_bwd(h[tail], w, ids[tail], lp[tail], lp[tail], adv[tail], **kw)
    # the same bf16 G and weights, summed in fp32 in another order
    scale = part.dhidden.abs().max()
    assert scale > 0 and (all_.dhidden[tail] - part.dhidden).abs().max() <= 1e-3 * scale
