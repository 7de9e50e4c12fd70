"""PS applies for worker counts that are no compile-time value of the kernels:
the shards behind the last chunk of eight go four, two and one at a time, and a
thread's two groups together."""
import pytest
import torch

from _helpers import dev, kernels, log
from paper_1706_03292_amd import api
from paper_1706_03292_amd import inputs as I

pytestmark = pytest.mark.gpu

# Nothing behind the chunk, every remainder, one chunk and three.
WORKERS = [3, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 17, 24, 25, 31, 33]


@pytest.mark.parametrize("P", WORKERS)
def test_ps_runtime_worker_count_is_the_sum_in_order(P):
    """Bitwise the shards added one after another in fp32, then one fused
    multiply-add per update (formed in 64 bits and rounded once, which equals
    the fused one unless the 64-bit sum itself is rounded to a tie, at most one
    unit of fp32's last place): sizes at the ends of a thread's two groups and
    of a workgroup's block, aligned and not, alone and batched."""
    d = dev()
    lr, mu = 0.01, 0.9
    for n in (1, 3, 255, 1024, 1028, 2047, 2048, 2052, 20480 + 1026):
        for off in (0, 1):
            for mom in (False, True):
                log(f"ps run-time P={P} n={n} offset={off} momentum={mom}")
                flat = I.randn(31 * P + n, (n + off,), 0.01).to(d)
                G = I.randn(37 * P + n, (P * n + off,), 0.001).to(d)[off:].view(P, n)
                W, b = flat.clone()[off:], I.randn(41 * P + n, (n + off,), 0.001).to(d)[off:]
                s = G[0].clone()
                for p in range(1, P):
                    s += G[p]
                f32 = lambda x: float(torch.tensor(x, dtype=torch.float32))   # noqa: E731
                want_b = (b.double() * f32(mu) + s.double()).float() if mom else s
                want_W = (W.double() - f32(lr) * want_b.double()).float()
                W2, b2 = flat.clone()[off:], b.clone()
                api.ps_apply(W, G, lr, mu if mom else 0.0, b if mom else None)
                api.ps_apply_batch([(W2, G, b2 if mom else None)], lr, mu if mom else 0.0)
                torch.cuda.synchronize()
                eps = 2.0 ** -23
                assert torch.equal(W, W2) and (not mom or torch.equal(b, b2))
                if mom:
                    assert bool(((b - want_b).abs() <= eps * want_b.abs()).all())
                    # (a unit of buf moves W by lr of it, and W by one of its own)
                    assert bool(((W - want_W).abs() <= eps * (want_W.abs() + lr * want_b.abs())).all())
                else:
                    assert bool(((W - want_W).abs() <= eps * want_W.abs()).all())


@pytest.mark.parametrize("P", [3, 7, 9, 13, 15, 17])
@pytest.mark.parametrize("n", [1 << 19, (1 << 19) + 4, (1 << 19) + 5, (1 << 21), (1 << 21) + 4, (1 << 21) + 2049])
@pytest.mark.parametrize("mom", [False, True])
def test_ps_runtime_worker_count_large(P, n, mom):
    """On both sides of one workgroup (2048 values) per CU, from which on aligned
    tensors load four shards at a time instead of eight, and of the size from
    which some worker counts keep one shard after another and the others four
    with a momentum buffer only: the batched pass gives the same bits, and the
    raw sum (W = 0, lr = -1, no momentum) is the shards' in order."""
    d = dev()
    cus = torch.cuda.get_device_properties(d).multi_processor_count
    many = n > 1 << 21
    at_once = 4 if n % 4 == 0 and P > 8 and -(-n // 2048) > cus and (mom or not many) else 8
    if many and (P < 8 or 12 < P < 16):
        at_once = 0
    log(f"ps run-time P={P} n={n} momentum={mom}")
    g = torch.Generator("cuda").manual_seed(P + n)
    G = torch.randn(P, n, generator=g, device=d)
    W, W2, b, b2 = (torch.zeros(n, device=d) for _ in range(4))
    s = G[0].clone()
    for p in range(1, P):
        s += G[p]
    mu = 0.9 if mom else 0.0
    assert kernels(lambda: api.ps_apply(W, G, -1.0, mu, b if mom else None)) == [
        f"ps_apply_kernel<0, {'true' if mom else 'false'}, {'true' if n % 4 == 0 else 'false'}, {at_once}>"]
    api.ps_apply_batch([(W2, G, b2 if mom else None)], -1.0, mu)
    torch.cuda.synchronize()
    assert torch.equal(W, s) and torch.equal(W2, s)
    if mom:
        assert torch.equal(b, s) and torch.equal(b2, s)
