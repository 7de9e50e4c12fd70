"""GPU parity of the SF rebuild with the split pipelined (64 x 64 tiles of at
most one per CU from K = 128, two from K = 640): the same products in the same order as the plain
split, so the same bits, at the edges of its tiles and K slices."""
import pytest
import torch

import oracle
from _helpers import W_TOL, assert_close, dev, kernels, log, sample_points, to_np
from paper_1706_03292_amd import api
from paper_1706_03292_amd import inputs as I

pytestmark = pytest.mark.gpu


# An odd and an even number of 32-row slices, whole and partial; M and N of one
# column, one tile, one past, one short, one tile per CU, and two, which take the
# plain split below K = 640.  The whole layer (1024 tiles) takes the plain split.
@pytest.mark.parametrize("K", [128, 129, 160, 191, 250, 639, 640, 673])
@pytest.mark.parametrize("momentum", [False, True])
def test_piped_split_equals_the_plain_one(K, momentum):
    d = dev()
    M, N = 2048, 2048
    W, U, V = I.randn(K, (M, N), 0.01), I.randn(K + 1, (K, M), 0.1), I.randn(K + 2, (K, N), 0.1)
    buf = I.randn(K + 3, (M, N), 1e-3)
    cus = torch.cuda.get_device_properties(d).multi_processor_count

    def apply(w, b, u, v):
        w, b, u, v = (t.contiguous().to(d) for t in (w, b, u, v))
        if momentum:
            api.sf_apply_momentum(w, b, u, v, 0.01, 0.9)
        else:
            api.sf_apply(w, u, v, 0.01)
        torch.cuda.synchronize()
        return w.cpu(), b.cpu()

    def ran(*args):
        got = []
        names = [k for k in kernels(lambda: got.extend(apply(*args))) if k.startswith("sf_")]
        assert len(names) == 1 and names[0].startswith("sf_apply_kernel<64, 64, ")
        return got, names[0].endswith(", true>")

    (whole_w, whole_b), piped = ran(W, buf, U, V)
    assert not piped
    for m, n in [(1, 1), (64, 64), (65, 127), (1000, 700), (1024, 1024), (1000, 1025), (1024, 2048), (2048, 1023)]:
        log(f"piped split {m}x{n} K={K} momentum={momentum}")
        (w, b), piped = ran(W[:m, :n], buf[:m, :n], U[:, :m], V[:, :n])
        assert piped == (K >= 640 or -(-m // 64) * -(-n // 64) <= cus)
        assert torch.equal(w, whole_w[:m, :n]) and torch.equal(b, whole_b[:m, :n])
    if not momentum:
        rows, cols = sample_points(1000, 700, 2000, seed=K)
        ref = oracle.sf_apply_points(W[:1000, :700].contiguous().numpy(), U[:, :1000].contiguous().numpy(),
                                     V[:, :700].contiguous().numpy(), 0.01, rows, cols)
        w, _ = apply(W[:1000, :700], buf[:1000, :700], U[:, :1000], V[:, :700])
        assert_close(to_np(w)[rows, cols], ref, W_TOL, "W")
