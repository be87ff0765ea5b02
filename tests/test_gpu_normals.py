"""GPU: the error of the synthetic gradients against 64-bit arithmetic, from the words of the oracle's generator."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def philox(q, k, seed):
    """Philox4x32-10 of the counters (q, k) of the gradient stream, vectorised."""
    mask = np.uint64(0xFFFFFFFF)
    c = [q & mask, q >> np.uint64(32), np.full_like(q, k & 0xFFFFFFFF), np.full_like(q, (k >> 32 & 0xFFFFFF) | 2 << 24)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & mask, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def normals(n, k, seed):
    w = philox(np.arange(n // 4, dtype=np.uint64), k, seed)
    out = np.empty((n // 4, 4))
    for i in range(2):
        r = np.sqrt(-2.0 * np.log(((w[2 * i] >> np.uint64(9)) + 0.5) * 2.0 ** -23))
        quarters = 4.0 * ((w[2 * i + 1] >> np.uint64(8)) * 2.0 ** -24)
        turn = np.rint(quarters)
        f = (quarters - turn) * (np.pi / 2)
        c, s, turn = np.cos(f), np.sin(f), turn.astype(np.int64) % 4
        out[:, 2 * i] = r * np.choose(turn, [c, -s, -c, s])
        out[:, 2 * i + 1] = r * np.choose(turn, [s, c, -s, -c])
    return out.reshape(-1)


# A rounding costs 2.8e-8 rms of a value.  A variate is a radius times a sine or cosine, each rounded once, and the product: three,
# 4.8e-8.  Where the radius takes the standard deviation with a rounding of its own there are four, 5.6e-8, of which the
# hardware's root has less than a whole one.  A power of two costs no rounding.
@pytest.mark.parametrize("std,bound", [(1.0, 4.9e-8), (0.5, 4.9e-8), (-4.0, 4.9e-8), (2.0 ** -40, 4.9e-8), (0.0316227766016838, 5.4e-8), (0.3, 5.4e-8), (1.5, 5.4e-8)])
def test_error_of_the_synthetic_gradients(std, bound):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_06952_amd as P
    print("normals, std %g" % std, flush=True)
    std, n = float(np.float32(std)), 4 << 20
    g = torch.empty(n, dtype=torch.float32, device="cuda:0")
    P.adpsgd_synth_gradient(11, 5, std, n, g.data_ptr(), torch.cuda.current_stream().cuda_stream)
    ref = normals(n, 5, 11) * std
    assert np.allclose(ref[:1000], oracle.synth_grad(11, 5, std, np.arange(1000)), rtol=1e-6, atol=0.0)       # the same generator
    inside = ref != 0.0
    err = (g.cpu().numpy().astype(np.float64)[inside] - ref[inside]) / ref[inside]
    assert np.sqrt(np.mean(err ** 2)) <= bound
    assert np.abs(err).max() <= 3e-7
