"""Weight gradients of large batches: a row's part is not lost in a sum over many others.

With all weights zero every row has the same last activations c (a bfloat16 number), so
the last layer's gradient is c times the sum of the output gradients over the batch.  In
each eighth of it the first 512 rows have 1 and the rest 2^-21 of it (over B, a power of
two): 16 rows of the latter, what one product adds, are less than half a unit in the last
place of the former, 512 rows of them four units.  Sums of 512 rows and then of those round
at most once for each of B / 4096 + 8 additions, 2^-24 relative each; a running sum over an
eighth of the batch loses every small row."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [4096, 65536, 262144])
def test_small_rows_count(B):
    from paper_1707_05163_amd import Surrogate
    net = Surrogate(0)
    layers = [(np.zeros_like(W), np.zeros_like(b)) for W, b in net.get_params()]
    layers[3][1][:] = 1.5
    net.set_params(layers)
    d = np.full((8, B // 8), 2.0 ** -21)
    d[:, :512] = 1.0
    T = np.zeros((B, 2), np.float32)
    T[:, 0] = -d.ravel()
    grads, _ = net.gradients(np.zeros((B, 64), np.float32), T)
    c = 179.0 / 128.0  # GELU(1.5) = 1.3996 to 8 bits
    want = c * d.sum() / B
    rel = np.abs(grads[4][0][:, 0].astype(np.float64) / want - 1.0).max()
    print(f"B {B}: relative error {rel:.2e}", flush=True)
    assert rel <= (B / 4096 + 8) * 2.0 ** -24
    bias = abs(float(grads[4][1][0]) * B / d.sum() - 1.0)
    assert bias <= (B / 512 + 8) * 2.0 ** -24
    for k in range(4):  # zero weights pass no gradient down
        assert not grads[k][0].any() and not grads[k][1].any()
