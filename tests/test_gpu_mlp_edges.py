"""The surrogate's training at the edges of its tiles and chunks: batches that
end anywhere in a block of 16 or 32 rows or in a chunk of 256, small batches
after large ones on the same network, vectors at any 4-byte address, and the
fused training step against its two halves, bit for bit."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from oracle import mlp as ref
from paper_2108_02419_amd import _bbe, inputs
from test_gpu_mlp import _bits, _features

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def test_gradients_of_any_batch_size(torch):
    rng = np.random.default_rng(21)
    params = inputs.surrogate_random(6)
    net = _bbe.Mlp(params, max_batch=600)
    buf = torch.empty(_bbe.MLP_NPARAMS + 1, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    # bfloat16 roundings that differ from the reference's: 2^-9 of an element,
    # the whole of it in a batch of one; a row missing or counted twice is 1/B
    for B in (600, 1, 15, 16, 17, 31, 32, 33, 255, 256, 257, 513, 2):
        announce(f"mlp gradients B={B}")
        X, n, T = _features(rng, B)
        grad = buf[B % 2:][:_bbe.MLP_NPARAMS]
        grad.fill_(7.0)
        net.loss_grad(_bits(torch, X), torch.tensor(n, device="cuda"),
                      torch.tensor(T, device="cuda"), loss, grad)
        torch.cuda.synchronize()
        l_ref, g_ref = ref.loss_and_grad(params.astype(np.float64), X, n, T)
        assert abs(float(loss.item()) - l_ref) <= 1e-3 * max(1.0, abs(l_ref))
        G = ref.unpack(grad.cpu().numpy().astype(np.float64))
        R = ref.unpack(g_ref)
        for name in G:
            scale = max(np.linalg.norm(R[name]), 1e-30)
            err = np.linalg.norm(G[name] - R[name]) / scale
            assert err <= 4e-3, (B, name, err)


@pytest.mark.parametrize("B", [7, 256, 300, 1024])
def test_train_step_is_its_two_halves(torch, B):
    rng = np.random.default_rng(B)
    params = inputs.surrogate_init(3)
    one, two = _bbe.Mlp(params, max_batch=1024), _bbe.Mlp(params, max_batch=1024)
    la, lb = (torch.empty(1, dtype=torch.float32, device="cuda") for _ in range(2))
    for _ in range(3):
        X, n, T = _features(rng, B)
        args = _bits(torch, X), torch.tensor(n, device="cuda"), torch.tensor(T, device="cuda")
        announce(f"mlp train step B={B}")
        one.train_step(*args, 1e-3, la)
        two.loss_grad(*args, lb)
        two.adam_step(1e-3)
        torch.cuda.synchronize()
        assert la.item() == lb.item()
    np.testing.assert_array_equal(one.params(), two.params())
