"""What the native binding accepts and returns, as the Python functions did: a Q with fewer dimensions, which the descriptor
lays out."""
import pytest
import torch

from paper_2105_13120_amd import rsa

pytestmark = pytest.mark.gpu


def rand(*shape):
    return torch.randn(*shape, device="cuda").bfloat16()


@pytest.mark.parametrize("dims", [1, 2, 3])
def test_q_with_fewer_dimensions(dims):
    torch.manual_seed(0)
    Q, K, V = (rand(1, 2, 256, 64) for _ in range(3))
    d = rsa.make_desc(K, 4)
    O, LSE = rsa.forward(d, Q, K, V)
    q = Q.reshape({1: (-1,), 2: (-1, 64), 3: (2, 256, 64)}[dims])
    O2, LSE2 = rsa.forward(d, q, K, V)
    assert O2.shape == q.shape and LSE2.shape == q.shape[:3]     # (a larger LSE than is written)
    assert torch.equal(O2.reshape(O.shape), O) and torch.equal(LSE2.flatten()[:512], LSE.flatten())
    K2 = rand(1, 2, 128, 64)
    O, LSE = rsa.linformer_forward(d, Q, K2, K2)
    O2, LSE2 = rsa.linformer_forward(d, q, K2, K2)
    assert torch.equal(O2.reshape(O.shape), O) and torch.equal(LSE2.flatten()[:512], LSE.flatten())
