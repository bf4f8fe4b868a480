"""Host tensors are refused by the transfers before any launch: their
pointers must not reach a kernel."""

import pytest
import torch

from paper_1711_11296_amd import transfer

G = torch.zeros(1, 5, 8)
S = torch.zeros(1, 6, 2)


@pytest.mark.parametrize("call", [
    lambda: transfer.spec_retruncate(S, 2, 1),
    lambda: transfer.grid_inject(G, 3, 4),
    lambda: transfer.grid_product(G, G),
    lambda: transfer.spec_laplacian(S, 2),
    lambda: transfer.grid_residual(G, G[0], G, G, 1.0),
], ids=["spec_retruncate", "grid_inject", "grid_product", "spec_laplacian", "grid_residual"])
def test_host_tensor_is_refused(call):
    with pytest.raises(ValueError, match="device"):
        call()
