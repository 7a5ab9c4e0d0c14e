"""kmp_dgemm_grouped in each of its forms (a wavefront per 16 x 16 block, 32 x
64 and 64 x 64 tiles; paired loads for even K on aligned rows, single ones
otherwise) against numpy, at remainders of every tile dimension. Bound: a sum
of K products in any order is within K eps sum |a| |b| of the exact one, on
both sides."""
import numpy as np
import pytest

from tests.gpu_common import announce, device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,M,N,K", [
    (1, 1, 1, 1), (2, 3, 5, 2), (1, 17, 16, 15), (3, 33, 31, 16), (2, 100, 7, 17), (1, 64, 65, 63),
    (4, 130, 33, 82),                                  # 16 x 16 blocks
    (9, 513, 100, 33), (9, 520, 97, 64), (40, 97, 129, 31),      # 32 x 64 tiles
    (9, 1025, 130, 33), (70, 130, 127, 18), (5, 1000, 300, 16)])  # 64 x 64 tiles
def test_grouped_product(G, M, N, K):
    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    announce(f"kmp_dgemm_grouped G={G} M={M} N={N} K={K}")
    rng = np.random.default_rng(G + M + N + K)
    A, B = rng.standard_normal((G, M, K)), rng.standard_normal((G, K, N))
    out = torch.full((G, M, N), np.nan, dtype=torch.float64, device=dev)
    km.kmp_dgemm_grouped(torch.as_tensor(A, device=dev), torch.as_tensor(B, device=dev), out)
    bound = 2.0 * (K + 1) * 2.0 ** -52 * np.matmul(np.abs(A), np.abs(B))
    assert np.all(np.abs(out.cpu().numpy() - np.matmul(A, B)) <= bound)
    # an odd offset: no pairs, the same sums
    buf = torch.empty(G * M * K + 1, dtype=torch.float64, device=dev)
    buf[1:] = torch.as_tensor(A.ravel(), device=dev)
    again = torch.full_like(out, np.nan)
    km.kmp_dgemm_grouped(buf[1:].view(G, M, K), torch.as_tensor(B, device=dev), again)
    assert torch.equal(out, again)


def test_grouped_product_keeps_infinities_to_their_rows():
    """Rows and columns past the end repeat valid ones and are not stored:
    non-finite entries stay in their own row and column."""
    import torch
    from paper_2606_06742_amd import kmpath as km
    dev = device()
    announce("kmp_dgemm_grouped with an infinite last row and column")
    A = torch.ones(1, 37, 19, dtype=torch.float64, device=dev)
    B = torch.ones(1, 19, 21, dtype=torch.float64, device=dev)
    A[0, 36, 18] = float("inf")
    B[0, 18, 20] = float("nan")
    out = torch.empty(1, 37, 21, dtype=torch.float64, device=dev)
    km.kmp_dgemm_grouped(A, B, out)
    assert bool((out[0, :36, :20] == 19.0).all()) and bool(out[0, 36, :20].isinf().all())
    assert bool(out[0, :, 20].isnan().all())
