"""The router projection of many tokens in tiles of 32 tokens x 32 (16) experts: remainders of either, uneven shares of the hidden
dimension, one slice and two, one round of workgroups and two, and shapes that padding or an uneven last round keeps in the smaller tiles."""
import pytest

from test_gpu_route_edges import check_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,k,d", [(4100, 64, 8, 1024), (4095, 63, 4, 1056), (8193, 16, 2, 1024), (8200, 9, 2, 1504), (8170, 17, 3, 1248),
                                     (2050, 61, 8, 2080), (2048, 64, 1, 2336), (4097, 33, 4, 1024), (4096, 64, 8, 1024), (4065, 63, 4, 1056), (8192, 16, 2, 1024),
                                     (8163, 9, 2, 1504), (7936, 64, 2, 1536), (2017, 61, 8, 2080), (5000, 9, 2, 3104)])
def test_projection_in_blocks(M, N, k, d):
    check_route(M, N, k, d, "softmax", "bf16")
