"""Every kernel of the tiled dense aggregation that the plan can choose: each
tile of the matrix-core kernel with an odd and an even number of chunks (an odd
one is done before the loop), whole and in k ranges, in fp32 with one and with
several chains of additions per range; the streaming kernel with each number of
column tiles, whole and in ranges.  Each shape asserts its plan, so that a
change of the prices that leaves a kernel without a shape is seen."""
import pytest
import torch

from paper_2010_12635_amd import gcn as G
from tests.test_gpu_dense_ranges import _adj as adj, plan, tile

ROWS64, STREAM, MM = 0, 1, 2

# prec, n, F: kernel, rows, columns, several ranges, odd chunks (MM) or column
# tiles (others), chains
SHAPES = {
    (0, 300, 50): (ROWS64, 64, 64, False, 4, False), (0, 300, 100): (ROWS64, 64, 64, False, 7, False),
    (1, 300, 1): (ROWS64, 64, 64, False, 1, False), (2, 2529, 200): (ROWS64, 64, 64, False, 13, False),
    (0, 2069, 1): (STREAM, 128, 64, True, 1, False), (0, 1886, 22): (STREAM, 128, 64, True, 2, False),
    (0, 1337, 36): (STREAM, 128, 64, True, 3, False), (0, 1032, 50): (STREAM, 128, 64, True, 4, False),
    (2, 6164, 8): (STREAM, 128, 64, True, 1, False), (1, 4953, 22): (STREAM, 128, 64, True, 2, False),
    (2, 4302, 36): (STREAM, 128, 64, True, 3, False), (1, 3868, 50): (STREAM, 128, 64, True, 4, False),
    (1, 20000, 1): (STREAM, 128, 64, False, 1, False), (2, 24000, 22): (STREAM, 128, 64, False, 2, False),
    (1, 24000, 36): (STREAM, 128, 64, False, 3, False), (2, 32768, 50): (STREAM, 128, 64, False, 4, False),
    # 16-bit tiles
    (1, 1215, 892): (MM, 128, 128, False, False, False), (2, 544, 1794): (MM, 128, 128, False, True, False),
    (2, 2191, 65): (MM, 128, 128, True, False, False), (1, 2252, 65): (MM, 128, 128, True, True, False),
    (1, 2366, 1712): (MM, 256, 128, False, False, False), (2, 2069, 1958): (MM, 256, 128, False, True, False),
    (2, 5387, 158): (MM, 256, 128, True, False, False), (1, 8208, 65): (MM, 256, 128, True, True, False),
    (1, 4519, 1794): (MM, 256, 192, False, False, False), (2, 4302, 1958): (MM, 256, 192, False, True, False),
    (2, 6906, 158): (MM, 256, 192, True, False, False), (1, 7123, 158): (MM, 256, 192, True, True, False),
    (2, 6255, 1958): (MM, 256, 256, False, False, False), (1, 5953, 2048): (MM, 256, 256, False, True, False),
    (1, 10595, 220): (MM, 256, 256, True, False, False), (2, 10161, 220): (MM, 256, 256, True, True, False),
    # fp32 tiles
    (0, 1947, 1958): (MM, 128, 128, False, False, False), (0, 6472, 1220): (MM, 128, 128, False, True, False),
    (0, 1276, 65): (MM, 128, 128, True, False, False), (0, 1581, 65): (MM, 128, 128, True, True, False),
    (0, 1337, 1958): (MM, 128, 128, False, False, True), (0, 1581, 1958): (MM, 128, 128, False, True, True),
    (0, 1093, 65): (MM, 128, 128, True, False, True), (0, 1032, 65): (MM, 128, 128, True, True, True),
    (0, 3868, 1712): (MM, 256, 128, False, False, False), (0, 3434, 1958): (MM, 256, 128, False, True, False),
    (0, 910, 1302): (MM, 256, 128, True, False, False), (0, 971, 1302): (MM, 256, 128, True, True, False),
    (0, 8208, 65): (MM, 256, 128, True, False, True), (0, 12331, 65): (MM, 256, 128, True, True, True),
    (0, 5170, 1958): (MM, 256, 192, False, False, False), (0, 5387, 1794): (MM, 256, 192, False, True, False),
    (0, 4085, 158): (MM, 256, 192, True, False, False), (0, 1520, 1384): (MM, 256, 192, True, True, False),
    (0, 6906, 1958): (MM, 256, 256, False, False, False), (0, 6689, 2040): (MM, 256, 256, False, True, False),
    (0, 2191, 974): (MM, 256, 256, True, False, False), (0, 2069, 974): (MM, 256, 256, True, True, False),
}


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_plan(shape):
    prec, n, F = shape
    kernel, rows, cols, ranges, chunks, chain = plan(prec, n, F)
    last = chunks % 2 == 1 if kernel == MM else (F + 15) // 16
    assert (kernel, rows, cols, ranges > 1, last, chain > 0) == SHAPES[shape]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_product(shape):
    """Operands of -1, 0 and 1: every sum is a whole number below 2^24, exact in any
    order, and the result is its rounding to storage, so that a chunk left out or
    taken twice shows at any n."""
    prec, n, F = shape
    dt = G.torch_dtype(prec)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + F)
    A = torch.randint(-1, 2, (n, n), generator=gen, device="cuda", dtype=torch.int8).to(dt)
    ld = (F + 7) // 8 * 8
    X = torch.full((n, ld), float("nan"), dtype=dt, device="cuda")   # padding is ignored
    X[:, :F] = torch.randint(-1, 2, (n, F), generator=gen, device="cuda").to(dt)
    bias = torch.randint(-9, 10, (ld,), generator=gen, device="cuda").float()
    At = tile(A, prec)
    a = adj(n, prec, At.data_ptr())
    Y = torch.full((n, ld + 8), 7.0, dtype=dt, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.full((G.gcn_aggregate_workspace_size(a, F, prec),), 255, dtype=torch.uint8, device="cuda")
    G.gcn_aggregate(a, F, prec, X, ld, bias, G.GCN_ACT_RELU, 0.0, False, 0, 0, 0, Y, ld + 8, flag, ws)
    want = (A.double() @ X[:, :F].double() + bias[:F].double()).clamp_(min=0)
    assert torch.equal(Y[:, :F], want.to(dt)) and flag.item() == 0
