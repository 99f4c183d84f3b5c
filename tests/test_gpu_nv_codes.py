"""NVFP4 products in one launch, both operands dequantized by every wave: each tile at ragged token counts and columns (also such that rows are stored value by value), and
shares of K from one fragment -- groups without a share -- to ones that differ from group to group.  Codes are random bytes and scales 1 and 1.5, so that every partial sum
is a multiple of 1/16 below 2^24 / 16: the result is the exact one, whatever the order of the sums."""
import pytest

from tests.test_nv_codes_dispatch import SHAPES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fp4():
    from paper_2509_23202_amd import binding
    return binding


def operand(fp4, g, rows, K):
    """Codes and scales in canonical order, and what they stand for."""
    import torch
    codes = torch.randint(0, 256, (rows, K // 2), device="cuda", dtype=torch.uint8, generator=g)
    scales = torch.where(torch.rand(rows, K // 16, device="cuda", generator=g) < 0.5, 0x38, 0x3c).to(torch.uint8)
    one = torch.ones(1, device="cuda")
    return codes.view(-1), scales.view(-1), one, fp4.fp4_dequantize(codes.view(-1), scales.view(-1), one, rows, K, fp4.NVFP4, flags=fp4.OUT_F32).double()


@pytest.mark.parametrize("tile", list(SHAPES))
def test_products_are_exact(fp4, tile):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(tile))
    for M, N, K in SHAPES[tile]:
        print(f"[case] nvfp4 codes tile={tile} M={M} N={N} K={K}", flush=True)
        ac, asc, one, a = operand(fp4, g, M, K)
        wc, wsc, _, w = operand(fp4, g, N, K)
        Y = a @ w.t()
        assert float((a.abs() @ w.abs().t()).max()) * 16 < 2 ** 24
        for flags in (fp4.OUT_F32, 0):
            room = torch.empty(fp4.workspace_bytes(fp4.OP_GEMM, M, N, K, fp4.NVFP4, flags), dtype=torch.uint8, device="cuda")
            out = fp4.fp4_gemm(ac, asc, one, wc, wsc, one, M, N, K, fp4.NVFP4, flags=flags, workspace=room)
            assert torch.equal(out, Y.to(out.dtype)), (M, N, K, flags)


@pytest.mark.parametrize("tile", list(SHAPES))
def test_every_scale_and_other_tensor_scales(fp4, tile):
    """Every finite E4M3 scale of either operand, zero and subnormal ones too, and tensor scales that are not 1.  A row of X has one group that is not zero, so that an output is a single
    s_x s_w times a sum of sixteen code products -- multiples of 1/4 up to 576, and 8 bits of scales: exact in fp32 -- times the rounded product of the tensor scales."""
    import torch
    M, N, K = SHAPES[tile][-1]
    G = K // 16
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(tile) + 100)
    at, wt = torch.full((1,), 0.0371, device="cuda"), torch.full((1,), 2.3e-3, device="cuda")
    one = torch.ones(1, device="cuda")
    for first in range(0, 127, M):
        print(f"[case] nvfp4 codes scales tile={tile} M={M} N={N} K={K} from {first}", flush=True)
        rows = torch.arange(M, device="cuda")
        asc = torch.zeros(M, G, dtype=torch.uint8, device="cuda")
        asc[rows, (first + 5 * rows) % G] = ((first + rows) % 127).to(torch.uint8)
        ac = torch.randint(0, 256, (M, K // 2), device="cuda", dtype=torch.uint8, generator=g)
        wsc = torch.randint(0, 127, (N, G), device="cuda", dtype=torch.uint8, generator=g)
        wc = torch.randint(0, 256, (N, K // 2), device="cuda", dtype=torch.uint8, generator=g)
        assert len(wsc.unique()) == 127
        a, w = (fp4.fp4_dequantize(c.view(-1), s.view(-1), one, r, K, fp4.NVFP4, flags=fp4.OUT_F32).double() for c, s, r in ((ac, asc, M), (wc, wsc, N)))
        Y = (a @ w.t()).float() * (at * wt)
        for flags in (fp4.OUT_F32, 0):
            room = torch.empty(fp4.workspace_bytes(fp4.OP_GEMM, M, N, K, fp4.NVFP4, flags), dtype=torch.uint8, device="cuda")
            out = fp4.fp4_gemm(ac.view(-1), asc.view(-1), at, wc.view(-1), wsc.view(-1), wt, M, N, K, fp4.NVFP4, flags=flags, workspace=room)
            assert torch.equal(out, Y.to(out.dtype)), (M, N, K, flags)


def test_replays_of_a_graph(fp4):
    """Captured, and replayed with work of its own in between: every replay is the eager result."""
    import torch
    M, N, K = 192, 4096, 2048
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    ac, asc, one, a = operand(fp4, g, M, K)
    wc, wsc, _, w = operand(fp4, g, N, K)
    Y = (a @ w.t()).float()
    room = torch.empty(fp4.workspace_bytes(fp4.OP_GEMM, M, N, K, fp4.NVFP4, fp4.OUT_F32), dtype=torch.uint8, device="cuda")
    out = torch.empty(M, N, device="cuda")
    call = lambda: fp4.fp4_gemm(ac, asc, one, wc, wsc, one, M, N, K, fp4.NVFP4, flags=fp4.OUT_F32, workspace=room, out=out)
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, Y)
        torch.randn(1024, 1024, device="cuda").sum().item()
