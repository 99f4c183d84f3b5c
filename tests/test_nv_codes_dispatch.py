"""Which NVFP4 products go to the kernel that dequantizes both operands in its waves, with which tile, and what a caller's workspace has to do
with it, as the library's host code decides it (the stand-in for HIP of test_dispatch; no GPU runs)."""
import pytest

from tests.test_dispatch import NV, MX, OP_GEMM, OP_SPLIT, host  # noqa: F401  (host: the fixture)

OP_FASTEST = 7
# tile (token blocks, column blocks, waves on the same tokens, groups that share K): shapes that it is the cheapest for
SHAPES = {
    (2, 2, 1, 8): [(350, 76, 128), (273, 71, 256), (424, 60, 384), (302, 68, 640), (514, 95, 1664)],
    (2, 4, 1, 8): [(489, 572, 640), (345, 758, 768), (545, 485, 1664), (518, 557, 2944)],
    (4, 4, 1, 8): [(100, 6261, 1920), (49, 9436, 1664), (52, 8387, 2944)],
    (3, 4, 1, 4): [(65, 3326, 256), (65, 3152, 128), (133, 3658, 1408), (65, 5571, 768), (133, 3658, 2944)],
    (4, 4, 1, 4): [(99, 5764, 128), (107, 5469, 256), (103, 5496, 384), (49, 8631, 1152)],
    (5, 4, 1, 4): [(66, 8720, 128), (129, 6126, 256), (66, 8772, 384), (71, 8270, 1152)],
    (6, 4, 1, 4): [(81, 8568, 128), (278, 4907, 256), (86, 8752, 384), (274, 4237, 1152)],
    (7, 4, 2, 2): [(132, 11144, 128), (217, 8394, 256), (525, 5452, 384), (295, 8998, 1152)],
    (8, 4, 2, 2): [(585, 5384, 128), (342, 8250, 256), (456, 7036, 384), (576, 5573, 1152)],
}


def kernel(tile):
    return "gemm_nv_codes_kernelI" + "".join(f"Li{v}E" for v in tile)


@pytest.mark.parametrize("tile", list(SHAPES))
def test_tiles_of_products_in_one_launch(host, tile):
    for M, N, K in SHAPES[tile]:
        need = host(["bytes", OP_GEMM, M, N, K, NV])[0]
        (launch,) = host(["device", 0, 256], ["gemm", M, N, K, NV, need])[1]
        assert kernel(tile) in launch["kernel"], (M, N, K, launch)
        columns = 16 * tile[1] * tile[2]
        assert launch["grid"][0] == -(-M // (16 * tile[0])) * -(-N // columns)


@pytest.mark.parametrize("M,N,K,codes", [(192, 4096, 4096, True), (320, 8192, 8192, True), (128, 4096, 4096, True), (600, 520, 2048, True), (320, 8192, 28672, False), (300, 10240, 14336, False),
                                         (128, 28672, 4096, True), (33, 57344, 8192, False), (640, 2048, 2048, True), (2048, 57344, 8192, False), (16, 8192, 8192, False)])
def test_more_room_never_leads_to_the_slower_kernel(host, M, N, K, codes):
    """The kernel follows the prices, not the bytes that are left over: with the size for parts and with far more, what is chosen with the size that
    promises the fastest call; that size is one of the two, and the larger only where the product runs in parts."""
    need, split, fastest = host(["device", 0, 256], *(["bytes", op, M, N, K, NV] for op in (OP_GEMM, OP_SPLIT, OP_FASTEST)))[1:]
    runs = host(["device", 0, 256], *(["gemm", M, N, K, NV, room] for room in (need, fastest, split, split + (1 << 30))))[1:]
    names = [[r["kernel"] for r in run] for run in runs]
    assert names[1] == names[2] == names[3]
    assert all(("gemm_nv_codes" in n[0]) == codes for n in names[1:])
    assert fastest == (split if "nv16_reduce" in names[2][-1] else need)
    if split > need and not codes:
        assert "nv16_reduce" in names[2][-1] and "nv16_reduce" not in names[0][-1]


@pytest.mark.parametrize("M,N,K", [(201, 4096, 14336), (128, 4096, 28672), (64, 4096, 4096)])
def test_mxfp4_is_always_fastest_with_room_for_parts(host, M, N, K):
    split, fastest = host(["device", 0, 256], *(["bytes", op, M, N, K, MX] for op in (OP_SPLIT, OP_FASTEST)))[1:]
    assert fastest == split


@pytest.mark.parametrize("M,N,K", [(1024, 8192, 8192), (1024, 8192, 14336), (512, 16384, 8192), (2048, 4096, 8192), (192, 57344, 4096), (192, 57344, 5120), (768, 10240, 14336), (2048, 10240, 8192)])
def test_a_whole_last_round_is_priced_as_a_last_one(host, M, N, K):
    """Launches that fill the last round, or nearly: 4 to 12 % slower on this kernel, which price it below the others where a round that is whole counts as one of many."""
    fastest = host(["device", 0, 256], ["bytes", OP_FASTEST, M, N, K, NV])[1]
    runs = host(["device", 0, 256], ["gemm", M, N, K, NV, fastest])[1]
    assert not any("gemm_nv_codes" in r["kernel"] for r in runs)
