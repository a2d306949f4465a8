"""bf16 products on 256 x 256 and 128 x 256 tiles: the same bits as the
128 x 128-tile kernel with register-staged loads (LSTMSS_OPT_GEMM_DMA = 0), which
sums every output in the same order, in the forward, the per-step dh product
(dense, gathered and with the selection inside) and the batched input gradient.

CASES names the product and tile each size is for (test_product_tiles.py checks
that the dispatch takes it): at least 192 work-groups of a step's tiles, steps and
splits; with rows and columns that end inside a tile, and more gathered rows than
the row table holds (K' > 2048).  Calls are enqueued in order on one stream, so
that the input gradient's launch covers all T steps.
"""
import pytest
import torch

from paper_1806_00512_amd.inputs import make_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1806_00512_amd.lstmss as lstmss
    lstmss.load()
    return lstmss


# T, B, I, H, sparsity, product, its tile
CASES = [
    (28, 200, 64, 512, 0.5, "input projection", (256, 256)),   # ragged columns
    (100, 136, 264, 640, 0.0, "input gradient", (256, 256)),   # ragged rows, dense
    (100, 256, 264, 1088, 0.5, "input gradient", (256, 256)),  # gathered, K' = 2176
    (70, 200, 264, 1088, 0.5, "input gradient", (128, 256)),   # gathered, ragged both ways
    (70, 200, 264, 640, 0.0, "input gradient", (128, 256)),    # dense
    (3, 256, 64, 2048, 0.5, "dh", (128, 256)),                 # selection inside
    (3, 192, 64, 2048, 0.0, "dh", (128, 256)),                 # dense, ragged columns
    (100, 128, 264, 1600, 0.25, "recurrent", (128, 128)),      # up to 128 columns
]


@pytest.mark.parametrize("T,B,I,H,sp", [c[:5] for c in CASES])
def test_big_tiles_same_bits(L, T, B, I, H, sp):
    d = make_layer(T, B, I, H, seed=3 * T + B + H, w_scale=0.05, dtype="bf16", state=True)
    g = {k: torch.from_numpy(d[k]).to("cuda:0") for k in ("b", "h0", "c0", "dH_up", "dhT", "dcT")}
    x, W = (torch.from_numpy(d[k]).to("cuda:0").to(torch.bfloat16) for k in ("x", "W"))
    outs = []
    try:
        L.set_option("wgrad_big", 0)
        L.set_option("side_stream", 0)
        for dma in (1, 0):
            L.set_option("gemm_dma", dma)
            h, cache = L.fwd_cache(x, W, g["b"], g["h0"], g["c0"])
            if sp:
                o = L.bwd_structsparse(x, W, cache, g["dH_up"], sparsity=sp, P=4, R=8, dhT=g["dhT"],
                                       dcT=g["dcT"])
            else:
                o = L.bwd_dense(x, W, cache, g["dH_up"], dhT=g["dhT"], dcT=g["dcT"])
            torch.cuda.synchronize()
            outs.append(dict({k: v for k, v in o.items() if torch.is_tensor(v)}, h=h))
    finally:
        L.set_option("gemm_dma", 1)
        L.set_option("wgrad_big", 1)
        L.set_option("side_stream", 2)
    assert set(outs[0]) >= {"dX", "dW", "db", "dh0", "dc0", "h"}
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k
        if outs[0][k].is_floating_point():
            assert torch.isfinite(outs[0][k]).all(), k
