"""fp32 products on bf16 matrix instructions (operands split three ways)
through the backward call, at the edges of their tiles: contraction lengths
with a tail, odd sizes, unaligned rows, the gathered-row table's refills, each
tile shape, and operands that are not finite.

The call returns its gate gradients (dbg) and kept indices, so the products
are checked on their own against fp64 sums of the same operands, element by
element, with an error bound from the arithmetic: a partial product of bf16
values is exact, the ones left out are below 4 * 2^-27 of |a b|, and every
group of 8 terms is rounded once into the accumulator (data gradient: one
accumulator for the leading partial products; weight gradient: all six in
one), each time by at most 2^-23 of the sum of |a b|.  That bound grows with the
number of terms, so the norm of the error is bounded too: without one of the
partial products of a low plane it is at least 2.4e-6 of the result's."""
import numpy as np
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


def gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def call(L, d, sp, kw, edit=None):
    x, W, dH = gpu(d["x"]), gpu(d["W"]), gpu(d["dH_up"])
    if edit is not None:
        edit(x, W, dH)
    _, cache = L.fwd_cache(x, W, gpu(d["b"]))
    o = L.bwd_structsparse(x, W, cache, dH, sparsity=sp, want_dbg=True, **kw)
    torch.cuda.synchronize()
    T, I, B = x.shape
    h = L.cache_views(cache, T, B, W.shape[0] // 4, "f32")[2][:T]
    return o, torch.cat([x, h], 1).double(), W.double()


def masked(o, sp, kw, T):
    """The sparsified gate gradients [T][4H][B] in fp64."""
    dG = o["dbg"].double()
    keep = torch.zeros(dG.shape, dtype=torch.bool, device=dG.device)
    if kw.get("kind"):
        Mx, My = kw["Mx"], kw["My"]
        idx = o["idx"].view(T, dG.shape[1] // Mx, -1).long()
        nb = -(-dG.shape[2] // My)
        blk = torch.zeros((T, idx.shape[1], nb), dtype=torch.bool, device=dG.device)
        blk.scatter_(2, idx, True)
        keep = blk.repeat_interleave(Mx, 1).repeat_interleave(My, 2)[:, :, :dG.shape[2]]
    else:
        P = kw.get("P", 4)
        rows = (o["idx"].long()[:, :, None] * P + torch.arange(P, device=dG.device)).view(T, -1)
        keep.scatter_(1, rows[:, :, None].expand(-1, -1, dG.shape[2]), True)
    return torch.where(keep, dG, torch.zeros((), dtype=dG.dtype, device=dG.device))


def check(got, ref, mag, terms, what):
    err = (got.double() - ref).abs()
    bound = (terms * 2.0 ** -23 + 2.0 ** -25) * mag + 1e-37
    assert bool((err <= bound).all()), "%s: %.3g of the bound" % (what, (err / bound).max().item())
    e = ((got.double() - ref).norm() / ref.norm()).item()
    assert e <= 8e-7, (what, e)


COARSE = {"P": 4, "R": 8}
FINE32 = {"kind": 1, "My": 32, "Mx": 32}


@pytest.mark.parametrize("T,B,I,H,sp,kw", [
    (2, 1, 7, 5, 0.0, COARSE),            # one column, odd rows, scalar loads
    (2, 13, 33, 31, 0.5, COARSE),         # odd everything, partial region
    (2, 20, 130, 150, 0.5, COARSE),       # K' with a 4-row tail, 128 x 32 tiles
    (3, 33, 64, 70, 0.25, COARSE),        # 33 columns: 64-column tiles, odd row length
    (2, 50, 66, 72, 0.75, {"P": 1, "R": 4}),   # even, rows of 8 but not 16 bytes
    (2, 17, 96, 64, 0.875, {"P": 4, "R": 8}),  # one kept slice per region
    (2, 40, 64, 64, 0.5, {"P": 8, "R": 8}),    # two temporary tiles per group
    (2, 70, 40, 96, 0.5, {"P": 16, "R": 8}),   # 64 kept, 128 original rows per group
    (2, 64, 96, 1096, 0.0, COARSE),       # K' = 4384: 137 stages of 32
    (2, 32, 256, 2200, 0.5, COARSE),      # 4400 gathered rows: refills of the row table
    (2, 130, 2050, 1030, 0.25, COARSE),   # 128 x 128 tiles with ragged edges, gathered
    (1, 40, 2060, 2044, 0.0, COARSE),     # 128 x 256 weight-gradient tiles, ragged
    (1, 32, 2048, 2048, 0.5, FINE32),     # 128 x 256 tiles, one block per slice
    (2, 96, 72, 64, 0.3333333, FINE32),   # fine blocks, ragged feature tiles
])
def test_products_against_fp64(L, T, B, I, H, sp, kw):
    if kw.get("kind") and B // 32 == 1:
        sp = 0.0
    d = make_layer(T, B, I, H, seed=T + 3 * B + I + H, w_scale=0.1)
    o, xh, W = call(L, d, sp, kw)
    dG = masked(o, sp, kw, T)
    kept = L.kept_rows(L.dims(T, B, I, H), sp, L.structure(**{"kind": 0, **kw}))
    ref = W[:, :I].t() @ dG
    mag = W[:, :I].t().abs() @ dG.abs()
    check(o["dX"], ref, mag, -(-kept // 8) + 1, "dX")
    ref = sum(dG[t] @ xh[t].t() for t in range(T))
    mag = sum(dG[t].abs() @ xh[t].t().abs() for t in range(T))
    check(o["dW"], ref, mag, 6 * T * (-(-B // 8) + 2) + T, "dW")


@pytest.mark.parametrize("T,B,I,H,sp,kw", [
    (35, 64, 96, 128, 0.0, COARSE), (35, 64, 96, 128, 0.5, COARSE), (35, 64, 96, 128, 0.5, FINE32),
    (40, 300, 96, 128, 0.75, COARSE),     # a step's columns in two sums
    (9, 128, 2048, 1024, 0.0, COARSE),    # 128 x 256 tiles
])
def test_weight_gradient_sums(L, T, B, I, H, sp, kw):
    # as accurate as fp32 matrix instructions with a sum per step (measured
    # 1.1e-7 to 2.4e-7), without a mean (those: below 1e-10; one long sum: 7e-7 and
    # -8e-8 at T * B = 2240)
    d = make_layer(T, B, I, H, seed=12, w_scale=0.1)
    o, xh, W = call(L, d, sp, kw)
    dG = masked(o, sp, kw, T)
    ref = sum(dG[t] @ xh[t].t() for t in range(T))
    e, rms = o["dW"].double() - ref, ref.square().mean().sqrt().item()
    assert e.square().mean().sqrt().item() <= 3e-7 * rms
    assert abs(e.mean().item()) <= 5e-9 * rms


@pytest.mark.parametrize("T,B,I,H", [(2, 20, 130, 150), (1, 130, 1040, 1030)])
def test_small_operands(L, T, B, I, H):
    # gate gradients of some 2^-120: all of their 24 bits count (without the 14
    # lowest the error would be 1e-5)
    d = make_layer(T, B, I, H, seed=11, w_scale=0.2)
    o, xh, W = call(L, d, 0.5, COARSE, lambda x, W, dH: dH.mul_(2.0 ** -118))
    dG = masked(o, 0.5, COARSE, T)
    assert 0 < dG.abs().max().item() < 2.0 ** -114
    ref = W[:, :I].t() @ dG
    assert ((o["dX"].double() - ref).norm() / ref.norm()).item() <= 1e-6
    ref = sum(dG[t] @ xh[t].t() for t in range(T))
    assert ((o["dW"].double() - ref).norm() / ref.norm()).item() <= 1e-6


@pytest.mark.parametrize("sp,kw", [(0.0, COARSE), (0.5, COARSE), (0.5, {"P": 16, "R": 8})])
def test_not_finite(L, sp, kw):
    # infinities and NaN reach exactly the results they reach in fp32
    T, B, I, H = 1, 36, 40, 64  # (one step: dh would carry them to every row)
    d = make_layer(T, B, I, H, seed=9, w_scale=0.2)

    def edit(x, W, dH):
        dH[0, 3, 5] = float("inf")
        dH[0, 20, 30] = float("-inf")
        dH[0, 9, 7] = float("nan")
    o, xh, W = call(L, d, sp, kw, edit)
    assert torch.isinf(o["dW"]).any() and torch.isfinite(o["dW"]).any()
    assert torch.isnan(o["dX"]).any() and torch.isfinite(o["dX"]).any()
    dG = masked(o, sp, kw, T)
    rows = [dG[t].abs().sum(1) != 0 for t in range(T)]  # kept rows (NaN != 0)

    def same(got, ref, what):
        got = got.double()
        assert torch.equal(torch.isnan(got), torch.isnan(ref)), what
        assert torch.equal(torch.isposinf(got), torch.isposinf(ref)), what
        assert torch.equal(torch.isneginf(got), torch.isneginf(ref)), what
        f = torch.isfinite(ref)
        e = (got[f] - ref[f]).norm() / ref[f].norm()
        assert e <= 1e-5, (what, e)
    same(o["dX"], torch.stack([W[rows[t], :I].t() @ dG[t][rows[t]] for t in range(T)]), "dX")
    ref = torch.zeros_like(W)
    for t in range(T):
        ref[rows[t]] += dG[t][rows[t]] @ xh[t].t()
    same(o["dW"], ref, "dW")


def test_fine_not_finite(L):
    # an infinite feature reaches the rows whose slice keeps its block, and no
    # others (removed blocks are not multiplied, nor in the fp32 recomputation)
    T, B, I, H = 1, 64, 40, 64
    d = make_layer(T, B, I, H, seed=10, w_scale=0.2)

    def edit(x, W, dH):
        x[0, 3, 40] = float("inf")
    o, xh, W = call(L, d, 0.5, FINE32, edit)
    kept = (o["idx"].view(-1) == 1).repeat_interleave(32)  # one block of two per slice
    assert kept.any() and not kept.all()
    bad = ~torch.isfinite(o["dW"])
    assert torch.equal(bad[:, 3], kept)
    bad[:, 3] = False
    assert not bad.any()


@pytest.mark.parametrize("T,B,I,H", [(2, 1, 7, 5), (2, 20, 130, 150), (2, 33, 66, 70),
                                     (2, 129, 520, 2050), (1, 128, 2048, 2048)])
def test_forward_products_against_fp64(L, T, B, I, H):
    # one step from h0 = 0: the pre-activations are the input projection alone
    # (rows of 4, 8 and 16 bytes); later steps add the recurrent product
    d = make_layer(T, B, I, H, seed=I + H, w_scale=0.5 / np.sqrt(H))
    x, W, b = gpu(d["x"]), gpu(d["W"]), gpu(d["b"])
    _, cache = L.fwd_cache(x, W, b)
    torch.cuda.synchronize()
    gates, c, h = [v.double() for v in L.cache_views(cache, T, B, H, "f32")]
    Wd = W.double()
    for t in range(T):
        z = Wd @ torch.cat([x[t].double(), h[t]]) + b.double()[:, None]
        g = torch.cat([z[:2 * H].sigmoid(), z[2 * H:3 * H].tanh(), z[3 * H:].sigmoid()])
        e = (gates[t] - g).norm() / g.norm()
        assert e <= 8e-7, (t, e)
