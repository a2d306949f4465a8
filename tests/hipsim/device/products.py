"""Runs the product kernels' launchers in the CPU stand-in of the device: cases as
JSON lines on the standard input, one line of relative errors against fp64 sums
for each.  Every operand and result has its exact size, so that the address
sanitizer sees any access past it; outputs and LDS start out as garbage."""
import ctypes
import json
import sys

import numpy as np

i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p


class Gemm1Args(ctypes.Structure):
    _fields_ = [("W", vp), ("ldw", i64), ("Gc", vp), ("idx", vp), ("P", i32), ("Kp", i64), ("M", i32),
                ("m_begin", i32), ("N", i32), ("out_row0", i32), ("m_lo", i32), ("part", vp),
                ("part_stride", i64), ("splitk", i32), ("k_chunk", i64), ("steps", i32),
                ("gc_step", i64), ("idx_step", i64), ("out_step", i64), ("tm", i32), ("tn", i32),
                ("kcol0", i32), ("fidx", vp), ("fkept", i32), ("fidx_step", i64),
                ("dma", i32), ("sel_sq", vp), ("sel_nch", i32), ("sel_R", i32), ("sel_S", i32),
                ("sel_nslices", i64), ("sel_gc", vp), ("sel_idx", vp)]


class WgradArgs(ctypes.Structure):
    _fields_ = [("Gc", vp), ("idx", vp), ("x", vp), ("h", vp), ("T", i32), ("I", i32), ("H", i32),
                ("B", i32), ("Kp", i32), ("kept", i32), ("P", i32), ("R", i32), ("S", i32), ("greg", i32),
                ("BC", i32), ("t_begin", i32), ("t_end", i32), ("accumulate", i32), ("dW", vp),
                ("fidx", vp), ("fkept", i32), ("fskip", i32), ("dma", i32), ("big", i32)]


lib = ctypes.CDLL(sys.argv[1])
fn = {n: getattr(lib, "_ZN6lstmss%d%sENS_%sEbP12ihipStream_t" % (len(n), n, a)) for n, a in
      (("launch_gemm1", "9Gemm1Args"), ("launch_gemm_fwd", "9Gemm1Args"))}
fn["launch_wgrad"] = getattr(lib, "_ZN6lstmss12launch_wgradENS_9WgradArgsEbbP12ihipStream_t")
fn["launch_gemm1"].argtypes = fn["launch_gemm_fwd"].argtypes = [Gemm1Args, ctypes.c_bool, vp]
fn["launch_wgrad"].argtypes = [WgradArgs, ctypes.c_bool, ctypes.c_bool, vp]


def store(a, bf16):
    """(stored array, the values it holds)"""
    a = np.ascontiguousarray(a, np.float32)
    if not bf16:
        return a, a.astype(np.float64)
    u = a.view(np.uint32)
    u = ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    return u, (u.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def junk(shape, dtype):
    a = np.empty(shape, dtype)
    a.view(np.uint8).reshape(-1)[:] = 0xc5
    return a


def ptr(a):
    return a.ctypes.data


def rel(got, ref):
    return float(np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-300))


def values(c, rng, *shape, scale="scale"):
    v = rng.standard_normal(shape).astype(np.float32) * np.float32(c.get(scale, 1.0))
    return v


def product(c, rng):
    """The data-gradient and forward products."""
    bf16, mode, P = c["bf16"], c["mode"], c.get("P", 4)
    M, N, m0, steps, rows = c["M"], c["N"], c.get("m_begin", 0), c.get("steps", 1), c["rows"]
    a = Gemm1Args()
    a.P, a.M, a.m_begin, a.out_row0, a.N, a.steps = P, M, m0, m0, N, steps
    a.splitk, a.tm, a.tn, a.dma = c.get("splitk", 1), c["tm"], c["tn"], c.get("dma", 1)
    keep = []
    if mode == "rowa":  # out = W[:, kcol0:] G
        kc, K = c.get("kcol0", 0), rows
        W, Wd = store(values(c, rng, M, kc + K, scale="wscale"), bf16)
        G, Gd = store(values(c, rng, steps, K, N), bf16)
        a.kcol0, a.ldw, a.Kp, a.gc_step = kc, kc + K, K, K * N
        ref = np.stack([Wd[:, kc:] @ Gd[s] for s in range(steps)])
    else:
        ldw = c.get("ldw", M)
        W, Wd = store(values(c, rng, rows, ldw, scale="wscale"), bf16)
        a.ldw = ldw
        R, S = c.get("R", 8), c.get("S", 4)
        nsl = rows // P
        if mode == "gather":
            kept = c["kept"] // P
            idx = np.stack([np.sort(rng.permutation(nsl)[:kept]) for _ in range(steps)]).astype(np.int32)
            K = kept * P
            G, Gd = store(values(c, rng, steps, K, N), bf16)
            a.idx, a.idx_step = ptr(idx), kept
            ref = np.stack([Wd[(idx[s][:, None] * P + np.arange(P)).ravel()][:, m0:M].T @ Gd[s]
                            for s in range(steps)])
        elif mode == "sel":
            G, Gd = store(values(c, rng, 1, rows, N), bf16)
            nch = -(-N // 64)
            sq = np.zeros((rows, nch))
            for ch in range(nch):
                sq[:, ch] = (Gd[0][:, 64 * ch:64 * ch + 64] ** 2).sum(1)
            score = sq.sum(1).reshape(nsl, P).sum(1)
            chosen = []
            for r0 in range(0, nsl, R):
                r = min(R, nsl - r0)
                order = np.argsort(-score[r0:r0 + r], kind="stable")
                chosen += sorted(r0 + order[:r - S * r // R])
            chosen = np.array(chosen, np.int32)
            rws = (chosen[:, None] * P + np.arange(P)).ravel()
            K = len(rws)
            gc, sidx = junk((K, N), G.dtype), junk(len(chosen), np.int32)
            a.sel_sq, a.sel_nch, a.sel_R, a.sel_S, a.sel_nslices = ptr(sq), nch, R, S, nsl
            a.sel_gc, a.sel_idx = ptr(gc), ptr(sidx)
            ref = (Wd[rws][:, m0:M].T @ Gd[0][rws])[None]
        elif mode == "fine":  # blocks of 32 x 32, masked
            K, kept, nb = rows, c["kept"], N // 32
            G = values(c, rng, steps, K, N)
            fidx = np.stack([[np.sort(rng.permutation(nb)[:kept]) for _ in range(K // 32)]
                             for _ in range(steps)]).astype(np.int32)
            mask = np.zeros((steps, K // 32, nb), bool)
            np.put_along_axis(mask, fidx, True, 2)
            G *= np.repeat(np.repeat(mask, 32, 1), 32, 2)
            G, Gd = store(G, bf16)
            a.fidx, a.fkept, a.fidx_step, a.P = ptr(fidx), kept, kept * (K // 32), 32
            ref = np.stack([Wd[:, m0:M].T @ Gd[s] for s in range(steps)])
        else:
            K = rows
            G, Gd = store(values(c, rng, steps, K, N), bf16)
            ref = np.stack([Wd[:, m0:M].T @ Gd[s] for s in range(steps)])
        a.Kp, a.gc_step = K, K * N
        keep = [v for k, v in locals().items() if k in ("idx", "sq", "gc", "sidx", "fidx")]
    unit = c.get("unit", 64)  # a split is a multiple of this many k
    per = -(-K // a.splitk)
    a.k_chunk = -(-per // unit) * unit
    a.splitk = -(-K // a.k_chunk)
    if c.get("wild"):
        idx[0, 3] = 1 << 20
    out = junk((steps, a.splitk, M - m0, N), np.float32)
    if c.get("short"):
        out = junk((steps, a.splitk, M - m0 - 1, N), np.float32)
    a.W, a.Gc, a.part = ptr(W), ptr(G), ptr(out)
    a.part_stride, a.out_step = (M - m0) * N, a.splitk * (M - m0) * N
    rc = fn["launch_gemm_fwd" if mode == "rowa" else "launch_gemm1"](a, bf16, None)
    assert rc == 0, rc
    r = {"out": rel(out.astype(np.float64).sum(1), ref), "splits": a.splitk}
    if mode == "sel":
        assert (sidx == chosen).all(), "index"
        assert (gc == G[0][rws]).all(), "compacted rows"
    del keep
    return r


def wgrad(c, rng):
    bf16, T, B, I, H, P, R, S = [c[k] for k in ("bf16", "T", "B", "I", "H", "P", "R", "S")]
    x, xd = store(values(c, rng, T, I, B, scale="wscale"), bf16)
    h, hd = store(values(c, rng, T + 1, H, B, scale="wscale"), bf16)
    dG = values(c, rng, T, 4 * H, B)
    a = WgradArgs()
    nsl, fine, dense = 4 * H // P, c.get("fine", 0), S == 0 and not c.get("fine", 0)
    mask = np.ones((T, 4 * H, B), bool)
    if fine:
        nb = B // 32
        fidx = np.stack([[np.sort(rng.permutation(nb)[:fine]) for _ in range(4 * H // 32)]
                         for _ in range(T)]).astype(np.int32)
        m = np.zeros((T, 4 * H // 32, nb), bool)
        np.put_along_axis(m, fidx, True, 2)
        mask = np.repeat(np.repeat(m, 32, 1), 32, 2)
        a.fidx, a.fkept, a.fskip, Kp, P, R = ptr(fidx), fine, c.get("skip", 1), 4 * H, 32, nb
        Gc, Gd = store(dG * mask, bf16)
        Gd = Gd.reshape(T, 4 * H, B)
    elif dense:
        Kp, P, R = 4 * H, 1, 1
        Gc, Gd = store(dG, bf16)
    else:
        idx = []
        for t in range(T):
            l = []
            for r0 in range(0, nsl, R):
                r = min(R, nsl - r0)
                l += sorted(r0 + rng.permutation(r)[:r - S * r // R])
            idx.append(l)
        idx = np.array(idx, np.int32)
        rows = (idx[:, :, None] * P + np.arange(P)).reshape(T, -1)
        Kp = rows.shape[1]
        Gc, Gcd = store(np.stack([dG[t][rows[t]] for t in range(T)]), bf16)
        Gd = np.zeros((T, 4 * H, B))
        for t in range(T):
            Gd[t][rows[t]] = Gcd[t]
        a.idx, a.kept = ptr(idx), idx.shape[1]
    for k, row, col in c.get("infs", []):  # infinite entries of x: (step, feature, column)
        x[k, row, col] = xd[k, row, col] = np.inf
    out = junk((4 * H, I + H), np.float32)
    a.Gc, a.x, a.h, a.dW = ptr(Gc), ptr(x), ptr(h), ptr(out)
    a.T, a.I, a.H, a.B, a.Kp, a.P, a.R, a.S = T, I, H, B, Kp, P, R, S
    a.dma, a.big = c.get("dma", 1), c.get("big", 1)
    cut = c.get("cut", 0)  # two launches, the second continuing from the stored dW
    for lo, hi, acc in ([(cut, T, 0), (0, cut, 1)] if cut else [(0, T, 0)]):
        a.t_begin, a.t_end, a.accumulate = lo, hi, acc
        rc = fn["launch_wgrad"](a, bool(a.idx), bf16, None)
        assert rc == 0, rc
    with np.errstate(all="ignore"):
        ref = np.zeros((4 * H, I + H))
        for t in range(T):
            f = np.concatenate([xd[t], hd[t]])
            if c.get("infs"):  # removed blocks are not multiplied
                for b in range(B):
                    rws = mask[t][:, b]
                    ref[rws] += np.outer(Gd[t][rws, b], f[:, b])
            else:
                ref += Gd[t] @ f.T
    if c.get("infs"):
        assert (np.isnan(out) == np.isnan(ref)).all(), "NaN"
        assert (np.isinf(out) == np.isinf(ref)).all(), "inf"
        ok = np.isfinite(ref)
        assert not ok.all()
        return {"dW": rel(out[ok].astype(np.float64), ref[ok])}
    return {"dW": rel(out.astype(np.float64), ref)}


for line in sys.stdin:
    c = json.loads(line)
    print("case", line.strip(), flush=True)
    rng = np.random.default_rng(c.get("seed", 1))
    best = None
    for early, rev in c.get("orders", [[0, 0], [1, 1]]):
        lib.devsim_config(1, early, rev, c.get("sample", 0), 1)
        r = (wgrad if "T" in c else product)(c, np.random.default_rng(c.get("seed", 1)))
        assert best is None or r == best, ("order changes the result", r, best)
        best = r
    print("ok", json.dumps(best), flush=True)
