"""The work a user of this library has it do, as measurable cases: products with SpQR matrices at batch 1 (token by
token decoding), at small batches, at prompt-sized batches, and the quantiser that produces the matrices.

A product case names the kind of call, the format of the matrices and their shapes; codes are random bits (every bit
pattern of the code words is a valid set of codes), second-level statistics, outlier sets and activations follow the
distributions of spqr_synth.  Packed buffers are written directly in the layouts of include/spqr.h.
"""
import functools
import math

import numpy as np
import torch

import paper_2306_03078_amd as P
import paper_2306_03078_amd.encode_binding as E

# Formats: (w_bits, beta1, beta2); group_axis 1 is the orientation of the benchmark layers, 0 the one of Alg. 1 (what
# the quantiser writes).  layout 1 is the method's bilevel format, 2 and 3 the variants with integer zero points and
# with 16-bit statistics.


def _block(hidden, ffn):
    return [(hidden, hidden)] * 4 + [(ffn, hidden)] * 2 + [(hidden, ffn)]


def listed():
    fmt16 = dict(beta1=16, beta2=16, axis=1, layout=1, perm=False)
    fmt8 = dict(w=3, beta1=8, beta2=32, axis=1, layout=1, perm=False)
    return [
        # One small projection for one token: the smallest call there is; launch latency counts.
        dict(name="decode-4096", kind="gemv", m=4096, n=4096, w=3, **fmt16, rate=0.01, structure="uniform", b=1, f16=False),
        # One projection as the quantiser writes it with activation order (groups along a row, permuted inputs), wide
        # input, 16-bit output for a 16-bit residual stream.
        dict(name="decode-actorder", kind="gemv", m=8192, n=22016, w=3, beta1=8, beta2=32, axis=0, layout=1, perm=True,
             rate=0.02, structure="cols64", b=1, f16=True),
        # A whole decoder block for one token: all seven projections in one call, at the 7B, 33B and 65B shapes.
        dict(name="decode-block-7b", kind="block", m=11008, n=4096, w=3, **fmt16, rate=0.01, structure="rows8cols4", b=1,
             f16=False),
        dict(name="decode-block-33b", kind="block", m=17920, n=6656, w=4, **fmt16, rate=0.01, structure="zipf", b=1,
             f16=False),
        dict(name="decode-block-65b", kind="block", m=22016, n=8192, **fmt8, rate=0.02, structure="cols64", b=1, f16=False),
        # A few sequences decoded together: q/k/v of one block for four of them.
        dict(name="batch4-qkv", kind="fused", m=6656, n=6656, count=3, w=4, **fmt16, rate=0.01, structure="zipf", b=4,
             f16=True),
        # Sixteen sequences decoded together, tall and wide layers of the two large shapes.
        dict(name="batch16-gate", kind="batch", m=17920, n=6656, w=4, **fmt16, rate=0.01, structure="zipf", b=16, f16=False),
        dict(name="batch16-down", kind="batch", m=8192, n=22016, **fmt8, rate=0.02, structure="cols64", b=16, f16=True),
        # A prompt: the largest batch the library takes, and a ragged one through gate and up together.
        dict(name="prompt256-gate", kind="batch", m=17920, n=6656, w=4, **fmt16, rate=0.01, structure="zipf", b=256,
             f16=False),
        dict(name="prompt77-gateup", kind="fused", m=11008, n=4096, count=2, w=3, **fmt16, rate=0.01, structure="rows8cols4",
             b=77, f16=True),
        # Quantising a layer, before the sweep: the Hessian of its calibration inputs and the factor of its inverse.
        dict(name="factor-4096", kind="factor", n=4096, d=4096),
        # The column sweep of one attention projection (the most frequent layer of a model), tau for about 1 % outliers.
        dict(name="quantize-4096", kind="quantize", m=4096, n=4096, w=3, beta1=16, beta2=16, tau=30.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemv", "gemv", "block", "batch", "batch", "fused", "prompt", "prompt", "factor", "quantize"])
    if kind == "factor":
        return dict(kind=kind, n=_log_int(rng, 200, 4000), d=_log_int(rng, 512, 4096))
    if kind == "quantize":
        beta1 = rng.choice([8, 16, 32])
        return dict(kind=kind, m=16 * _log_int(rng, 8, 250), n=32 * _log_int(rng, 8, 127), w=rng.choice([3, 4]), beta1=beta1,
                    beta2=16, tau=rng.choice([20.0, 40.0, math.inf]))
    w = rng.choice([3, 4])
    beta1, beta2 = rng.choice([(16, 16), (16, 16), (8, 32)])
    axis = rng.choice([0, 1])
    c = dict(kind=kind, m=0, n=0, w=w, beta1=beta1, beta2=beta2, axis=axis, layout=1, perm=False,
             rate=rng.choice([0.005, 0.01, 0.02]), structure=rng.choice(["uniform", "rows8cols4", "cols64", "zipf"]), b=1,
             f16=rng.choice([False, True]))
    # sizes in units of 32 (a multiple of every tile side), odd multiples as likely as even ones
    if kind == "block":
        h = 32 * _log_int(rng, 24, 240)
        c.update(n=h, m=32 * round(h * 2.69 / 32))
        return c
    c.update(m=32 * _log_int(rng, 32, 560), n=32 * _log_int(rng, 32, 560))
    if c["m"] * c["n"] > 17920 * 6656:           # one large layer at most
        c["m"] = 32 * max(1, 17920 * 6656 // c["n"] // 32)
    n, size = c["n"], c["m"] * c["n"]             # full rows and columns where the rate leaves room for them
    if (c["structure"] == "cols64" and 64 > c["rate"] * n) or (c["structure"] == "rows8cols4" and
                                                               8 * n + 4 * c["m"] > c["rate"] * size):
        c["structure"] = "uniform"
    if kind == "gemv":
        c.update(layout=rng.choice([1, 1, 2, 3]), perm=rng.choice([False, True]))
    elif kind == "prompt":
        c.update(kind="batch", b=rng.randint(17, 256), perm=rng.choice([False, True]))
    elif kind == "batch":
        c.update(b=rng.randint(2, 16))
    else:
        c.update(m=max(32, c["m"] // 64 * 32), count=2, b=rng.randint(2, 256))
    return c


# ---------------------------------------------------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------------------------------------------------
def _generator(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * seed + salt)
    return g


class _Layout:
    """Geometry of a packed buffer (include/spqr.h, spqr_matrix_t)."""

    def __init__(self, m, n, case):
        self.w, self.axis, self.layout, b1, b2 = case["w"], case["axis"], case["layout"], case["beta1"], case["beta2"]
        self.tr, self.tc = (b2, b1) if self.axis == 0 else (b1, b2)
        self.beta2 = b2
        self.ntr, self.ntc = m // self.tr, n // self.tc
        self.kw = self.tr * self.tc * self.w // 128
        self.nc = 3 * b2 // 16
        self.sd = {1: self.nc + 2, 2: self.nc + 1, 3: b2}[self.layout]
        self.tile_dwords = 4 * self.kw + self.sd

    def blocks(self, rows):
        """The interleaved runs of up to 64 tiles of `rows` (a [r, ntc * tile_dwords] view): (run, tiles)."""
        for t0 in range(0, self.ntc, 64):
            tiles = min(64, self.ntc - t0)
            yield rows[:, t0 * self.tile_dwords:(t0 + tiles) * self.tile_dwords], t0, tiles

    def stat(self, run, tiles, d):
        """View of statistic dword d of the run's tiles: [r, tiles]."""
        at, swf = 4 * self.kw * tiles, self.sd // 4
        if d < 4 * swf:
            return run[:, at + (d // 4) * tiles * 4:at + (d // 4 + 1) * tiles * 4].unflatten(1, (tiles, 4))[:, :, d % 4]
        at += 4 * swf * tiles + (d - 4 * swf) * tiles
        return run[:, at:at + tiles]

    def codes(self, run, tiles):
        """Code dwords of the run's tiles: [r, tiles, 4 * kw]."""
        return run[:, :4 * self.kw * tiles].unflatten(1, (self.kw, tiles, 4)).transpose(1, 2).flatten(2)


def _f16_pairs(lo, hi):
    """Two float tensors -> int32 dwords with binary16(lo) in the low half."""
    return torch.stack([lo.to(torch.float16), hi.to(torch.float16)], dim=-1).view(torch.int32).squeeze(-1)


@functools.lru_cache(maxsize=64)
def _zipf_counts(m, n, total):
    """Outliers per row, Zipf(1.2) over the rows with what exceeds a row handed down."""
    weights = np.arange(1, m + 1, dtype=np.float64) ** -1.2
    share = weights / np.cumsum(weights[::-1])[::-1]
    counts, left = np.zeros(m), total
    for k in range(m):
        counts[k] = max(0, min(n, int(round(left * share[k])), left))
        left -= counts[k]
    return counts


def _outliers(m, n, rate, structure, g):
    """row_ptr, col_idx, val, longest row."""
    total = int(round(rate * m * n))
    p = torch.full((m, 1), rate, device="cuda")
    rows = torch.randperm(m, generator=g, device="cuda")
    cols = torch.randperm(n, generator=g, device="cuda")
    nrows, ncols = {"rows8cols4": (8, 4), "cols64": (0, 64)}.get(structure, (0, 0))
    if structure == "zipf":
        p[rows, 0] = torch.from_numpy(_zipf_counts(m, n, total) / n).float().cuda()
    elif nrows or ncols:
        p.fill_(max(0.0, (total - nrows * n - ncols * m) / (m * n)))
    mask = torch.rand((m, n), generator=g, device="cuda") < p
    mask[rows[:nrows]] = True
    mask[:, cols[:ncols]] = True
    counts = mask.sum(1)
    row_ptr = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = counts.cumsum(0)
    col = mask.nonzero()[:, 1].to(torch.int16).contiguous()
    val = (0.2 * torch.randn(col.numel(), generator=g, device="cuda")).to(torch.float16)
    return row_ptr, col, val, int(counts.max().item())


def _matrix(m, n, case, seed, salt):
    g = _generator(seed, salt)
    lay = _Layout(m, n, case)
    packed = torch.randint(-2 ** 31, 2 ** 31, (lay.ntr, lay.ntc * lay.tile_dwords), generator=g, device="cuda",
                           dtype=torch.int64).to(torch.int32)

    def uniform(lo, hi, shape):
        return lo + (hi - lo) * torch.rand(shape, generator=g, device="cuda")

    for run, _, tiles in lay.blocks(packed):
        shape = (lay.ntr, tiles)
        if lay.layout == 3:
            for d in range(lay.sd):
                lay.stat(run, tiles, d).copy_(_f16_pairs(uniform(0.02, 0.2, shape), uniform(0.0, 2 ** lay.w - 1.0, shape)))
        else:
            for d in range(lay.nc, lay.sd):
                lay.stat(run, tiles, d).copy_(_f16_pairs(uniform(0.01, 0.05, shape), uniform(2.0, 5.0, shape)))
    row_ptr, col, val, longest = _outliers(m, n, case["rate"], case["structure"], g)
    perm = torch.randperm(n, generator=g, device="cuda").to(torch.int32) if case["perm"] else None
    bits = 16 if lay.layout == 3 else 3
    return P.SpQRMatrix(m, n, lay.w, case["beta1"], case["beta2"], lay.axis, packed.view(torch.uint8).flatten(), row_ptr, col,
                        val, perm, bits, bits, lay.layout, longest)


def _shapes(case):
    if case["kind"] == "block":
        return _block(case["n"], case["m"])
    return [(case["m"], case["n"])] * case.get("count", 1)


def prepare(case, seed):
    if case["kind"] == "factor":
        n, d, g = case["n"], case["d"], _generator(seed, 1)
        X = torch.randn((n, d), generator=g, device="cuda", dtype=torch.float64)
        common = torch.randn((8, d), generator=g, device="cuda", dtype=torch.float64)      # correlated inputs
        mix = torch.randn((n, 8), generator=g, device="cuda", dtype=torch.float64) * 0.3
        for k in range(8):
            X += mix[:, k:k + 1] * common[k]
        need = int(P.load_library().spqr_inverse_cholesky_workspace_bytes(n)) if _typed() else 0
        return dict(X=X, lam=0.01 * 2 * d, ws=torch.empty(need, dtype=torch.uint8, device="cuda"))
    if case["kind"] == "quantize":
        m, n, g = case["m"], case["n"], _generator(seed, 2)
        W = 0.05 * torch.randn((m, n), generator=g, device="cuda", dtype=torch.float64)
        W[torch.rand((m, n), generator=g, device="cuda") < 0.02] *= 6.0
        # an upper factor as the calibration inputs of a layer give it: diagonal of a narrow range, small entries right
        # of it
        diag = 0.01 * (0.5 + torch.rand((n, 1), generator=g, device="cuda", dtype=torch.float64))
        U = torch.randn((n, n), generator=g, device="cuda", dtype=torch.float64) * (0.3 / math.sqrt(n))
        U = (diag * (U.triu(1) + torch.eye(n, device="cuda", dtype=torch.float64))).contiguous()
        ng, nt = n // case["beta1"], m // case["beta2"]
        u8, f16 = dict(dtype=torch.uint8, device="cuda"), dict(dtype=torch.float16, device="cuda")
        out = dict(Q=torch.empty((m, n), **u8), s_q=torch.empty((m, ng), **u8), z_q=torch.empty((m, ng), **u8),
                   s_s=torch.empty((nt, ng), **f16), z_s=torch.empty((nt, ng), **f16), s_z=torch.empty((nt, ng), **f16),
                   z_z=torch.empty((nt, ng), **f16), outlier_mask=torch.empty((m, n), **u8),
                   outlier_val=torch.empty((m, n), **f16), row_ptr=torch.empty(m + 1, dtype=torch.int32, device="cuda"),
                   W_final=torch.empty((m, n), dtype=torch.float64, device="cuda"))
        _typed()
        ws = torch.empty(max(256, int(P.load_library().spqr_quantize_workspace_bytes(m, n))), dtype=torch.uint8, device="cuda")
        return dict(W=W, U=U, out=out, ws=ws, case=case)
    shapes, b = _shapes(case), case["b"]
    As = [_matrix(m, n, case, seed, 10 + i) for i, (m, n) in enumerate(shapes)]
    if len(As) > 1 and case["perm"]:             # matrices that share an input share its order
        raise ValueError("several matrices: no permutation")
    g = _generator(seed, 3)
    xs = [torch.randn((b, n), generator=g, device="cuda").to(torch.float16)
          for _, n in (shapes if case["kind"] == "block" else shapes[:1])]
    ydt = torch.float16 if case["f16"] else torch.float32
    ys = [torch.empty((b, m), dtype=ydt, device="cuda") for m, _ in shapes]
    st = dict(kind=case["kind"], As=As, xs=xs, ys=ys, ydt=P.SPQR_F16 if case["f16"] else P.SPQR_F32, case=case)
    if case["kind"] == "fused":
        st["ws"] = torch.empty(max(256, P.spqr_workspace_bytes(As, b)), dtype=torch.uint8, device="cuda")
    return st


@functools.lru_cache(maxsize=1)
def _typed():
    """Declares the quantiser's entry points on the loaded library."""
    E._lib()
    return True


def run(state):
    if "lam" in state:
        H = E.spqr_hessian(state["X"])
        return H, E.spqr_inverse_cholesky(H, state["lam"], state["ws"])
    if "U" in state:
        c, out = state["case"], state["out"]
        E.spqr_quantize_device(state["W"], state["U"], c["w"], c["beta1"], c["beta2"], c["tau"], workspace=state["ws"], outputs=out)
        return {k: v for k, v in out.items() if k != "workspace"}
    As, xs, ys, ydt = state["As"], state["xs"], state["ys"], state["ydt"]
    if state["kind"] == "gemv":
        return P.spqr_gemv(As[0], xs[0].view(-1), out=ys[0].view(-1), y_dtype=ydt)
    if state["kind"] == "block":
        return P.spqr_gemv_grouped(As, [x.view(-1) for x in xs], outs=ys, y_dtype=ydt)
    if state["kind"] == "batch":
        return P.spqr_gemm_smallbatch(As[0], xs[0], out=ys[0], y_dtype=ydt)
    return P.spqr_gemm_fused_ws(As, xs[0], state["ws"], outs=ys, y_dtype=ydt)


def work(case):
    if case["kind"] == "factor":
        n, d = case["n"], case["d"]
        # one triangle of X X^T, a Cholesky factorisation and a triangular inverse of n^3 / 3 multiply-adds each way
        return {"bytes": 8 * (n * d + 2 * n * n), "flops": n * (n + 1) * d + 2 * n ** 3 / 3}
    if case["kind"] == "quantize":
        m, n, b1 = case["m"], case["n"], case["beta1"]
        outputs = m * n * (1 + 1 + 2 + 8) + m * n // b1 * 2 + 8 * m * n // (b1 * case["beta2"]) + 4 * (m + 1)
        return {"bytes": 8 * m * n + 4 * n * n + outputs, "flops": m * n * n + 20 * m * n * b1}
    b, total, flops = case["b"], 0, 0
    shared = case["kind"] != "block"
    for i, (m, n) in enumerate(_shapes(case)):
        lay = _Layout(m, n, case)
        total += 4 * lay.ntr * lay.ntc * lay.tile_dwords + 4 * round(case["rate"] * m * n) + 4 * (m + 1)
        total += (2 * b * n if i == 0 or not shared else 0) + (2 if case["f16"] else 4) * b * m + (4 * n if case["perm"] else 0)
        flops += 2 * m * n * b
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"                           # binary64 steps in a stated order: bit for bit
    if case["kind"] == "factor":
        return {"rel": 2e-12}                    # binary64 sums in any order; the factor measured 4e-13 from exact()
    # binary16 weights or products s*x, binary32 sums: 2.1e-4 measured from exact(), 2.9e-4 with 16-bit outputs
    return {"rel": 1e-3, "max": 6e-3}


# ---------------------------------------------------------------------------------------------------------------------
# The same results from plain torch / numpy in 64 bits.
# ---------------------------------------------------------------------------------------------------------------------
def _pairs(dw, bits):
    """[..., D] dwords -> [..., 2 * pairs] codes, low half first."""
    dw = dw.to(torch.int32)

    def half(off):
        if bits == 4:
            sh = torch.arange(0, 16, 4, device=dw.device, dtype=torch.int32) + off
            return ((dw[..., None] >> sh) & 15).flatten(-2)
        t = dw.unflatten(-1, (-1, 3))
        sh = torch.arange(0, 15, 3, device=dw.device, dtype=torch.int32) + off
        first = ((t[..., None] >> sh) & 7).flatten(-2)
        last = sum(((t[..., i] >> (15 + off)) & 1) << i for i in range(3))
        return torch.cat([first, last[..., None]], dim=-1).flatten(-2)

    return torch.stack([half(0), half(16)], dim=-1).flatten(-2)


def _halves(dw):
    h = dw.contiguous().view(torch.float16).unflatten(-1, (-1, 2)).double()
    return h[..., 0], h[..., 1]


def _dense64(A, case):
    """The stored matrix, outliers added, in binary64."""
    lay = _Layout(A.m, A.n, case)
    packed = A.packed.view(torch.int32).view(lay.ntr, -1)
    W = torch.empty((A.m, A.n), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 24) // (lay.tr * A.n))
    for r0 in range(0, lay.ntr, step):
        rows = packed[r0:r0 + step]
        r = rows.shape[0]
        for run, t0, tiles in lay.blocks(rows):
            q = _pairs(lay.codes(run, tiles), lay.w).double().unflatten(-1, (lay.tr, lay.tc))
            st = torch.stack([lay.stat(run, tiles, d) for d in range(lay.sd)], dim=-1)
            if lay.layout == 3:
                s, z = _halves(st)
            else:
                c = _pairs(st[..., :lay.nc], 3).double()
                s_s, z_s = _halves(st[..., lay.nc])
                s = s_s[..., None] * (c[..., :lay.beta2] - z_s[..., None])
                z = c[..., lay.beta2:]
                if lay.layout == 1:
                    s_z, z_z = _halves(st[..., lay.nc + 1])
                    z = s_z[..., None] * (z - z_z[..., None])
            s, z = (s[..., None], z[..., None]) if lay.axis == 0 else (s[..., None, :], z[..., None, :])
            w = (s * (q - z)).permute(0, 2, 1, 3).reshape(r * lay.tr, tiles * lay.tc)
            W[r0 * lay.tr:(r0 + r) * lay.tr, t0 * lay.tc:(t0 + tiles) * lay.tc] = w
    row = torch.repeat_interleave(torch.arange(A.m, device="cuda"), A.row_ptr.diff().long())
    W.view(-1).index_add_(0, row * A.n + A.col_idx.long(), A.val.double())
    return W


def exact(case, seed):
    if case["kind"] == "quantize":
        return None                              # integers and binary64 values that are compared bit for bit
    st = prepare(case, seed)
    if case["kind"] == "factor":
        # X in three parts of 20 bits and less, so that the large products and their sums are exact
        X, n = st["X"], case["n"]
        X1 = torch.round(X * 2.0 ** 17) / 2.0 ** 17
        X2 = torch.round((X - X1) * 2.0 ** 37) / 2.0 ** 37
        X3 = X - X1 - X2
        a, c = X1 @ X2.T, X1 @ X3.T
        H = 2.0 * (X1 @ X1.T + ((a + a.T) + (X2 @ X2.T + (c + c.T))))
        R = H.cpu().numpy()[::-1, ::-1] + st["lam"] * np.eye(n)
        U = np.linalg.inv(np.linalg.cholesky(R))[::-1, ::-1]
        return H, torch.from_numpy(np.ascontiguousarray(np.triu(U)))
    out = []
    for i, A in enumerate(st["As"]):
        x = st["xs"][i if case["kind"] == "block" else 0].double()
        if A.perm is not None:
            x = x[:, A.perm.long()]
        out.append(x @ _dense64(A, case).T)
    if case["kind"] == "gemv":
        return out[0].view(-1)
    return out[0] if case["kind"] == "batch" else out
