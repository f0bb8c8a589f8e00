"""GPU tests of the one-pass product of prompt-sized batches and of the batch kernel's edges (ragged groups of strips, units
and blocks of vectors, outliers beyond what a thread has in flight, every split pinned; against the oracle), of the
permutation at batch 1, and of the quantiser's two ways of sharing out rows (against each other, bit for bit)."""
import numpy as np
import pytest

import spqr_synth as synth
from oracle import spqr_oracle as orc

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(600)]

# Weights rounded once to binary16, weights with an outlier twice: 2^-11 / sqrt(3) of a term at most in the mean square,
# 2.8e-4 and 4.0e-4, of the root of the sum of a row's squared terms (measured 2.2e-4 on average, 3.7e-4 at most).  Against
# the result itself, whose terms may cancel, the nearest binary16 weights give 1.007e-3 at 16 rows (3-bit, 8 x 32, 129 vectors).
REL_L2 = 1e-3


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_2306_03078_amd as P
    P.load_library()
    assert torch.cuda.is_available()
    return P


def run(P, f, b, steps=0, shares=0, prompt=0):
    import torch
    A = P.SpQRMatrix.from_logical(f)
    X = synth.make_x(f.n, b, seed=(71, b))
    P.spqr_set_option(P.SPQR_OPT_BATCH_STEPS, steps)
    P.spqr_set_option(P.SPQR_OPT_BATCH_SHARES, shares)
    P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, prompt)
    try:
        need = P.spqr_workspace_bytes(A, b)
        buf = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device="cuda:0")
        Y = P.spqr_gemm_smallbatch_ws(A, torch.from_numpy(X).to("cuda:0"), buf[256:256 + need])
        again = P.spqr_gemm_smallbatch_ws(A, torch.from_numpy(X).to("cuda:0"), buf[256:256 + need])
        assert torch.equal(Y, again)
        assert bool((buf[:256] == 0xA5).all()) and bool((buf[256 + need:] == 0xA5).all())
    finally:
        P.spqr_set_option(P.SPQR_OPT_BATCH_STEPS, 0)
        P.spqr_set_option(P.SPQR_OPT_BATCH_SHARES, 0)
        P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 0)
    ref = orc.matvec(f, X)
    Xp = X.astype(np.float64) if f.perm is None else X.astype(np.float64)[:, f.perm]
    terms = np.sqrt(Xp ** 2 @ (orc.reconstruct(f) ** 2).T)
    got = Y.cpu().numpy().astype(np.float64)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(terms, axis=1)
    assert err.max() <= REL_L2, (int(err.argmax()), float(err.max()))


# strips: one, 16 k + 1, a full group; tile columns: one, a unit and one, many units
@pytest.mark.parametrize("w,b1,b2,axis,ntr,ntc,structure,rate", [
    (3, 16, 16, 1, 1, 1, "uniform", 0.1), (4, 16, 16, 1, 17, 17, "zipf", 0.1), (3, 16, 16, 0, 16, 67, "rows8cols4", 0.2),
    (4, 8, 32, 1, 33, 65, "cols64", 0.2), (3, 8, 32, 0, 9, 131, "uniform", 0.24), (3, 8, 32, 1, 2, 160, "uniform", 0.2)])
# prompts with the plan pinned: at this size the library's own choice is the dense copy, which has tests of its own
@pytest.mark.parametrize("b,steps", [(4, 0), (4, 1), (4, 1000), (16, 0), (16, 1), (16, 1000)] +
                         [(b, s) for b in (49, 65, 129, 256) for s in (1, 3, 1000)])
def test_edges(P, w, b1, b2, axis, ntr, ntc, structure, rate, b, steps):
    tr, tc = synth.tile_shape(b1, b2, axis)
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX if b <= 16 else P.SPQR_BATCH_PATH_AUTO)
    try:
        f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=rate,
                              outlier_structure=structure, seed=(72, w, axis, ntr, ntc))
        if (ntr + b) % 2:
            f.perm = np.random.default_rng(5).permutation(f.n).astype(np.int32)
        run(P, f, b, steps if b <= 16 else 0, prompt=steps if b > 16 else 0)
    finally:
        P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_AUTO)


# ragged groups of strips, last units and blocks of vectors at every number of vectors a workgroup takes
@pytest.mark.parametrize("w,b1,b2,axis,ntr,ntc,structure,rate", [
    (3, 16, 16, 1, 17, 67, "rows8cols4", 0.2), (4, 16, 16, 0, 3, 18, "none", 0.0), (4, 8, 32, 1, 33, 35, "cols64", 0.24),
    (3, 8, 32, 1, 18, 17, "none", 0.0), (3, 8, 32, 0, 9, 67, "zipf", 0.1)])
@pytest.mark.parametrize("vectors", [1, 2, 4])
@pytest.mark.parametrize("b,units", [(48, 0), (65, 1), (77, 3), (129, 1000), (255, 2)])
def test_every_width_of_the_one_pass_kernel(P, w, b1, b2, axis, ntr, ntc, structure, rate, vectors, b, units):
    tr, tc = synth.tile_shape(b1, b2, axis)
    f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=rate,
                          outlier_structure=structure, seed=(81, w, axis, ntr, ntc))
    if (ntr + b) % 2:
        f.perm = np.random.default_rng(5).permutation(f.n).astype(np.int32)
    run(P, f, b, prompt=1024 * vectors + units)


def test_two_blocks_of_vectors_by_itself(P):
    """8-row strips and 200 vectors, nothing pinned: 172 groups of 2 units, two blocks of 128 vectors, runs of 3 units from one
    group into the next, the last rows and columns ragged."""
    f = synth.make_matrix(8 * 2751, 32 * 19, w_bits=3, beta1=8, beta2=32, group_axis=1, outlier_rate=0.02,
                          outlier_structure="cols64", seed=(82,))
    run(P, f, 200)


def test_permutation_wider_than_the_room_of_the_products(P):
    """Batch 1 and 2 with a permutation: x through LDS where the products leave it room, gathered from memory where not."""
    import torch
    for w, b1, b2, axis, ntr, ntc in ((3, 8, 32, 0, 3, 300), (3, 16, 16, 1, 5, 3000), (4, 16, 16, 0, 4, 67)):
        tr, tc = synth.tile_shape(b1, b2, axis)
        f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=0.01, seed=(73, ntc))
        f.perm = np.random.default_rng(6).permutation(f.n).astype(np.int32)
        A = P.SpQRMatrix.from_logical(f)
        for b in (1, 2):
            X = synth.make_x(f.n, b, seed=(74, b))
            got = P.spqr_gemm_smallbatch(A, torch.from_numpy(X).to("cuda:0")).cpu().numpy().astype(np.float64)
            ref = orc.matvec(f, X)
            assert (np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)).max() <= REL_L2


def test_sweep_is_the_same_on_both_row_splits(P):
    """Rows are independent outside their tile: the first rows of a layer so tall that it takes 64 rows per workgroup come out bit
    for bit as when they are a layer of their own, which takes 16 rows per workgroup."""
    import torch
    import paper_2306_03078_amd.encode_binding as E
    for b1, b2, n, m, tau in ((16, 16, 160, 12304, float("inf")), (8, 2, 72, 12304, 5.0), (32, 8, 128, 8208, float("inf")), (4, 16, 68, 8208, 5.0)):
        rows_of = lambda rows: E._lib().spqr_sweep_rows(rows, n, b1, b2, int(tau < float("inf")))
        assert rows_of(m) == 64 and rows_of(4096) == rows_of(48) == 16
        W, _ = synth.make_quantizer_problem(7, m, n, 8)
        rng = np.random.default_rng(8)
        U = np.triu(rng.normal(size=(n, n)) * 0.02, 1) + np.diag(0.01 + 0.01 * rng.random(n))
        Wd, Ud = torch.from_numpy(W).to("cuda:0"), torch.from_numpy(U).to("cuda:0")
        tall = E.spqr_quantize_device(Wd, Ud, 3, b1, b2, tau)
        for rows in (4096, 48):
            own = E.spqr_quantize_device(Wd[:rows].contiguous(), Ud, 3, b1, b2, tau)
            for k in ("Q", "s_q", "z_q", "outlier_mask"):
                assert torch.equal(own[k], tall[k][:rows]), k
            for k in ("s_s", "z_s", "s_z", "z_z"):
                assert torch.equal(own[k].view(torch.int16), tall[k][:rows // b2].view(torch.int16)), k
            assert torch.equal(own["outlier_val"].view(torch.int16), tall["outlier_val"][:rows].view(torch.int16))
            assert torch.equal(own["W_final"].view(torch.int64), tall["W_final"][:rows].view(torch.int64))
            assert torch.equal(own["row_ptr"], tall["row_ptr"][:rows + 1])
        # without W_final the workspace is the working copy
        none = E.spqr_quantize_device(Wd[:48].contiguous(), Ud, 3, b1, b2, tau, want_final=False)
        assert torch.equal(none["Q"], tall["Q"][:48])


# 16 vectors: the slices; 64: the one-pass kernel (the split pinned)
@pytest.mark.parametrize("w,b1,b2,axis", [(3, 16, 16, 1), (4, 16, 16, 1), (3, 8, 32, 1), (4, 8, 32, 1), (3, 16, 16, 0), (4, 8, 32, 0)])
@pytest.mark.parametrize("b", [16, 64])
def test_weights_are_rounded_from_an_exact_code(P, w, b1, b2, axis, b):
    """A batch of unit vectors returns columns of the matrix as the matrix cores see it: binary16 numbers.  The binary32
    arithmetic before that rounding may move a weight by about 2 units of 2^-24 of its largest term, s_hat * 2^W, and turns
    a rounding only where the exact weight lies that close to the middle of two binary16 numbers: under 1 % of the weights
    (measured 0 with groups along the columns, 0.3 % along the rows; 8 to 11 % with an offset of 128 in the code)."""
    import torch
    tr, tc = synth.tile_shape(b1, b2, axis)
    f = synth.make_matrix(64 * tr, 16 * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_structure="none", seed=(75, w, axis, b1))
    cols = np.random.default_rng(9).permutation(f.n)[:b]
    X = np.zeros((b, f.n), np.float16)
    X[np.arange(b), cols] = 1
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX if b <= 16 else P.SPQR_BATCH_PATH_AUTO)
    P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 1000)
    got = P.spqr_gemm_smallbatch(P.SpQRMatrix.from_logical(f), torch.from_numpy(X.view(np.float16)).to("cuda:0")).cpu().numpy()
    want = orc.decode_dense(f)[:, cols].T.astype(np.float16)
    assert np.array_equal(got, got.astype(np.float16).astype(np.float32))
    assert (got != want.astype(np.float32)).mean() <= 0.01


@pytest.mark.parametrize("w,b1,b2,axis,structure", [(3, 16, 16, 1, "uniform"), (4, 16, 16, 0, "rows8cols4"), (3, 8, 32, 1, "zipf"), (4, 8, 32, 0, "cols64")])
@pytest.mark.parametrize("b", [4, 16, 64])
def test_an_infinite_activation_meets_only_its_own_columns_weights(P, w, b1, b2, axis, structure, b):
    """One infinite activation per vector (NaN in the last vector): every row whose weight there is not zero gives the
    infinity of the product's sign, whatever the outliers of the rows next to it.  (Not compared: a row with an outlier
    there.  Slices add w * inf and value * inf, which may be of opposite signs.)"""
    import torch
    tr, tc = synth.tile_shape(b1, b2, axis)
    m, n = 33 * 32, 1664
    f = synth.make_matrix(m, n, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=0.1, outlier_structure=structure, seed=(76, w, axis))
    rng = np.random.default_rng(10)
    X = synth.make_x(n, b, seed=(77, b))
    at = rng.permutation(n)[:b]
    X[np.arange(b), at] = np.where(np.arange(b) % 2 == 0, np.float16(np.inf), np.float16(-np.inf))
    X[b - 1, at[b - 1]] = np.nan
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX if b <= 16 else P.SPQR_BATCH_PATH_AUTO)
    P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 1000)
    got = P.spqr_gemm_smallbatch(P.SpQRMatrix.from_logical(f), torch.from_numpy(X).to("cuda:0")).cpu().numpy()
    weight = orc.reconstruct(f)[:, at].T                      # the weight each infinity meets, [b, m]
    sure = (np.abs(weight) > 1e-6) & (weight == orc.decode_dense(f)[:, at].T)   # not a zero in binary16, no outlier
    assert sure.mean() > 0.7
    assert np.isnan(got[b - 1]).all()
    want = np.copysign(np.inf, weight * np.where(np.arange(b) % 2 == 0, 1.0, -1.0)[:, None])
    ok = (got == want) | ~sure
    ok[b - 1] = True
    assert ok.all(), np.argwhere(~ok)[:5]


# strips: one, 16 k + 1, ragged; units: one, a piece of XT and one more, many; rows beyond what a wavefront takes at once
@pytest.mark.parametrize("w,b1,b2,axis,ntr,ntc,structure,rate", [
    (3, 16, 16, 1, 1, 1, "uniform", 0.1), (4, 16, 16, 1, 19, 113, "zipf", 0.1), (3, 16, 16, 0, 33, 65, "rows8cols4", 0.2),
    (4, 8, 32, 1, 33, 65, "cols64", 0.2), (3, 8, 32, 0, 9, 211, "zipf", 0.05), (3, 8, 32, 1, 2, 160, "uniform", 0.2)])
@pytest.mark.parametrize("shares", [1, 2, 3, 5])
@pytest.mark.parametrize("b,steps", [(4, 1), (16, 1), (16, 7), (11, 1000)])
def test_outliers_beside_the_dense_workgroups(P, w, b1, b2, axis, ntr, ntc, structure, rate, shares, b, steps):
    tr, tc = synth.tile_shape(b1, b2, axis)
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX)
    f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=rate,
                          outlier_structure=structure, seed=(78, w, axis, ntr, ntc))
    if (ntr + b) % 2:
        f.perm = np.random.default_rng(5).permutation(f.n).astype(np.int32)
    run(P, f, b, steps, shares)


@pytest.mark.parametrize("shares", [0, 1, 2, 5])
def test_outliers_beside_the_dense_workgroups_of_several_matrices(P, shares):
    """One of the matrices without outliers, one shorter than a group of strips."""
    import torch
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX)
    P.spqr_set_option(P.SPQR_OPT_BATCH_SHARES, shares)
    fs = [synth.make_matrix(m, 1616, w_bits=4, beta1=16, beta2=16, group_axis=1, outlier_rate=0.05, outlier_structure=st, seed=(79, m))
          for m, st in ((528, "zipf"), (48, "none"), (256, "uniform"))]
    X = synth.make_x(1616, 13, seed=(80,))
    Ys = P.spqr_gemm_fused([P.SpQRMatrix.from_logical(f) for f in fs], torch.from_numpy(X).to("cuda:0"))
    for f, Y in zip(fs, Ys):
        ref = orc.matvec(f, X)
        err = np.linalg.norm(Y.cpu().numpy().astype(np.float64) - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= REL_L2


def _one_pass_layer(P, b, perm):
    """A layer and batch the library gives to the one-pass kernel by itself: its scratch holds no dense copy."""
    f = synth.make_matrix(2056, 2080, w_bits=3, beta1=8, beta2=32, group_axis=1, outlier_rate=0.02, outlier_structure="zipf", seed=(83,))
    if perm:
        f.perm = np.random.default_rng(6).permutation(f.n).astype(np.int32)
    A = P.SpQRMatrix.from_logical(f)
    need = P.spqr_workspace_bytes(A, b)
    assert 0 < need < 2 * f.m * f.n
    return f, A, synth.make_x(f.n, b, seed=(84, b)), need


@pytest.mark.parametrize("perm", [False, True])
def test_one_pass_with_a_workspace_under_capture(P, perm):
    """Kernel nodes only, and every replay gives the eager result bit for bit, with eager work in the same workspace and
    another batch in the input between the replays."""
    import ctypes as C
    import torch
    from test_gpu_workspace import _graph_node_types
    f, A, X, need = _one_pass_layer(P, 77, perm)
    Xd = torch.from_numpy(X).to("cuda:0")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    eager = P.spqr_gemm_smallbatch_ws(A, Xd, ws).clone()
    turned = P.spqr_gemm_smallbatch_ws(A, Xd.flip(0).contiguous(), ws).clone()
    run(P, f, 77)                                            # the same path against the oracle
    Xg, Y = Xd.clone(), torch.zeros_like(eager)
    torch.cuda.synchronize()
    types, ex, graph, st, hip = _graph_node_types(lambda s: P.spqr_gemm_smallbatch_ws(A, Xg, ws, out=Y, stream=s))
    assert len(types) == (5 if perm else 4) and all(t == 0 for t in types), types       # (gather,) count, sort, product, sums
    for rep in range(4):
        Xg.copy_(Xd if rep % 2 == 0 else Xd.flip(0))
        Y.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(ex, C.c_void_p(st.cuda_stream)) == 0
        torch.cuda.synchronize()
        assert torch.equal(Y, eager if rep % 2 == 0 else turned), rep
        ws.fill_(0xA5)
        P.spqr_gemm_smallbatch_ws(A, Xd, ws)
        torch.cuda.synchronize()
    assert hip.hipGraphExecDestroy(ex) == 0 and hip.hipGraphDestroy(graph) == 0


def test_one_pass_scratch_limits_and_the_static_array(P):
    """One byte too little: the slices of 16, bit for bit what they give when asked for; the entry that allocates nothing
    and the one with the library's scratch: the one-pass result."""
    import torch
    b = 64
    f, A, X, need = _one_pass_layer(P, b, True)
    Xd = torch.from_numpy(X).to("cuda:0")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    one = P.spqr_gemm_smallbatch_ws(A, Xd, ws).clone()
    run(P, f, b)
    few = P.spqr_gemm_smallbatch_ws(A, Xd, ws[:need - 1]).clone()
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX)
    try:
        small = P.spqr_workspace_bytes(A, b)
        assert 0 < small < need
        slices = P.spqr_gemm_smallbatch_ws(A, Xd, ws[:small]).clone()
    finally:
        P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_AUTO)
    assert torch.equal(few, slices) and not torch.equal(few, one)
    assert torch.equal(P.spqr_gemm_smallbatch_ws(A, Xd, ws[:small]), slices)
    assert need <= P.SPQR_STATIC_SCRATCH_BYTES
    out = torch.zeros_like(one)
    P.spqr_gemm_smallbatch_noalloc(A, Xd, out)
    assert torch.equal(out, one)
    assert torch.equal(P.spqr_gemm_smallbatch(A, Xd), one)
    half = torch.zeros((b, f.m), dtype=torch.float16, device="cuda:0")
    P.spqr_gemm_smallbatch_noalloc(A, Xd, half, y_dtype=P.SPQR_F16)
    assert torch.equal(half, one.to(torch.float16))


# rows of up to 64 entries inside a piece of 1536 columns are taken by 4 lanes each, longer ones by a whole wavefront
@pytest.mark.parametrize("w,b1,b2,axis,ntr", [(3, 16, 16, 1, 20), (4, 8, 32, 1, 40), (3, 8, 32, 0, 10)])
@pytest.mark.parametrize("b", [5, 16])
@pytest.mark.parametrize("steps,shares", [(1, 0), (1000, 0), (1, 3), (1000, 1)])
def test_rows_around_what_counts_as_long_in_a_piece(P, w, b1, b2, axis, ntr, b, steps, shares):
    tr, tc = synth.tile_shape(b1, b2, axis)
    f = synth.make_matrix(ntr * tr, 4096, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_structure="none", seed=(85, w, axis))
    rng = np.random.default_rng(86)
    cols = {}
    for r, (first, second) in {0: (63, 0), 1: (64, 0), 2: (65, 0), 3: (64, 64), 4: (65, 64), 5: (0, 65), 17: (1, 129), 40: (128, 63),
                               41: (127, 0), 42: (1536, 0), 43: (1535, 1), 100: (66, 66), 255: (64, 65), 256: (65, 0), 319: (2, 64)}.items():
        # so many entries in the columns 0 .. 1535 and 1536 .. 3071, a few behind them
        cols[r] = np.concatenate([np.sort(rng.choice(1536, first, replace=False)), 1536 + np.sort(rng.choice(1536, second, replace=False)),
                                  3072 + np.sort(rng.choice(1024, r % 3, replace=False))])
    for r in range(6, 320, 5):
        cols.setdefault(r, np.sort(rng.choice(4096, 3, replace=False)))
    counts = np.zeros(f.m, np.int64)
    for r, c in cols.items():
        counts[r] = len(c)
    f.row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    f.col_idx = np.concatenate([cols[r] for r in sorted(cols)]).astype(np.uint16)
    f.val = rng.standard_normal(len(f.col_idx)).astype(np.float16)
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX)
    try:
        run(P, f, b, steps, shares)
    finally:
        P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_AUTO)


# runs of units that end inside a group, at its end and behind several groups and matrices; one matrix without outliers, one
# shorter than a group
@pytest.mark.parametrize("w,b1,b2,axis,ntc", [(3, 16, 16, 1, 35), (4, 16, 16, 0, 18), (4, 8, 32, 1, 33), (3, 8, 32, 0, 67)])
@pytest.mark.parametrize("b,vectors,units", [(48, 1, 1), (65, 2, 5), (130, 4, 1000), (256, 4, 3), (77, 0, 2)])
def test_one_pass_of_several_matrices(P, w, b1, b2, axis, ntc, b, vectors, units):
    """Against the oracle; twice the same; nothing written outside the workspace; on a capturing stream matrix by matrix, bit
    for bit what the single calls give."""
    import ctypes as C
    import torch
    from test_gpu_workspace import _graph_node_types
    tr, tc = synth.tile_shape(b1, b2, axis)
    fs = [synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=rate,
                            outlier_structure=st, seed=(87, w, axis, ntr)) for ntr, st, rate in ((33, "zipf", 0.1), (2, "none", 0.0), (17, "rows8cols4", 0.2))]
    if b % 2:
        for f in fs:
            f.perm = np.random.default_rng(5).permutation(f.n).astype(np.int32)
    As = [P.SpQRMatrix.from_logical(f) for f in fs]
    for A in As[1:]:
        A.desc.perm = As[0].desc.perm          # descriptors must name the same device permutation
    X = synth.make_x(fs[0].n, b, seed=(88, b))
    Xd = torch.from_numpy(X).to("cuda:0")
    P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 1024 * vectors + units)
    need = P.spqr_workspace_bytes(As, b)
    buf = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device="cuda:0")
    Ys = P.spqr_gemm_fused_ws(As, Xd, buf[256:256 + need])
    again = P.spqr_gemm_fused_ws(As, Xd, buf[256:256 + need])
    assert bool((buf[:256] == 0xA5).all()) and bool((buf[256 + need:] == 0xA5).all())
    for f, Y, Z in zip(fs, Ys, again):
        assert torch.equal(Y, Z)
        Xp = X.astype(np.float64) if f.perm is None else X.astype(np.float64)[:, f.perm]
        terms = np.sqrt(Xp ** 2 @ (orc.reconstruct(f) ** 2).T)
        err = np.linalg.norm(Y.cpu().numpy() - orc.matvec(f, X), axis=1) / np.linalg.norm(terms, axis=1)
        assert err.max() <= REL_L2
    if units != 2:
        return
    singles = [P.spqr_gemm_smallbatch_ws(A, Xd, buf[256:256 + need]).clone() for A in As]
    torch.cuda.synchronize()
    types, ex, graph, st, hip = _graph_node_types(lambda s: P.spqr_gemm_fused_ws(As, Xd, buf[256:256 + need], outs=Ys, stream=s))
    assert all(t == 0 for t in types), types
    for rep in range(3):
        for Y in Ys:
            Y.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(ex, C.c_void_p(st.cuda_stream)) == 0
        torch.cuda.synchronize()
        assert all(torch.equal(Y, S) for Y, S in zip(Ys, singles)), rep
    assert hip.hipGraphExecDestroy(ex) == 0 and hip.hipGraphDestroy(graph) == 0


def test_static_array_takes_a_plan_of_fewer_partial_results(P):
    """The fastest plan's scratch does not fit the static array, one partial result of every row does: the one-pass kernel
    runs all the same (the slices would have added the outliers in binary32: other bits)."""
    import torch
    f = synth.make_matrix(8 * 2040, 32 * 100, w_bits=3, beta1=8, beta2=32, group_axis=1, outlier_rate=0.02, outlier_structure="uniform", seed=(89,))
    A = P.SpQRMatrix.from_logical(f)
    assert P.spqr_workspace_bytes(A, 200) > P.SPQR_STATIC_SCRATCH_BYTES
    X = synth.make_x(f.n, 200, seed=(90,))
    Xd = torch.from_numpy(X).to("cuda:0")
    out = torch.zeros((200, f.m), dtype=torch.float32, device="cuda:0")
    P.spqr_gemm_smallbatch_noalloc(A, Xd, out)
    ref = orc.matvec(f, X)
    assert (np.linalg.norm(out.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)).max() <= REL_L2
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX)
    slices = torch.zeros_like(out)
    P.spqr_gemm_smallbatch_noalloc(A, Xd, slices)
    assert not torch.equal(out, slices)
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_AUTO)
    assert (out - P.spqr_gemm_smallbatch(A, Xd)).norm() <= 1e-5 * out.norm()   # the same weights, sums in another order


def test_scratch_without_room_for_the_copy_is_the_slices(P):
    """A layer that the one-pass kernel took over from the dense copy, which never fitted the static array: without room for the
    copy its outliers are added in binary32 as they always were, bit for bit the slices, one matrix or several."""
    import torch
    fs = [synth.make_matrix(m, 4096, w_bits=3, beta1=16, beta2=16, group_axis=1, outlier_rate=0.005, outlier_structure="uniform", seed=(91, m))
          for m in (4096, 4112)]
    As = [P.SpQRMatrix.from_logical(f) for f in fs]
    b = 48
    Xd = torch.from_numpy(synth.make_x(4096, b, seed=(92,))).to("cuda:0")
    need = P.spqr_workspace_bytes(As, b)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_MATRIX)
    slices = [P.spqr_gemm_smallbatch_ws(A, Xd, ws).clone() for A in As]
    P.spqr_set_option(P.SPQR_OPT_BATCH_PATH, P.SPQR_BATCH_PATH_AUTO)
    one = P.spqr_gemm_smallbatch_ws(As[0], Xd, ws).clone()
    assert not torch.equal(one, slices[0])
    out = torch.zeros_like(one)
    assert torch.equal(P.spqr_gemm_smallbatch_noalloc(As[0], Xd, out), slices[0])
    few = ws[:2 * 4096 * 4096]                 # more than a plan of the one-pass kernel needs, less than the copy and its sums
    assert torch.equal(P.spqr_gemm_smallbatch_ws(As[0], Xd, few), slices[0])
    assert all(torch.equal(Y, S) for Y, S in zip(P.spqr_gemm_fused_ws(As, Xd, few), slices))


# groups of many chunks of the sort with a workgroup for each, and with one workgroup for all of them (a hint that is too small)
@pytest.mark.parametrize("w,b1,b2,axis,ntr,ntc,structure,rate", [(3, 16, 16, 1, 9, 131, "zipf", 0.15), (4, 8, 32, 0, 3, 450, "rows8cols4", 0.2)])
@pytest.mark.parametrize("hint", [0, 1, None])
def test_sort_with_any_number_of_workgroups(P, w, b1, b2, axis, ntr, ntc, structure, rate, hint):
    import torch
    tr, tc = synth.tile_shape(b1, b2, axis)
    f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=rate,
                          outlier_structure=structure, seed=(93, w, axis))
    A = P.SpQRMatrix.from_logical(f)
    X = torch.from_numpy(synth.make_x(f.n, 64, seed=(94,))).to("cuda:0")
    P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 1000)
    want = P.spqr_gemm_smallbatch(A, X).clone()
    if hint is None:
        P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 0)
        run(P, f, 64, prompt=1000)
        return
    A.desc.max_row_nnz = hint
    assert torch.equal(P.spqr_gemm_smallbatch(A, X), want)
    P.spqr_set_option(P.SPQR_OPT_PROMPT_PLAN, 0)


# 77 vectors: runs of 2 of 8 units; 256: of 5, two blocks of vectors
@pytest.mark.parametrize("b,perm", [(77, True), (256, False)])
def test_one_pass_of_several_matrices_by_itself(P, b, perm):
    """Nothing pinned, layers just above the size from which it is this kernel's, rows that differ: against the oracle, other partial
    sums than the single calls' (so they went together), and the binary16 outputs are the binary32 ones rounded."""
    import torch
    fs = [synth.make_matrix(m, 2000, w_bits=3, beta1=16, beta2=16, group_axis=1, outlier_rate=0.01, outlier_structure=st, seed=(95, m))
          for m, st in ((2064, "zipf"), (2128, "uniform"), (2000, "rows8cols4"))]
    if perm:
        for f in fs:
            f.perm = np.random.default_rng(5).permutation(f.n).astype(np.int32)
    As = [P.SpQRMatrix.from_logical(f) for f in fs]
    for A in As[1:]:
        A.desc.perm = As[0].desc.perm          # descriptors must name the same device permutation
    X = synth.make_x(2000, b, seed=(96, b))
    Xd = torch.from_numpy(X).to("cuda:0")
    ws = torch.empty(P.spqr_workspace_bytes(As, b), dtype=torch.uint8, device="cuda:0")
    Ys = P.spqr_gemm_fused_ws(As, Xd, ws)
    halves = P.spqr_gemm_fused_ws(As, Xd, ws, y_dtype=P.SPQR_F16)
    own = [P.spqr_gemm_smallbatch_ws(A, Xd, ws).clone() for A in As]
    assert not all(torch.equal(Y, O) for Y, O in zip(Ys, own))
    for f, Y, H, O in zip(fs, Ys, halves, own):
        assert torch.equal(H, Y.to(torch.float16))
        assert (Y - O).norm() <= 1e-5 * O.norm()               # the same weights, sums in another order
        Xp = X.astype(np.float64) if f.perm is None else X.astype(np.float64)[:, f.perm]
        terms = np.sqrt(Xp ** 2 @ (orc.reconstruct(f) ** 2).T)
        err = np.linalg.norm(Y.cpu().numpy() - orc.matvec(f, X), axis=1) / np.linalg.norm(terms, axis=1)
        assert err.max() <= REL_L2
