"""Host-side logic of the library (no GPU): size model, packer round trip
through the oracle-side layout reader, descriptor validation, exported symbols."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import paper_2306_03078_amd as P
import spqr_synth as synth
from oracle import layout_reader, spqr_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared(path):
    hdr = open(path).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    return set(re.findall(r"\b(spqr_[a-z_0-9]+)\s*\(", hdr))


def test_library_exports_every_declared_symbol():
    names = _declared(os.path.join(ROOT, "include", "spqr.h"))
    assert {"spqr_pack_check", "spqr_gemv", "spqr_gemv_fused", "spqr_gemv_grouped", "spqr_gemm_fused", "spqr_gemm_smallbatch",
            "spqr_gemm_smallbatch_ws", "spqr_gemm_fused_ws", "spqr_workspace_bytes", "spqr_dequant_dense", "spqr_set_option",
            "spqr_pack_host", "spqr_packed_bytes", "spqr_pack_host_layout", "spqr_packed_bytes_layout", "spqr_strerror",
            "spqr_version"} <= names
    assert "spqr_plan_batch" not in names      # a test hook, not part of the public interface
    enc = _declared(os.path.join(ROOT, "include", "spqr_encode.h"))
    assert {"spqr_hessian", "spqr_inverse_cholesky", "spqr_inverse_cholesky_workspace_bytes", "spqr_quantize",
            "spqr_quantize_workspace_bytes", "spqr_gather_outliers", "spqr_act_order", "spqr_act_order_workspace_bytes",
            "spqr_permute_columns", "spqr_permute_symmetric"} == enc
    names = names | enc
    hooks = _declared(os.path.join(ROOT, "paper_2306_03078_amd", "csrc", "spqr_test_hooks.h"))
    assert hooks == {"spqr_plan_batch", "spqr_plan_grouped", "spqr_sort_ranges", "spqr_batch_route", "spqr_plan_prompt", "spqr_sweep_rows"}
    lib = C.CDLL(P.library_path())
    for nm in sorted(names | hooks):
        assert hasattr(lib, nm), nm


@pytest.mark.parametrize("w,b1,b2", [(3, 16, 16), (4, 16, 16), (3, 8, 32), (3, 16, 32), (3, 32, 16),
                                     (4, 8, 16), (3, 64, 64), (3, 128, 128), (3, 8, 16), (3, 32, 128)])
@pytest.mark.parametrize("axis", [0, 1])
def test_packed_size_is_the_papers_size_model(w, b1, b2, axis):
    # App. D Eq. 4 without outliers: b_w + (b_s+b_z)/beta1 + 64/(beta1*beta2), no padding.
    tr, tc = synth.tile_shape(b1, b2, axis)
    m, n = 3 * tr, 5 * tc
    nbytes = P.packed_bytes(m, n, w, 3, 3, b1, b2, axis)
    assert 8.0 * nbytes / (m * n) == orc.average_bits(w, 3, 3, b1, b2)


@pytest.mark.parametrize("w,b1,b2", [(3, 16, 16), (4, 16, 16), (3, 8, 32), (3, 48, 16), (4, 8, 64)])
@pytest.mark.parametrize("axis", [0, 1])
def test_packed_size_of_the_statistic_variants(w, b1, b2, axis):
    # Sec. 5 ablations: integer zero-point (one second-level pair per tile), 16-bit statistics (none); no padding.
    tr, tc = synth.tile_shape(b1, b2, axis)
    m, n = 3 * tr, 5 * tc
    assert 8.0 * P.packed_bytes(m, n, w, 3, 3, b1, b2, axis, P.SPQR_LAYOUT_ROUND_ZERO) / (m * n) \
        == orc.average_bits_round_zero(w, 3, 3, b1, b2)
    assert 8.0 * P.packed_bytes(m, n, w, 16, 16, b1, b2, axis, P.SPQR_LAYOUT_STATS16) / (m * n) \
        == orc.average_bits_stats16(w, b1)
    lib = P.load_library()
    assert lib.spqr_packed_bytes_layout(P.SPQR_LAYOUT_STATS16, m, n, w, 3, 3, b1, b2, axis) == -3
    assert lib.spqr_packed_bytes_layout(P.SPQR_LAYOUT_ROUND_ZERO, m, n, w, 16, 16, b1, b2, axis) == -3
    assert lib.spqr_packed_bytes_layout(4, m, n, w, 3, 3, b1, b2, axis) == -3
    assert lib.spqr_packed_bytes_layout(1, m, n, w, 3, 3, b1, b2, axis) == P.packed_bytes(m, n, w, 3, 3, b1, b2, axis)


def test_printed_bit_counts_for_config_tiles():
    # 3.625 bits (beta1=beta2=16) and 4 bits (beta1=8, beta2=32), App. C table.
    assert 8 * P.packed_bytes(4096, 4096, 3, 3, 3, 16, 16, 1) / 4096 ** 2 == 3.625
    assert 8 * P.packed_bytes(8192, 8192, 3, 3, 3, 8, 32, 1) / 8192 ** 2 == 4.0
    # an outlier costs 32 bits + the per-row 32-bit count: "32.03 to 32.1 bits" (Sec. 4.2)
    f = synth.make_matrix(4096, 4096, outlier_rate=0.01, seed=(0, 0))
    per_outlier = (f.col_idx.nbytes + f.val.nbytes + f.row_ptr.nbytes) * 8 / f.nnz
    assert 32.0 < per_outlier < 32.9


def test_unsupported_parameters_are_rejected():
    assert P.load_library().spqr_packed_bytes(64, 64, 5, 3, 3, 16, 16, 0) == -3
    assert P.load_library().spqr_packed_bytes(64, 64, 3, 4, 3, 16, 16, 0) == -3
    assert P.load_library().spqr_packed_bytes(64, 64, 3, 3, 3, 16, 8, 0) == -3
    assert P.load_library().spqr_packed_bytes(60, 64, 3, 3, 3, 16, 16, 0) == -2
    assert P.load_library().spqr_packed_bytes(64, 1 << 17, 3, 3, 3, 16, 16, 0) == -2
    assert "NULL" in P.spqr_strerror(-1)


@pytest.mark.parametrize("w,b1,b2,axis,ntr,ntc", [
    (3, 16, 16, 1, 2, 3), (3, 16, 16, 0, 3, 70), (4, 16, 16, 1, 2, 130), (4, 16, 16, 0, 1, 64),
    (3, 8, 32, 1, 3, 65), (3, 8, 32, 0, 2, 129), (3, 16, 32, 0, 2, 5), (4, 32, 64, 1, 2, 3),
])
def test_pack_round_trip_through_independent_reader(w, b1, b2, axis, ntr, ntc):
    tr, tc = synth.tile_shape(b1, b2, axis)
    f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis,
                          outlier_rate=0.0, seed=(21, w, b1, b2, axis))
    buf = P.pack_host(f)
    got = layout_reader.read_packed(buf, f.m, f.n, w, b1, b2, axis)
    assert np.array_equal(got["Q"], f.Q)
    assert np.array_equal(got["s_q"], f.s_q)
    assert np.array_equal(got["z_q"], f.z_q)
    for k in ("s_s", "z_s", "s_z", "z_z"):
        assert np.array_equal(got[k].view(np.uint16), getattr(f, k).view(np.uint16)), k


@pytest.mark.parametrize("layout,lv", [("round_zero", 2), ("stats16", 3)])
@pytest.mark.parametrize("w,b1,b2,axis,ntr,ntc", [
    (3, 16, 16, 1, 2, 3), (3, 16, 16, 0, 3, 70), (4, 16, 16, 1, 2, 130), (3, 8, 32, 1, 3, 65), (3, 8, 32, 0, 2, 129),
    (3, 48, 16, 0, 2, 5), (4, 32, 64, 1, 2, 3),
])
def test_variant_pack_round_trip_through_independent_reader(layout, lv, w, b1, b2, axis, ntr, ntc):
    tr, tc = synth.tile_shape(b1, b2, axis)
    f = synth.make_matrix(ntr * tr, ntc * tc, w_bits=w, beta1=b1, beta2=b2, group_axis=axis, outlier_rate=0.0,
                          seed=(22, w, b1, b2, axis), stat_layout=layout)
    got = layout_reader.read_packed(P.pack_host(f), f.m, f.n, w, b1, b2, axis, lv)
    assert np.array_equal(got["Q"], f.Q)
    if lv == 2:
        assert set(got) == {"Q", "s_q", "z_q", "s_s", "z_s"}
        keys = ("s_q", "z_q", "s_s", "z_s")
    else:
        assert set(got) == {"Q", "s16", "z16"}
        keys = ("s16", "z16")
    for k in keys:
        a, b = got[k], getattr(f, k)
        assert np.array_equal(a.view(np.uint16) if a.dtype == np.float16 else a,
                              b.view(np.uint16) if b.dtype == np.float16 else b), k


def test_packer_rejects_out_of_range_codes():
    f = synth.make_matrix(32, 32, outlier_rate=0.0)
    f.Q[3, 3] = 9
    with pytest.raises(P.SpQRError) as ei:
        P.pack_host(f)
    assert ei.value.status == -3


def test_host_side_descriptor_checks_need_no_gpu():
    # NULL descriptor and bad parameters are refused before any HIP call.
    lib = P.load_library()
    assert lib.spqr_gemv(None, None, None, 0, None) == -1
    d = P.binding.spqr_matrix_t()
    d.m = d.n = 64; d.w_bits = 7; d.s_bits = d.z_bits = 3; d.beta1 = d.beta2 = 16
    d.layout_version = 1
    assert lib.spqr_gemv(C.byref(d), None, None, 0, None) == -3
    d.w_bits = 3
    assert lib.spqr_gemv(C.byref(d), None, None, 0, None) == -1      # packed is NULL
    d.max_row_nnz = -5
    assert lib.spqr_gemv(C.byref(d), None, None, 0, None) == -3      # the hint is a count
    d.max_row_nnz = 0
    d.layout_version = 2
    assert lib.spqr_dequant_dense(C.byref(d), 0, None, None) == -1   # the integer zero-point layout: packed is NULL
    d.layout_version = 3
    assert lib.spqr_dequant_dense(C.byref(d), 0, None, None) == -3   # 16-bit statistics need s_bits = z_bits = 16
    d.layout_version = 4
    assert lib.spqr_dequant_dense(C.byref(d), 0, None, None) == -3


def test_option_values():
    lib = C.CDLL(P.library_path())
    assert lib.spqr_set_option(2, -1) == -3 and lib.spqr_set_option(9, 0) == -3 and lib.spqr_set_option(0, 4) == -3
    assert all(lib.spqr_set_option(6, v) == -3 for v in (-1, 3 * 1024, 5 * 1024)) and lib.spqr_set_option(6, 4 * 1024 + 7) == 0
    assert lib.spqr_set_option(6, 0) == 0                                                                            # SPQR_OPT_PROMPT_PLAN
    assert lib.spqr_set_option(3, 96) == -3 and lib.spqr_set_option(3, 64) == 0 and lib.spqr_set_option(3, 0) == 0   # SPQR_OPT_DENSE_ROWS


# ---- plan of a grouped batch-1 launch (host arithmetic; the launcher checks the same invariants before it launches) ----

def _plan_grouped(ms, ns, hints, nnz, w, b1, b2, axis, layout, max_waves, slots, mf):
    lib = C.CDLL(P.library_path())
    fn = lib.spqr_plan_grouped
    fn.restype = C.c_int
    k = len(ms)
    I, L = C.c_int32 * k, C.c_int64 * k
    ent, nw, lds = (C.c_int32 * (7 * k))(), C.c_int32(), C.c_int64()
    rc = fn(k, I(*ms), I(*ns), I(*hints), L(*nnz), w, b1, b2, axis, layout, max_waves, slots, mf, ent, C.byref(nw), C.byref(lds))
    return rc, [tuple(ent[7 * j:7 * j + 7]) for j in range(max(rc, 0))], nw.value, lds.value


def _check_grouped_plan(entries, nw, lds, ms, ns, hints, tr, tc, max_waves):
    """What the kernel assumes of every table entry."""
    assert 1 <= nw <= max_waves and lds <= 160 * 1024
    assert len({e[0] for e in entries}) == len(entries)
    for idx, R, Pw, cap, shared, spare, wgs in entries:
        m, n = ms[idx], ns[idx]
        xbytes = (2 * n + 15) // 16 * 16
        assert R * Pw == nw and R * tr <= 64 and 1 <= Pw <= -(-(n // tc) // 64)
        assert 64 * nw <= cap <= 8 * 64 * nw                       # a chunk per thread at least, eight at most
        assert wgs == -(-(m // tr) // R)
        assert xbytes <= lds
        if shared:
            assert 32 * cap <= lds and xbytes + 32 * spare <= lds and spare <= cap
        else:
            assert xbytes + 32 * cap <= lds and spare == 0
    wide = [e for e in entries if ns[e[0]] > ns[0]]
    assert entries[:len(wide)] == wide                             # the wider matrices first in the grid
    assert all(e[4] == 1 for e in wide) and all(e[4] == 0 for e in entries[len(wide):])


def test_grouped_plan_of_the_65b_block_takes_down_along_with_its_products_over_x():
    ms, ns = [8192] * 4 + [22016] * 2 + [8192], [8192] * 6 + [22016]
    hints = [205, 204, 203, 202, 207, 201, 509]
    nnz = [int(0.02 * m * n) for m, n in zip(ms, ns)]
    rc, ent, nw, lds = _plan_grouped(ms, ns, hints, nnz, 3, 8, 32, 1, 1, 8, 12, 1)
    assert rc == 7 and nw == 4
    _check_grouped_plan(ent, nw, lds, ms, ns, hints, 8, 32, 8)
    down = ent[0]
    assert down[0] == 6 and down[1:3] == (2, 2) and down[4] == 1 and down[6] == 512
    assert 2 * 8 * 509 // 8 + 2 <= down[3]                         # by the hint, a workgroup's chunks fit one round
    assert all(e[1:3] == (4, 1) for e in ent[1:])                  # the six: four strips, one wavefront each
    assert 3 * (lds + 6144) <= 160 * 1024                          # three workgroups per compute unit still
    # without the hint on down's longest row it waits for a launch of its own; without outliers it needs none
    rc, ent, nw, lds = _plan_grouped(ms, ns, hints[:6] + [0], nnz, 3, 8, 32, 1, 1, 8, 12, 1)
    assert rc == 6 and all(e[0] != 6 for e in ent)
    rc, ent, nw, lds = _plan_grouped(ms, ns, hints[:6] + [0], nnz[:6] + [0], 3, 8, 32, 1, 1, 8, 12, 1)
    assert rc == 7 and ent[0][0] == 6 and ent[0][4] == 1


def test_grouped_plan_with_long_outlier_rows_depends_on_the_length_of_the_launch():
    # LLaMA-33B shapes, rows of up to n outliers: one strip per workgroup for down, rounds on the LDS behind x
    ms, ns = [6656] * 4 + [17920] * 2 + [6656], [6656] * 6 + [17920]
    nnz = [int(0.01 * m * n) for m, n in zip(ms, ns)]
    rc, ent, nw, lds = _plan_grouped(ms, ns, ns, nnz, 4, 16, 16, 1, 1, 8, 12, 0)
    assert rc == 7
    _check_grouped_plan(ent, nw, lds, ms, ns, ns, 16, 16, 8)
    assert ent[0][0] == 6 and ent[0][1:3] == (1, nw) and ent[0][4] == 1 and ent[0][5] >= 64 * nw
    # LLaMA-7B shapes: the whole block is long enough (2.3 steps per wavefront slot), q and down alone are not
    ms, ns = [4096] * 4 + [11008] * 2 + [4096], [4096] * 6 + [11008]
    nnz = [int(0.01 * m * n) for m, n in zip(ms, ns)]
    rc, ent, nw, lds = _plan_grouped(ms, ns, ns, nnz, 3, 16, 16, 1, 1, 16, 16, 0)
    assert rc == 7 and ent[0][0] == 6 and ent[0][1:3] == (1, nw)
    _check_grouped_plan(ent, nw, lds, ms, ns, ns, 16, 16, 16)
    rc, ent, nw, lds = _plan_grouped([4096, 4096], [4096, 11008], [4096, 11008], [167772, 450888], 3, 16, 16, 1, 1, 16, 16, 0)
    assert rc == 1 and ent[0][0] == 0
    # the same pair with short rows everywhere: together
    rc, ent, nw, lds = _plan_grouped([4096, 4096], [4096, 11008], [66, 145], [167772, 450888], 3, 16, 16, 1, 1, 16, 16, 0)
    assert rc == 2 and ent[0][0] == 1 and ent[0][4] == 1
    _check_grouped_plan(ent, nw, lds, [4096, 4096], [4096, 11008], [66, 145], 16, 16, 16)


@pytest.mark.parametrize("w,b1,b2,axis,tr,tc,max_waves,slots,mf", [
    (3, 8, 32, 1, 8, 32, 8, 12, 1), (4, 16, 16, 1, 16, 16, 8, 12, 0), (3, 16, 16, 0, 16, 16, 16, 16, 0),
    (3, 8, 32, 0, 32, 8, 8, 12, 0), (4, 8, 32, 0, 32, 8, 8, 8, 0)])
def test_grouped_plans_keep_the_kernels_invariants(w, b1, b2, axis, tr, tc, max_waves, slots, mf):
    rng = np.random.default_rng(7)
    for _ in range(200):
        k = int(rng.integers(1, 9))
        base_n = tc * int(rng.integers(20, 400))
        ns = [base_n] + [base_n if rng.random() < 0.5 else tc * int(rng.integers(20, 1500)) for _ in range(k - 1)]
        ns = [min(n, 65536 // tc * tc) for n in ns]
        ms = [tr * int(rng.integers(1, 3000)) for _ in range(k)]
        nnz = [int(rng.choice([0.0, 0.005, 0.02, 0.1]) * m * n) for m, n in zip(ms, ns)]
        hints = [0 if z == 0 else int(rng.choice([0, max(1, 2 * z // m), n])) for z, m, n in zip(nnz, ms, ns)]
        rc, ent, nw, lds = _plan_grouped(ms, ns, hints, nnz, w, b1, b2, axis, 1, max_waves, slots, mf)
        if rc < 0:
            assert rc == -3                                        # no plan (an x that does not fit the LDS)
            continue
        assert 1 <= rc <= k and any(e[0] == 0 for e in ent)        # the base matrix is always taken
        _check_grouped_plan(ent, nw, lds, ms, ns, hints, tr, tc, max_waves)
        for idx, R, Pw, cap, shared, spare, wgs in ent:
            if shared and nnz[idx]:
                assert hints[idx] > 0                              # never without a hint


def test_grouped_plan_arguments():
    lib = C.CDLL(P.library_path())
    fn = lib.spqr_plan_grouped
    fn.restype = C.c_int
    one32, one64 = (C.c_int32 * 1)(4096), (C.c_int64 * 1)(0)
    ent, nw, lds = (C.c_int32 * 7)(), C.c_int32(), C.c_int64()
    assert fn(1, one32, one32, one32, one64, 3, 16, 16, 1, 1, 16, 16, 0, ent, C.byref(nw), C.byref(lds)) == 1
    assert fn(0, one32, one32, one32, one64, 3, 16, 16, 1, 1, 16, 16, 0, ent, C.byref(nw), C.byref(lds)) == -3
    assert fn(1, one32, one32, one32, one64, 3, 16, 16, 1, 1, 0, 16, 0, ent, C.byref(nw), C.byref(lds)) == -3
    assert fn(1, None, one32, one32, one64, 3, 16, 16, 1, 1, 16, 16, 0, ent, C.byref(nw), C.byref(lds)) == -1
    assert fn(1, one32, one32, one32, one64, 5, 16, 16, 1, 1, 16, 16, 0, ent, C.byref(nw), C.byref(lds)) == -3   # w_bits


# ---- the outlier sort of the one-pass product: where its groups read and write ----

def _sort_ranges(row_ptr, nnz, rows):
    lib = C.CDLL(P.library_path())
    fn = lib.spqr_sort_ranges
    fn.restype, fn.argtypes = C.c_int64, [C.c_void_p, C.c_int, C.c_int64, C.c_int, C.c_void_p]
    m = len(row_ptr) - 1
    out = np.zeros((-(-m // rows), 3), np.int32)
    row_ptr = np.ascontiguousarray(row_ptr, np.int32)
    return fn(row_ptr.ctypes.data, m, nnz, rows, out.ctypes.data), out.astype(np.int64)


@pytest.mark.parametrize("rows", [128, 256])
def test_sort_ranges_of_valid_prefixes_are_the_groups_and_their_slots_never_meet(rows):
    rng = np.random.default_rng(11)
    for m in (1, 8, 127, 128, 129, 256, 4000):
        for scale in (0, 3, 200, 9000):
            ptr = np.concatenate([[0], np.cumsum(rng.integers(0, scale + 1, m) * (rng.random(m) < 0.7))])
            nnz = int(ptr[-1])
            slots, got = _sort_ranges(ptr, nnz, rows)
            bounds = ptr[np.minimum(np.arange(len(got) + 1) * rows, m)]
            assert (got[:, 0] == bounds[:-1]).all() and (got[:, 1] == bounds[1:]).all()
            used = [s + k for a, z, s in got for k in range(-(-(z - a) // 4096))]
            assert len(used) == len(set(used)) and all(0 <= u < slots for u in used)


@pytest.mark.parametrize("rows", [128, 256])
def test_sort_ranges_stay_inside_the_arrays_whatever_the_row_pointers_hold(rows):
    rng = np.random.default_rng(12)
    for _ in range(300):
        m, nnz = int(rng.integers(1, 3000)), int(rng.integers(0, 200000))
        ptr = rng.integers(-2 ** 31, 2 ** 31, m + 1) if rng.random() < 0.5 else rng.integers(-1000, nnz + 100000, m + 1)
        slots, got = _sort_ranges(ptr, nnz, rows)
        a, z, s = got.T
        assert (0 <= a).all() and (a <= z).all() and (z <= nnz).all()
        assert (s >= 0).all() and (s + -(-(z - a) // 4096) <= slots).all()


# ---- the plan of a slice of 4 to 16 vectors: splits of the columns, workgroups for the outliers ----

def _plan_batch(ms, n, nnz, hints, w, b1, b2, axis, b, widths=False):
    lib = C.CDLL(P.library_path())
    fn = lib.spqr_plan_batch
    fn.restype = C.c_int
    k = len(ms)
    I, L = C.c_int32 * k, C.c_int64 * k
    out = (C.c_int32 * 6)()
    units = fn(k, I(*ms), I(*([n] * k)), I(*hints), L(*nnz), w, b1, b2, axis, b, out)
    return (units, *(out if widths else out[:3]))


FORMATS = [(3, 16, 16, 1, 256), (4, 16, 16, 0, 256), (3, 8, 32, 1, 128), (4, 8, 32, 0, 256)]      # the last: rows of a group


def test_batch_plans_keep_the_kernels_invariants():
    rng = np.random.default_rng(13)
    for w, b1, b2, axis, rows in FORMATS:
        tr, tc = synth.tile_shape(b1, b2, axis)
        for _ in range(300):
            k = int(rng.integers(1, 9)) if rng.random() < 0.4 else 1
            n = tc * int(rng.integers(1, 65536 // tc // 4))
            ms = [tr * int(rng.integers(1, 3000 if rng.random() < 0.9 else 40000)) for _ in range(k)]
            nnz = [int(rng.choice([0.0, 0.005, 0.02, 0.2]) * m * n) for m in ms]
            hints = [0 if z == 0 else int(rng.choice([0, z // m + 1, n])) for z, m in zip(nnz, ms)]
            b = int(rng.integers(1, 17))
            units, per, splits, shares = _plan_batch(ms, n, nnz, hints, w, b1, b2, axis, b)
            assert units == -(-(n // tc) // 16)
            assert 1 <= per <= units and splits == -(-units // per) and (splits - 1) * per < units   # no split is empty
            assert shares in (0, 1, 2, 4) and shares <= rows // 64 and (shares == 0 or sum(nnz) > 0)
            parts = splits * (2 if shares else 1)
            assert parts == 1 or 4 * parts * b * sum(ms) <= 24 << 20


def test_widths_of_a_batch_plans_splits_cover_the_columns():
    """All units once, no split empty, none wider than a piece of XT or than the plan's, the wider ones first and where every CU gets two
    workgroups that do both parts; even where the plan has outliers apart and for 8 x 32 tiles, whose few units a split cannot be shared out."""
    rng = np.random.default_rng(14)
    uneven = 0
    for w, b1, b2, axis, rows in FORMATS:
        tr, tc = synth.tile_shape(b1, b2, axis)
        for _ in range(800):
            k = int(rng.integers(1, 4))
            n = tc * int(rng.integers(1, 20000 // tc))
            ms = [tr * int(rng.integers(1, 20000 // tr)) for _ in range(k)]
            nnz = [int(rng.choice([0.0, 0.005, 0.02]) * m * n) for m in ms]
            hints = [0 if z == 0 else int(rng.choice([0, z // m + 1, n])) for z, m in zip(nnz, ms)]
            units, per, splits, shares, width, lead, more = _plan_batch(ms, n, nnz, hints, w, b1, b2, axis, int(rng.integers(1, 17)), True)
            first = [y * width + min(y, lead) * more for y in range(splits + 1)]
            assert first[splits] >= units and first[splits - 1] < units and width >= 1 and lead >= 0 and more >= 0
            assert width + more <= max(1536 // (16 * tc), per)
            if more == 0:
                assert width == per
                continue
            uneven += 1
            groups = sum(-(-m // rows) for m in ms)
            assert shares == 0 and sum(nnz) > 0 and 256 < groups * splits <= 512 and groups * lead <= 256 and tc != 32
    assert uneven > 20


def test_widths_of_the_layers_that_lost_time():
    """Even where splits of unequal width were up to a tenth slower, wider first ones where they are 4 to 12 % faster (all timed)."""
    def widths(ms, n, rate, hint, w, b1, b2, axis, b):
        units, _, splits, _, width, lead, more = _plan_batch(ms, n, [int(rate * m * n) for m in ms], [hint] * len(ms), w, b1, b2, axis, b, True)
        first = [min(units, y * width + min(y, lead) * more) for y in range(splits + 1)]
        return [z - a for a, z in zip(first, first[1:])]
    assert widths([8384] * 3, 3616, 0.02, 3616, 3, 16, 16, 0, 4) == [3] * 5                          # 5 5 2 2 1: 44.8 -> 48.9 us
    assert widths([12768] * 2, 5024, 0.01, 5024, 3, 16, 16, 0, 4) == [4] * 5                         # 6 6 3 3 2: 39.7 -> 41.8
    assert widths([8768] * 3, 1728, 0.02, 1728, 3, 8, 32, 1, 15) == [2, 2]                           # 3 1: 33.6 -> 36.4
    assert widths([6656] * 3, 6656, 0.01, 6656, 4, 16, 16, 1, 4) == [5, 5, 5, 4, 4, 3]               # 5 5 5 5 5 1: 44.5 -> 41.2
    assert widths([13248] * 3, 2464, 0.02, 2464, 3, 16, 16, 0, 6) == [4, 3, 3]                       # 4 4 2: 43.6 -> 38.5


def test_batch_plans_of_the_layers_that_lost_time():
    """The splits and shares that are within 4 % of the fastest of all on these layers (16 vectors, all of them timed)."""
    def plan(ms, n, rate, hint, fmt):
        return _plan_batch(ms, n, [int(rate * m * n) for m in ms], [hint] * len(ms), *fmt[:4], 16)[1:]
    t8, t16 = FORMATS[2], FORMATS[0]
    assert plan([22016], 8192, 0.02, 230, t8) in ((3, 6, 0), (3, 6, 1))        # 6 units: 80 us against 64
    assert plan([22016, 22016], 8192, 0.01, 130, t16)[0] == 6                  # 7 units: 118 against 98
    assert plan([1024], 1024, 0.01, 1024, t16)[2] >= 2                         # heavy rows in their own workgroups: 16.9 -> 11.1
    assert plan([5120], 5120, 0.01, 5120, t16) in ((5, 4, 2), (4, 5, 4))       # 24.9 -> 18.3
    assert plan([17920], 6656, 0.01, 6656, t16) == (4, 7, 0)                   # no CUs to spare: 44.6, apart 46.9


def test_batch_plan_pins():
    lib = C.CDLL(P.library_path())
    args = ([4096], 4096, [167772], [66], 3, 16, 16, 1, 16)
    try:
        for per in (1, 3, 16, 1000):
            for code, shares in ((1, 0), (2, 1), (3, 2), (5, 4)):
                assert lib.spqr_set_option(2, per) == 0 and lib.spqr_set_option(5, code) == 0
                assert _plan_batch(*args) == (16, min(per, 16), -(-16 // min(per, 16)), shares)
        assert lib.spqr_set_option(5, 4) == -3 and lib.spqr_set_option(5, -1) == -3
        assert _plan_batch([4096], 4096, [0], [0], 3, 16, 16, 1, 16)[3] == 0   # nothing to share out
        assert _plan_batch([4096], 4096, [167772], [66], 3, 8, 32, 1, 16)[3] == 2   # two sets of 64 rows
    finally:
        assert lib.spqr_set_option(2, 0) == 0 and lib.spqr_set_option(5, 0) == 0
    assert _plan_batch([4096], 4096, [0], [0], 3, 32, 32, 1, 16)[0] == -3      # no such instance


# ---- scratch of large batches (host arithmetic on descriptors whose pointers are never followed) ----

def _workspace_bytes(m, n, w, b1, b2, axis, rate, b, perm=False):
    from paper_2306_03078_amd import binding as B
    lib = B.load_library()
    d = B.spqr_matrix_t(m=m, n=n, w_bits=w, s_bits=3, z_bits=3, beta1=b1, beta2=b2, group_axis=axis, layout_version=1,
                        packed=4096, packed_bytes=P.packed_bytes(m, n, w, 3, 3, b1, b2, axis), row_ptr=4096, col_idx=4096,
                        out_val=4096, nnz=int(rate * m * n), perm=4096 if perm else None)
    return lib.spqr_workspace_bytes((C.POINTER(B.spqr_matrix_t) * 1)(C.pointer(d)), 1, b)


def test_workspace_of_the_one_pass_kernel_holds_no_dense_copy():
    for m, n, w, b1, b2, rate, b in ((17920, 6656, 4, 16, 16, 0.01, 256), (8192, 22016, 3, 8, 32, 0.02, 128), (8192, 8192, 3, 8, 32, 0.02, 64)):
        need = _workspace_bytes(m, n, w, b1, b2, 1, rate, b)
        # 4 bytes per outlier, partial results of 64 MB at most where there are several, the sort's ranges and counts
        assert 4 * int(rate * m * n) < need < 4 * int(rate * m * n) + max(64 << 20, 4 * b * m) + (8 << 20)
        assert need < 2 * m * n                                            # the copy alone
    # more outliers than one weight in four, or a layer too small: the copy
    assert _workspace_bytes(8192, 4096, 4, 16, 16, 1, 0.3, 128) > 2 * 8192 * 4096
    assert _workspace_bytes(1024, 1024, 4, 16, 16, 1, 0.01, 64) > 2 * 1024 * 1024


SLICES, COPY, ONE_PASS = 0, 1, 2
LIBRARY, STATIC = -1, -2


def _route(m, n, w, b1, b2, axis, rate, b, scratch, perm=False, hint=0):
    from paper_2306_03078_amd import binding as B
    return B.load_library().spqr_batch_route(m, n, C.c_int64(int(rate * m * n)), hint, int(perm), w, b1, b2, axis, b, C.c_int64(scratch))


# both sides of 4 M weights, of 512 columns and of 12 M weights with tiles of 8 columns
@pytest.mark.parametrize("m,n,w,b1,b2,axis,b,route", [
    (17920, 2048, 4, 16, 16, 1, 256, ONE_PASS), (17920, 2048, 4, 16, 16, 1, 192, ONE_PASS), (17920, 1536, 3, 16, 16, 1, 256, ONE_PASS),
    (17920, 2064, 4, 16, 16, 1, 256, ONE_PASS), (5120, 5120, 3, 16, 16, 1, 256, ONE_PASS), (4864, 4864, 4, 16, 16, 1, 128, ONE_PASS),
    (2000, 2000, 3, 16, 16, 0, 48, ONE_PASS), (1984, 2000, 3, 16, 16, 0, 48, COPY), (1984, 2000, 3, 16, 16, 0, 47, SLICES),
    (8192, 512, 4, 16, 16, 1, 128, ONE_PASS), (8192, 496, 4, 16, 16, 1, 128, COPY), (17920, 256, 3, 8, 32, 1, 128, COPY),
    (17920, 480, 3, 8, 32, 1, 128, COPY), (8192, 512, 3, 8, 32, 1, 128, ONE_PASS), (2048, 2048, 3, 8, 32, 1, 64, ONE_PASS),
    (1024, 1024, 3, 8, 32, 1, 64, COPY), (3488, 3440, 3, 8, 32, 0, 64, COPY), (3488, 3448, 3, 8, 32, 0, 64, ONE_PASS)])
def test_sizes_of_the_one_pass_kernel(m, n, w, b1, b2, axis, b, route):
    assert _route(m, n, w, b1, b2, axis, 0.01, b, LIBRARY) == route


# `line`: the scratch from which on a call of that size has had 16-bit sums of weight and outlier since it could, the dense copy
# (a multiple of it: `copy`) or the plan of the one-pass kernel's first form; `static`: what 32 MB are
@pytest.mark.parametrize("m,n,w,b1,b2,axis,rate,perm,b,line,copy,static", [
    (4096, 4096, 3, 16, 16, 1, 0.01, False, 48, 39845888, True, SLICES), (4096, 4096, 4, 16, 16, 0, 0.01, True, 256, 69206016, True, SLICES),
    (4864, 4864, 4, 16, 16, 1, 0.01, False, 128, 67239936, True, SLICES), (2048, 8192, 3, 8, 32, 0, 0.01, False, 48, 36700160, True, SLICES),
    (17920, 2048, 4, 16, 16, 1, 0.01, True, 256, 221249536, True, SLICES), (2048, 2048, 3, 16, 16, 1, 0.01, False, 48, 11534336, True, ONE_PASS),
    (5120, 5120, 3, 16, 16, 1, 0.01, False, 256, 27280128, False, ONE_PASS), (17920, 2064, 4, 16, 16, 1, 0.01, False, 256, 19846912, False, ONE_PASS),
    (8192, 8192, 3, 8, 32, 1, 0.02, False, 64, 13874432, False, ONE_PASS), (2048, 2048, 3, 8, 32, 1, 0.01, True, 64, 2530304, False, ONE_PASS),
    (6464, 8416, 3, 16, 16, 1, 0.05, True, 96, 35025408, False, SLICES), (4528, 13536, 4, 16, 16, 0, 0.01, False, 128, 34987776, False, SLICES),
    (5376, 5800, 4, 8, 32, 0, 0.005, False, 256, 33669120, False, SLICES), (17920, 6656, 4, 16, 16, 1, 0.01, False, 256, 59911680, False, SLICES),
    (16320, 3200, 3, 8, 32, 1, 0.02, False, 200, 17291776, False, ONE_PASS), (22016, 8192, 3, 8, 32, 1, 0.02, True, 192, 34796800, False, SLICES)])
def test_a_batch_is_rounded_no_earlier_for_a_smaller_plan(m, n, w, b1, b2, axis, rate, perm, b, line, copy, static):
    """With less scratch than `line` the outliers are added in binary32 (slices), however little a plan of the one-pass kernel
    needs, and what spqr_workspace_bytes reports is never less than that."""
    need = _workspace_bytes(m, n, w, b1, b2, axis, rate, b, perm)
    route = [_route(m, n, w, b1, b2, axis, rate, b, scratch, perm) for scratch in (LIBRARY, need, line - 1, 0, STATIC)]
    assert route == [ONE_PASS, ONE_PASS, SLICES, SLICES, static] and need >= line
    if copy:
        assert _route(m, n, w, b1, b2, axis, rate, b, line, perm) == ONE_PASS


@pytest.mark.parametrize("m,n,b,hint,route", [
    (4096, 4096, 48, 4096, ONE_PASS), (4096, 4096, 95, 0, ONE_PASS), (4096, 4096, 96, 4096, COPY), (4096, 4096, 256, 0, COPY),
    (4096, 4096, 256, 80, ONE_PASS), (2048, 8192, 192, 8192, COPY), (3584, 3584, 128, 700, COPY), (3584, 3584, 128, 60, ONE_PASS),
    (512, 24576, 256, 24576, ONE_PASS), (2016, 8192, 256, 8192, ONE_PASS), (2048, 8192, 256, 8192, COPY),
    (17920, 1024, 256, 1024, ONE_PASS), (3072, 6144, 128, 0, ONE_PASS), (3456, 3456, 64, 60, COPY)])
def test_narrow_tiles_with_heavy_rows_take_the_copy(m, n, b, hint, route):
    """Tiles of 8 columns between 12 and 18 M weights: the copy is up to 15 % faster there where a few rows hold the outliers (hint:
    the longest row; 0: not known) and the batch is not small."""
    assert _route(m, n, 3, 8, 32, 0, 0.01, b, LIBRARY, hint=hint) == route


def test_a_batch_with_the_reported_scratch_goes_as_with_the_librarys():
    rng = np.random.default_rng(14)
    for w, b1, b2, axis, _ in FORMATS:
        tr, tc = synth.tile_shape(b1, b2, axis)
        for _ in range(200):
            m, n = tr * int(rng.integers(1, 24000 // tr)), tc * int(rng.integers(1, 24000 // tc))
            args = (m, n, w, b1, b2, axis, float(rng.choice([0.0, 0.01, 0.02, 0.3])), int(rng.integers(1, 257)))
            perm = bool(rng.integers(2))
            assert _route(*args, _workspace_bytes(*args, perm), perm) == _route(*args, LIBRARY, perm)


def _plan_prompt(ms, n, nnz, hints, w, b1, b2, axis, b, most_slots=0):
    """units, vectors and units per workgroup, workgroups per block of vectors, partial results, workgroups of the sort, us"""
    from paper_2306_03078_amd import binding as B
    k = len(ms)
    plan, us = (C.c_int32 * 5)(), C.c_double()
    rc = B.load_library().spqr_plan_prompt(k, (C.c_int32 * k)(*ms), (C.c_int32 * k)(*[n] * k), (C.c_int32 * k)(*hints), (C.c_int64 * k)(*nnz),
                                           w, b1, b2, axis, b, most_slots, plan, C.byref(us))
    return (rc, *plan, us.value)


def test_one_pass_plans_keep_the_kernels_invariants():
    rng = np.random.default_rng(15)
    for w, b1, b2, axis, _ in FORMATS:
        tr, tc = synth.tile_shape(b1, b2, axis)
        for _ in range(300):
            k = int(rng.integers(1, 9)) if rng.random() < 0.4 else 1
            n = tc * int(rng.integers(1, 32768 // tc // 2))
            ms = [tr * int(rng.integers(1, 40000 // tr)) for _ in range(k)]
            b, most = int(rng.integers(1, 257)), int(rng.integers(0, 4))
            units, vectors, run, runs, slots, wgs, us = _plan_prompt(ms, n, [0] * k, [0] * k, w, b1, b2, axis, b, most)
            total = units * sum(-(-m // 128) for m in ms)
            assert vectors in (64, 96, 128, 192) and runs == -(-total // run) and 1 <= run <= 2048 // (tc // 8)
            assert slots >= max(((g * units + units - 1) // run - g * units // run + 1) for g in range(min(total // units, 300)))
            assert slots == 1 or (slots <= (most or slots) and 4 * slots * b * 128 * total // units <= 64 << 20)
            assert 0 < us < 1e6


def test_one_pass_plans_of_few_partial_results_are_as_wide_as_they_should_be():
    """Whole groups per workgroup are priced like any other plan: 256 vectors are 2 x 128 and not 2 x 192 (128 and 192 vectors a
    workgroup, runs of a group, timed: two of 22016 x 8192 289 and 324 us, two of 17920 x 6656 236 and 261)."""
    z8, z16 = int(0.01 * 22016 * 8192), int(0.01 * 17920 * 6656)
    assert _plan_prompt([22016] * 2, 8192, [z8] * 2, [0, 0], 3, 8, 32, 1, 256)[1:5] == (128, 16, 344, 1)
    for b, most in ((256, 0), (256, 1), (200, 1)):
        assert _plan_prompt([17920] * 2, 6656, [z16] * 2, [0, 0], 4, 16, 16, 1, b, most)[1] <= 128
    assert _plan_prompt([17920] * 2, 6656, [z16] * 2, [0, 0], 4, 16, 16, 1, 128)[1:5] == (128, 15, 486, 3)   # nothing in the way


def test_matrices_go_one_by_one_where_that_is_faster():
    """The scratch of two is that of one where they don't share launches: gate and up 17920 x 6656 with 256 vectors (251 us together,
    222 one by one), not with 192 (156 and 191), not 22016 x 8192 with 256 (289 and 361)."""
    def together(m, n, w, b1, b2, b):
        from paper_2306_03078_amd import binding as B
        d = B.spqr_matrix_t(m=m, n=n, w_bits=w, s_bits=3, z_bits=3, beta1=b1, beta2=b2, group_axis=1, layout_version=1,
                            packed=4096, packed_bytes=P.packed_bytes(m, n, w, 3, 3, b1, b2, 1), row_ptr=4096, col_idx=4096,
                            out_val=4096, nnz=int(0.01 * m * n))
        two = (C.POINTER(B.spqr_matrix_t) * 2)(C.pointer(d), C.pointer(d))
        return B.load_library().spqr_workspace_bytes(two, 2, b) != B.load_library().spqr_workspace_bytes(two, 1, b)
    assert not together(17920, 6656, 4, 16, 16, 256)
    assert together(17920, 6656, 4, 16, 16, 192) and together(22016, 8192, 3, 8, 32, 256) and together(11008, 4096, 3, 16, 16, 77)


def test_the_outlier_sort_of_a_few_heavy_rows_has_a_workgroup_for_every_chunk():
    """A chunk is 4096 outliers.  Four workgroups a group, whatever it held, cost up to 60 of 107 us on layers of few rows."""
    wgs = lambda ms, n, nnz, hints: _plan_prompt(ms, n, nnz, hints, 3, 16, 16, 1, 128)[5]
    full, even = 128 * 24576, [256] * 4
    assert wgs([512], 24576, [300000], [24576]) == -(-300000 // 4096)       # any group may hold all of them
    assert wgs([512], 24576, [300000], [0]) == -(-300000 // 4096)           # nothing known of the rows
    assert wgs([512], 24576, [125829], [300]) == -(-128 * 300 // 4096)      # rows of much the same length
    assert wgs([512], 24576, [0], [0]) == 1
    assert wgs([17920], 6656, [1192755], [6656]) == 1024 // 140             # no more than the chip takes at once
    assert wgs([512] * 4, 24576, [100000] * 3 + [full], even[:3] + [24576]) == 1024 // 16
    assert wgs([65536], 4096, [2684354], [4096]) == 4


def test_direct_calls_take_tensors_by_address_and_refuse_what_they_cannot_pass():
    """The extension module's call: a one-element integer tensor is an address like any other, not the number it holds;
    statuses come back as they are; nothing else than integers, tensors and None is passed."""
    import torch
    from paper_2306_03078_amd import binding as B
    B.load_library()
    d, one = B.spqr_matrix_t(), torch.tensor([7])
    seen = []

    @C.CFUNCTYPE(C.c_int, *[C.c_int64] * 8)
    def entry(*args):
        seen.append(args)
        return -5
    address = C.cast(entry, C.c_void_p).value
    assert B._call(address, d, one, None, np.int32(3), -2, 2 ** 63 + 5) == -5
    assert seen == [(C.addressof(d), one.data_ptr(), 0, 3, -2, 2 ** 63 + 5 - 2 ** 64, 0, 0)]
    for bad in ((address,), (address, 5), (address, d, "x"), (address, d, 1.5), (address, d) + (0,) * 8):
        with pytest.raises(TypeError):
            B._call(*bad)
    assert B._call(B._entry["spqr_gemv"], d, one, one, 0, None) == -3      # refused before any HIP call


@pytest.mark.parametrize("extension", [True, False])
def test_product_calls_refuse_what_they_always_did_with_and_without_the_extension_module(extension, monkeypatch):
    """A number is no output, None no dtype; a library that was built without the extension module loads and gives the same
    statuses.  (A descriptor of zeros is refused before any HIP call.)"""
    import sys
    from types import SimpleNamespace
    import torch
    from paper_2306_03078_amd import binding as B
    B.load_library()
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_call", None)
    monkeypatch.setattr(B, "_entry", {})
    if not extension:
        monkeypatch.setitem(sys.modules, "paper_2306_03078_amd._calls", None)
        monkeypatch.delattr(sys.modules["paper_2306_03078_amd"], "_calls", raising=False)
    B.load_library()
    assert (B._call is B._ctypes_call) != extension
    stream = SimpleNamespace(cuda_stream=0)
    A = SimpleNamespace(desc=B.spqr_matrix_t(), m=4, n=8)
    x, X, y, Y, ws = (torch.zeros(k, dtype=torch.float16) for k in (8, (2, 8), 4, (2, 4), 256))
    calls = (lambda out, dt: B.spqr_gemv(A, x, out=out, y_dtype=dt, stream=stream),
             lambda out, dt: B.spqr_gemm_smallbatch(A, X, out=out, y_dtype=dt, stream=stream),
             lambda out, dt: B.spqr_gemm_smallbatch_ws(A, X, ws, out=out, y_dtype=dt, stream=stream))
    for call, out in zip(calls, (y, Y, Y)):
        with pytest.raises(AttributeError):
            call(out.data_ptr(), B.SPQR_F16)
        for dtype in (None, 1.0):
            with pytest.raises((TypeError, C.ArgumentError)):
                call(out, dtype)
        with pytest.raises(B.SpQRError) as e:
            call(out, B.SPQR_F16)
        assert e.value.status == -3


def test_build_does_without_the_extension_module(monkeypatch, tmp_path):
    """No compiler or no Python.h: no command for it, rather than a build that fails."""
    import shutil
    import sysconfig
    from paper_2306_03078_amd import build
    assert build.calls_command()[-1].endswith("spqr_calls.c")
    paths = dict(sysconfig.get_paths())
    with monkeypatch.context() as m:
        m.setattr(sysconfig, "get_paths", lambda *a: dict(paths, include=str(tmp_path)))
        assert build.calls_command() is None
    monkeypatch.setattr(shutil, "which", lambda name: None)
    assert build.calls_command() is None
