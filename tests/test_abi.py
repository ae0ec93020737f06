"""The C ABI without a GPU: the library loads, exports every function that
include/last.h declares, and rejects malformed calls on the host before any
HIP call (so these run on a machine with no GPU). Fake device pointers are
host buffers filled with a sentinel; a rejected call must leave them as is.
"""
import ctypes
import math
import os
import re
from fractions import Fraction

import numpy as np
import pytest

from paper_2607_27952_amd import last

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "last.h")


def _declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    names = set(re.findall(r"^\s*[A-Za-z_][\w\s\*]*?\b([a-z_][a-z0-9_]*)\s*\(", src, flags=re.M))
    return sorted(n for n in names if not n.startswith("__"))


def test_header_declares_the_path():
    names = _declared_functions()
    for n in ("last_token_scores", "diverse_select", "gather_kept", "last_budget",
              "last_token_scores_workspace", "diverse_select_workspace", "last_status_string"):
        assert n in names


def test_library_exports_every_declared_function():
    L = last.lib()
    for n in _declared_functions():
        assert hasattr(L, n), f"{n} declared in last.h but not exported"
    assert set(last.EXPORTS) <= set(_declared_functions())
    assert L.last_version() == 100


def test_status_strings():
    for s in range(5):
        assert last.status_string(s)
    assert last.status_string(0) == "ok"


def test_budget_matches_eq2():
    for n in range(1, 400):
        for num, den in [(1, 8), (3, 8), (5, 8), (1, 9), (2, 3), (1, 1)]:
            assert last.budget(n, num, den) == math.ceil(Fraction(n * num, den))
    assert last.budget(0, 1, 8) == -1
    assert last.budget(10, 0, 8) == -1
    assert last.budget(10, 9, 8) == -1


class Fake:
    """Host buffers standing in for device pointers; never dereferenced by a rejected call."""

    def __init__(self, n=4096):
        self.buf = np.full(n, 0x5A5A5A5A, dtype=np.uint32)

    @property
    def p(self):
        return self.buf.ctypes.data

    def untouched(self):
        return bool(np.all(self.buf == 0x5A5A5A5A))


def _batch(R=2, G=1, Hq=4, Hkv=2, Dh=128, P=(20, 30), N=(10, 12), vis=(2, 3), dtype=last.LAST_BF16):
    cs = np.zeros(R + 1, np.int32)
    cs[1:] = np.cumsum(P)
    cv = np.zeros(R + 1, np.int32)
    cv[1:] = np.cumsum(N)
    vs = np.asarray(vis, np.int32)
    dev = Fake()
    b = last._Batch(R, G, Hq, Hkv, Dh, dtype, 0.0, dev.p, cs.ctypes.data, dev.p, vs.ctypes.data,
                    dev.p, cv.ctypes.data)
    return b, (cs, cv, vs, dev)


def _scores_call(b, ws_bytes=1 << 30):
    q, k, out, ws = Fake(), Fake(), Fake(), Fake()
    st = last.lib().last_token_scores(ctypes.byref(b), q.p, k.p, out.p, None, ws.p, ws_bytes, None)
    assert out.untouched() and ws.untouched()
    return st


def test_scores_workspace_query():
    b, keep = _batch()
    assert last.lib().last_token_scores_workspace(ctypes.byref(b)) > 0
    b.Hq = 3
    assert last.lib().last_token_scores_workspace(ctypes.byref(b)) == 0


@pytest.mark.parametrize("field,value,expect", [
    ("R", 0, last.LAST_ERR_INVALID),
    ("G", 0, last.LAST_ERR_INVALID),
    ("Hq", 3, last.LAST_ERR_INVALID),          # Hq % Hkv != 0
    ("Hkv", 0, last.LAST_ERR_INVALID),
    ("Dh", 96, last.LAST_ERR_UNSUPPORTED),
    ("qk_dtype", 7, last.LAST_ERR_INVALID),
    ("softmax_scale", float("nan"), last.LAST_ERR_INVALID),
    ("G", 2000, last.LAST_ERR_UNSUPPORTED),    # G * Hq over the finalize limit
])
def test_scores_rejects_bad_shapes(field, value, expect):
    b, keep = _batch()
    setattr(b, field, value)
    assert _scores_call(b) == expect


def test_scores_rejects_bad_csr():
    b, keep = _batch(P=(20, 30), N=(10, 12), vis=(2, 3))
    cs, cv, vs, dev = keep
    cs[1] = 40                                    # decreasing offsets
    assert _scores_call(b) == last.LAST_ERR_INVALID
    b, keep = _batch(P=(20, 30), N=(10, 12), vis=(10, 3))   # span runs into the last token
    assert _scores_call(b) == last.LAST_ERR_INVALID
    b, keep = _batch(P=(20, 30), N=(10, 12), vis=(-1, 3))
    assert _scores_call(b) == last.LAST_ERR_INVALID
    b, keep = _batch(P=(1, 30), N=(0, 12), vis=(0, 3))        # P_r < 2 and N_r < 1
    assert _scores_call(b) == last.LAST_ERR_INVALID
    b, keep = _batch()
    b.cu_vis_h = None
    assert _scores_call(b) == last.LAST_ERR_INVALID


def test_scores_rejects_null_and_small_workspace():
    b, keep = _batch()
    q, out, ws = Fake(), Fake(), Fake()
    L = last.lib()
    assert L.last_token_scores(ctypes.byref(b), None, q.p, out.p, None, ws.p, 1 << 30, None) == last.LAST_ERR_INVALID
    need = L.last_token_scores_workspace(ctypes.byref(b))
    assert L.last_token_scores(ctypes.byref(b), q.p, q.p, out.p, None, ws.p, need - 1, None) == last.LAST_ERR_WORKSPACE
    assert L.last_token_scores(ctypes.byref(b), q.p, q.p, out.p, None, None, need, None) == last.LAST_ERR_WORKSPACE
    assert L.last_token_scores(ctypes.byref(b), q.p + 2, q.p, out.p, None, ws.p, need, None) == last.LAST_ERR_INVALID
    assert out.untouched() and ws.untouched()


def _select_call(cv, ck, Dv=64, fdtype=last.LAST_BF16, mode=last.KCENTER, ws_bytes=1 << 40):
    cv = np.asarray(cv, np.int32)
    ck = None if ck is None else np.asarray(ck, np.int32)
    dev, out, ws = Fake(), Fake(), Fake()
    st = last.lib().diverse_select(len(cv) - 1, Dv, fdtype, mode, dev.p, dev.p, dev.p, cv.ctypes.data,
                                   dev.p, None if ck is None else ck.ctypes.data, out.p, out.p, out.p,
                                   ws.p, ws_bytes, None)
    assert out.untouched() and ws.untouched()
    return st


def test_select_rejects_bad_budgets_and_shapes():
    E = last.LAST_ERR_INVALID
    assert _select_call([0, 10, 30], [0, 11, 15]) == E            # K_r > N_r
    assert _select_call([0, 10, 30], [0, 0, 5]) == E              # K_r = 0
    assert _select_call([0, 10, 30], None) == E                   # no host budgets
    assert _select_call([0, 10, 10], [0, 5, 5]) == E              # N_r = 0
    assert _select_call([1, 10, 30], [0, 5, 6]) == E              # offsets not from 0
    assert _select_call([0, 10, 30], [0, 5, 6], Dv=0) == E
    assert _select_call([0, 10, 30], [0, 5, 6], mode=5) == E
    assert _select_call([0, 10, 30], [0, 5, 6], fdtype=3) == E
    U = last.LAST_ERR_UNSUPPORTED
    assert _select_call([0, 131073], [0, 5]) == U                 # request beyond the largest selected
    assert _select_call([0, 10, 30], [0, 5, 6], Dv=60) == U       # bf16 rows not 16-byte multiples
    assert _select_call([0, 10, 30], [0, 5, 6], Dv=62, fdtype=last.LAST_F32) == U


def test_select_workspace_and_small_workspace():
    cv = np.array([0, 100, 350], np.int32)
    need = last.lib().diverse_select_workspace(2, cv.ctypes.data, 64, last.LAST_BF16, last.KCENTER)
    assert need >= (100 * 100 + 250 * 250) * 4
    assert _select_call(cv, [0, 5, 6], ws_bytes=need - 1) == last.LAST_ERR_WORKSPACE
    topk = last.lib().diverse_select_workspace(2, cv.ctypes.data, 64, last.LAST_BF16, last.TOPK)
    assert 0 < topk < need
    assert last.lib().diverse_select_workspace(2, cv.ctypes.data, 0, last.LAST_BF16, last.KCENTER) == 0


def test_kcenter_form_and_workspace(monkeypatch):
    """The k-center's form decides its workspace: the rounds keep no N x N
    matrix (28 bytes a token and 1.3 KB a request), the matrix form 4 N_r^2
    bytes. By default the rounds take batches whose every request has 8192
    tokens or more (bf16, Dv a multiple of 256 up to 4096, N_r <= 32768);
    LAST_KCENTER_FORM forces either; the two-call form always keeps the
    matrix."""
    L = last.lib()
    long_ = np.array([0, 16384, 32768], np.int32)          # two 16384-token requests
    mixed = np.array([0, 16384, 16384 + 500], np.int32)    # one short request
    mat = (2 * 16384 * 16384) * 4
    def ws(cv, Dv=3584, dt=last.LAST_BF16):
        return L.diverse_select_workspace(2, cv.ctypes.data, Dv, dt, last.KCENTER)
    monkeypatch.delenv("LAST_KCENTER_FORM", raising=False)
    def rounds_bytes(cv):                                  # with 256-byte padding of a dozen arrays
        return 28 * int(cv[-1]) + 1316 * (len(cv) - 1) + 2 * 8 * 128 + 13 * 256
    assert 28 * 32768 < ws(long_) <= rounds_bytes(long_)   # rounds: no matrix
    assert ws(mixed) > (16384 ** 2) * 4                    # matrix form
    assert ws(long_, Dv=3600) > mat                        # Dv not a multiple of 256: matrix
    assert ws(long_, dt=last.LAST_F32) > mat               # fp32 features: matrix
    assert ws(long_, Dv=4352) > mat                        # wider than 4096: matrix
    pair = L.diverse_select_similarity_workspace(2, long_.ctypes.data, 3584, last.LAST_BF16)
    assert pair > mat
    monkeypatch.setenv("LAST_KCENTER_FORM", "gram")
    assert ws(long_) == pair
    monkeypatch.setenv("LAST_KCENTER_FORM", "rounds")
    assert ws(mixed) <= rounds_bytes(mixed)
    big = np.array([0, 32769], np.int32)                   # past the rounds' 32768 tokens: matrix
    assert L.diverse_select_workspace(1, big.ctypes.data, 256, last.LAST_BF16, last.KCENTER) > 32769 ** 2 * 4


def test_estimated_forms_keep_the_matrix_workspace(monkeypatch):
    """Batches whose form the budgets decide (the rounds outright, or by their
    relevance on the device, or the matrix) all need what the query says, the
    matrix form's size: one byte less is refused."""
    monkeypatch.delenv("LAST_KCENTER_FORM", raising=False)
    L = last.lib()
    for R, N, Dv, keep in ((32, 4096, 3584, 256),      # rounds
                           (32, 2880, 4096, 320),      # by the relevance
                           (64, 576, 4096, 64)):       # matrix
        cv, ck = (np.arange(R + 1) * N).astype(np.int32), (np.arange(R + 1) * keep).astype(np.int32)
        need = L.diverse_select_workspace(R, cv.ctypes.data, Dv, last.LAST_BF16, last.KCENTER)
        assert need == L.diverse_select_similarity_workspace(R, cv.ctypes.data, Dv, last.LAST_BF16)
        assert need > 4 * R * N * N
        assert _select_call(cv, ck, Dv=Dv, ws_bytes=need - 1) == last.LAST_ERR_WORKSPACE


def _two_phase_call(phase, cv, ck, Dv=64, fdtype=last.LAST_BF16, ws_bytes=1 << 40, misalign=0):
    """Status of diverse_select_similarity ("sim") or diverse_select_pick ("pick"); every
    case here must be rejected on the host, so no buffer may change."""
    cv = np.asarray(cv, np.int32)
    ck = None if ck is None else np.asarray(ck, np.int32)
    dev, out, ws = Fake(), Fake(), Fake()
    L = last.lib()
    if phase == "sim":
        st = L.diverse_select_similarity(len(cv) - 1, Dv, fdtype, dev.p + misalign, dev.p, cv.ctypes.data,
                                         ws.p, ws_bytes, None)
    else:
        st = L.diverse_select_pick(len(cv) - 1, Dv, fdtype, dev.p, dev.p, cv.ctypes.data, dev.p,
                                   None if ck is None else ck.ctypes.data, out.p, out.p, out.p, ws.p, ws_bytes,
                                   None)
    assert st != last.LAST_OK
    assert out.untouched() and ws.untouched() and dev.untouched()
    return st


def test_two_phase_select_rejects_what_diverse_select_rejects():
    E, U, W = last.LAST_ERR_INVALID, last.LAST_ERR_UNSUPPORTED, last.LAST_ERR_WORKSPACE
    assert _two_phase_call("pick", [0, 10, 30], [0, 11, 15]) == E     # K_r > N_r
    assert _two_phase_call("pick", [0, 10, 30], None) == E            # no host budgets
    assert _two_phase_call("sim", [0, 10, 30], None, misalign=2) == E  # features not 16-byte aligned
    for ph in ("sim", "pick"):
        assert _two_phase_call(ph, [0, 10, 10], [0, 5, 5]) == E        # N_r = 0
        assert _two_phase_call(ph, [0, 10, 30], [0, 5, 6], Dv=0) == E
        assert _two_phase_call(ph, [0, 10, 30], [0, 5, 6], fdtype=3) == E
        assert _two_phase_call(ph, [0, 131073], [0, 5]) == U
        assert _two_phase_call(ph, [0, 10, 30], [0, 5, 6], Dv=60) == U
        cv = np.array([0, 100, 350], np.int32)
        need = last.lib().diverse_select_similarity_workspace(2, cv.ctypes.data, 64, last.LAST_BF16)
        assert _two_phase_call(ph, cv, [0, 5, 6], ws_bytes=need - 1) == W


def test_gather_rejects_bad_arguments():
    cv = np.array([0, 10, 30], np.int32)
    ck = np.array([0, 4, 6], np.int32)
    dev, out = Fake(), Fake()
    L = last.lib()
    assert L.gather_kept(2, 64, 3, dev.p, dev.p, cv.ctypes.data, dev.p, dev.p, ck.ctypes.data, out.p, None) == last.LAST_ERR_INVALID
    assert L.gather_kept(0, 64, 2, dev.p, dev.p, cv.ctypes.data, dev.p, dev.p, ck.ctypes.data, out.p, None) == last.LAST_ERR_INVALID
    bad = np.array([0, 4, 2], np.int32)
    assert L.gather_kept(2, 64, 2, dev.p, dev.p, cv.ctypes.data, dev.p, dev.p, bad.ctypes.data, out.p, None) == last.LAST_ERR_INVALID
    assert L.gather_kept(2, 64, 2, None, dev.p, cv.ctypes.data, dev.p, dev.p, ck.ctypes.data, out.p, None) == last.LAST_ERR_INVALID
    assert out.untouched()


# ------------------------------------------------- attention sources (Table 4)

def _rows_call(b, cu_rows, row_pos, ws_bytes=1 << 30):
    cr = None if cu_rows is None else np.asarray(cu_rows, np.int32)
    rp = None if row_pos is None else np.asarray(row_pos, np.int32)
    dev, q, k, out, ws = Fake(), Fake(), Fake(), Fake(), Fake()
    st = last.lib().last_rows_scores(ctypes.byref(b), dev.p, None if cr is None else cr.ctypes.data, dev.p,
                                     None if rp is None else rp.ctypes.data, q.p, k.p, out.p, ws.p,
                                     ws_bytes, None)
    assert out.untouched() and ws.untouched()
    return st


def test_rows_reject_bad_row_sets():
    b, keep = _batch(P=(20, 30), N=(10, 12), vis=(2, 3))
    E = last.LAST_ERR_INVALID
    assert _rows_call(b, [0, 1, 2], [1, 29]) == E          # row before the visual span (sees no visual token)
    assert _rows_call(b, [0, 1, 2], [20, 29]) == E         # row past the last token
    assert _rows_call(b, [0, 0, 2], [5, 29]) == E          # a request without rows
    assert _rows_call(b, [0, 2, 3], [5, 19, 30]) == E      # second request: row past its last token
    assert _rows_call(b, None, [5, 29]) == E
    assert _rows_call(b, [0, 1, 2], None) == E
    b.Dh = 96
    assert _rows_call(b, [0, 1, 2], [5, 29]) == last.LAST_ERR_UNSUPPORTED


def test_rows_workspace_query_and_small_workspace():
    b, keep = _batch(P=(20, 30), N=(10, 12), vis=(2, 3))
    L = last.lib()
    one = np.array([0, 1, 2], np.int32), np.array([19, 29], np.int32)
    many = np.array([0, 3, 5], np.int32), np.array([2, 12, 19, 15, 29], np.int32)
    for cr, rp in (one, many):
        need = L.last_rows_scores_workspace(ctypes.byref(b), cr.ctypes.data, rp.ctypes.data)
        assert need > 0
        assert _rows_call(b, cr, rp, ws_bytes=need - 1) == last.LAST_ERR_WORKSPACE
    bad = np.array([0, 3, 5], np.int32), np.array([2, 12, 19, 15, 30], np.int32)
    assert L.last_rows_scores_workspace(ctypes.byref(b), bad[0].ctypes.data, bad[1].ctypes.data) == 0


def test_source_rows_match_golden():
    import json
    gold = json.load(open(os.path.join(ROOT, "tests", "golden", "source_rows.json")))
    for case in gold["cases"]:
        for name, code in gold["sources"].items():
            assert last.source_rows(code, case["q_begin"], case["q_end"]).tolist() == case[name], (name, case)
    for qb, qe, src in ((5, 5, 0), (-1, 3, 1), (0, 4, 9)):
        with pytest.raises(ValueError):
            last.source_rows(src, qb, qe)


# ------------------------------------------------- prefill attention (Sec. 3.3)

def _prefill_call(b, ws_bytes=1 << 34, v_null=False):
    q, k, v, out, sc, ws = Fake(), Fake(), Fake(), Fake(), Fake(), Fake()
    st = last.lib().last_prefill_attention(ctypes.byref(b), q.p, k.p, None if v_null else v.p, out.p, sc.p,
                                           ws.p, ws_bytes, None)
    assert out.untouched() and sc.untouched() and ws.untouched()
    return st


def test_prefill_rejects_bad_calls_on_the_host():
    b, keep = _batch(dtype=last.LAST_BF16)
    L = last.lib()
    need = L.last_prefill_attention_workspace(ctypes.byref(b))
    assert need > 0
    assert _prefill_call(b, ws_bytes=need - 1) == last.LAST_ERR_WORKSPACE
    assert _prefill_call(b, v_null=True) == last.LAST_ERR_INVALID
    b32, keep32 = _batch(dtype=last.LAST_F32)
    assert _prefill_call(b32) == last.LAST_ERR_UNSUPPORTED
    assert L.last_prefill_attention_workspace(ctypes.byref(b32)) == 0
    b.Dh = 96
    assert _prefill_call(b) == last.LAST_ERR_UNSUPPORTED


# ------------------------------------- cloud connector (Sec. 3.2, 3.4 after Eq. 12)

def _connector_call(dtype=last.LAST_BF16, K=5, Dv=128, Dh=192, Do=64, eps=1e-5, ws_bytes=1 << 34, null=None,
                    shift=None):
    bufs = {n: Fake() for n in ("x", "gamma", "beta", "w1", "b1", "w2", "b2", "out", "ws")}
    ptr = {n: b.p for n, b in bufs.items()}
    if null:
        ptr[null] = None
    if shift:
        ptr[shift] += 8
    st = last.lib().last_connector(dtype, K, Dv, Dh, Do, eps, ptr["x"], ptr["gamma"], ptr["beta"], ptr["w1"],
                                   ptr["b1"], ptr["w2"], ptr["b2"], ptr["out"], ptr["ws"], ws_bytes, None)
    assert all(b.untouched() for b in bufs.values())
    return st


def test_connector_workspace_query():
    L = last.lib()
    # xhat [K][Dv] and h [K][Dh] in bf16, each segment 256-byte aligned
    assert L.last_connector_workspace(5, 128, 192) == 1280 + 2048
    assert L.last_connector_workspace(0, 128, 192) == 0
    assert L.last_connector_workspace(-1, 128, 192) == 0
    assert L.last_connector_workspace(4, 0, 64) == 0


def test_connector_rejects_bad_calls_on_the_host():
    I, U, W_ = last.LAST_ERR_INVALID, last.LAST_ERR_UNSUPPORTED, last.LAST_ERR_WORKSPACE
    assert _connector_call(K=-1) == I
    assert _connector_call(K=1 << 31) == I
    assert _connector_call(Do=0) == I
    assert _connector_call(eps=0.0) == I
    assert _connector_call(eps=float("nan")) == I
    assert _connector_call(eps=float("inf")) == I
    assert _connector_call(dtype=7) == I
    assert _connector_call(dtype=last.LAST_F32) == U
    assert _connector_call(Dv=96) == U          # not a multiple of 64
    assert _connector_call(Dh=32) == U
    assert _connector_call(Do=66) == U          # not a multiple of 4
    assert _connector_call(Do=60) == U          # under 64
    for n in ("x", "gamma", "beta", "w1", "b1", "w2", "b2", "out"):
        assert _connector_call(null=n) == I, n
    for n in ("x", "gamma", "beta", "w1", "w2", "b1", "b2", "out"):
        assert _connector_call(shift=n) == I, n
    assert _connector_call(null="ws") == W_
    assert _connector_call(ws_bytes=last.lib().last_connector_workspace(5, 128, 192) - 1) == W_
    # nothing to do: no rows
    assert _connector_call(K=0, null="x") == last.LAST_OK
