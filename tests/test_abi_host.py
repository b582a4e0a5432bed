"""Host-side checks of the C boundary that need no GPU: the library loads, exports every
symbol the header declares, its host helpers agree with the oracle, and argument errors are
reported before anything is enqueued."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from oracle import compactor_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "compactor.h")


@pytest.fixture(scope="module")
def B():
    from paper_2507_08143_amd import compactor
    return compactor


def _declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(compactor_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(B):
    names = _declared_functions()
    assert {"compactor_score", "compactor_select", "compactor_compact", "compactor_compress"} <= set(names)
    for n in names:
        assert hasattr(B._lib, n), "libcompactor.so does not export %s" % n
    assert set(B.EXPORTS) == set(names)


def test_struct_layouts_match_the_header(B):
    # sizes the C compiler gives for the two structs of the header (x86-64 ABI)
    assert C.sizeof(B._Request) == 4 * 8 + 3 * 8 + 4 + 4
    assert C.sizeof(B._Params) == 4 * 4 + 8 + 4 + 4 + 8 + 4 + 4 + 4 + 4 + 8   # incl. 4 bytes of padding


def test_keep_count_matches_oracle(B):
    rng = np.random.default_rng(0)
    for n, r in [(4096, 0.5), (32768, 0.3), (131072, 0.2), (100000, 0.32), (1000, 0.001), (3, 1 / 3),
                 (1, 0.01), (10, 1.0), (0, 0.5)]:
        assert B.compactor_keep_count(n, r) == O.keep_count(n, r)
    for _ in range(2000):
        n = int(rng.integers(1, 200000))
        r = float(np.float32(rng.uniform(1e-4, 1.0)))
        assert B.compactor_keep_count(n, r) == O.keep_count(n, r)


def test_keep_count_against_the_plain_ceiling(B):
    """k = ceil(r N) of the paper's overview, with r the float32 that crosses the boundary: the
    library (and the oracle) shrink the product by 2^-23 before the ceiling.  Decimal ratios whose
    product is an integer on paper then give that integer; for arbitrary float ratios the count is
    the plain ceiling except where the product lies within r N 2^-23 above an integer, and then it
    is one less."""
    import math
    for n, r, want in [(1000, 0.001, 1), (1000, 0.3, 300), (50, 0.1, 5), (10000000, 0.1, 1000000),
                       (32768, 0.3, 9831), (49907, 0.39685819, 19806)]:
        assert B.compactor_keep_count(n, r) == want
    rng = np.random.default_rng(3)
    less = 0
    for _ in range(20000):
        n = int(rng.integers(8192, 65537))
        r = float(np.float32(rng.uniform(0.2, 0.6)))
        x = r * n
        plain = max(1, min(n, math.ceil(x)))
        got = B.compactor_keep_count(n, r)
        assert got in (plain, plain - 1)
        if got != plain:
            assert x - math.floor(x) <= x * 2.0 ** -23
            less += 1
    assert less <= 100          # about 0.2 % of arbitrary pairs


def test_calibrated_ratio_matches_oracle(B):
    for nll, a, b, tau in [(1.0, np.log(2.0), 0.0, 0.5), (2.3, 0.7, 0.2, 0.95), (0.4, 3.0, 1.0, 0.9),
                           (1.0, 0.0, 0.0, 0.8), (5.0, 2.0, 0.0, 1.0)]:
        assert abs(B.compactor_calibrated_ratio(nll, a, b, tau) - O.calibrated_ratio(nll, a, b, tau)) < 1e-14
    assert abs(B.compactor_calibrated_ratio(1.0, np.log(2.0), 0.0, 0.5) - np.log2(1.5)) < 1e-14


def _req(B, n=100, ratio=0.5, ptr=0x1000, stride_t=128):
    return B._Request(ptr, 0, ptr, 0, 8 * n * stride_t, n * stride_t, stride_t, n, ratio)


def test_layout_offsets(B):
    p = B._Params(3, 2, 128, 48, 0, 0.0, 0.3, 0, 0, 0, 0, None)
    reqs = (B._Request * 3)(_req(B, 100, 0.5), _req(B, 7, 1.0), _req(B, 1000, 0.25))
    so, ko, kk = (C.c_int64 * 4)(), (C.c_int64 * 4)(), (C.c_int32 * 3)()
    assert B._lib.compactor_layout(C.byref(p), reqs, 3, so, ko, kk) == 0
    assert list(kk) == [50, 7, 250]
    assert list(so) == [0, 600, 642, 6642]
    assert list(ko) == [0, 300, 342, 1842]


def test_argument_errors_are_reported_on_the_host(B):
    good = B._Params(2, 2, 128, 48, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    reqs = (B._Request * 1)(_req(B))
    nbytes = C.c_size_t(0)
    assert B._lib.compactor_workspace_size(C.byref(good), reqs, 1, C.byref(nbytes)) == 0
    assert nbytes.value > 0

    def score(p, r, scores=0x3000, status=0x4000, ws=0x10000, wsb=1 << 40):
        return B._lib.compactor_score(C.byref(p), r, 1, scores, status, ws, wsb, None)

    bad_dim = B._Params(2, 2, 64, 48, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    assert score(bad_dim, reqs) == B.EUNSUPPORTED
    bad_ks = B._Params(2, 2, 128, 40, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    assert score(bad_ks, reqs) == B.EUNSUPPORTED
    no_phi = B._Params(2, 2, 128, 48, 0, 0.0, 0.3, 0, 0, 0, 0, None)
    assert score(no_phi, reqs) == B.EINVAL
    bad_scope = B._Params(2, 2, 128, 48, 0x2000, 0.0, 0.3, 0, 0, 0, 7, None)
    assert score(bad_scope, reqs) == B.EINVAL
    neg_ridge = B._Params(2, 2, 128, 48, 0x2000, -1.0, 0.3, 0, 0, 0, 0, None)
    assert score(neg_ridge, reqs) == B.EINVAL
    assert score(good, (B._Request * 1)(_req(B, ratio=0.0))) == B.EINVAL
    assert score(good, (B._Request * 1)(_req(B, ratio=1.5))) == B.EINVAL
    assert score(good, (B._Request * 1)(_req(B, n=0))) == B.EINVAL
    assert score(good, (B._Request * 1)(_req(B, ptr=0x1004))) == B.EALIGN
    assert score(good, (B._Request * 1)(_req(B, stride_t=132))) == B.EALIGN
    assert score(good, (B._Request * 1)(_req(B, stride_t=64))) == B.EINVAL
    assert score(good, reqs, scores=0) == B.EINVAL
    assert score(good, reqs, ws=0) == B.EWORKSPACE
    assert score(good, reqs, wsb=16) == B.EWORKSPACE
    assert score(good, reqs, ws=0x10010) == B.EALIGN
    assert B._lib.compactor_select(C.byref(good), reqs, 1, 0, 0x3000, 0x4000, 0, 0, None) == B.EINVAL
    assert B._lib.compactor_compact(C.byref(good), reqs, 1, 0x3000, 0x4000, 0, 0x6000, None) == B.EINVAL
    assert B._lib.compactor_compress(C.byref(good), reqs, 1, 0, 0x3000, 0x4000, 0x5000, 0x6000, 0,
                                     0x10000, 1 << 40, None) == B.EINVAL
    assert B.compactor_error_string(B.EWORKSPACE).startswith("workspace")
    assert B.compactor_error_string(0) == "ok"
    assert B.compactor_version().count(".") == 1


def _accepts(B, p, reqs, nbytes, fused=True):
    """Whether a call (compress with its scores in the workspace, or score) takes a workspace of nbytes: the place is
    misaligned, which is found out after the size and before anything is enqueued."""
    args = (C.byref(p), reqs, len(reqs))
    if fused:
        rc = B._lib.compactor_compress(*args, 0, 0x3000, 0x4000, 0x5000, 0x6000, 0x7000, 0x10010, nbytes, None)
    else:
        rc = B._lib.compactor_score(*args, 0x3000, 0x4000, 0x10010, nbytes, None)
    assert rc in (B.EALIGN, B.EWORKSPACE)
    return rc == B.EALIGN


@pytest.mark.parametrize("heads,n,ks", [(600, 64, 48), (600, 256, 48), (700, 64, 48), (800, 64, 16), (640, 128, 48),
                                        (600, 100, 64)])
def test_many_short_heads_fit_the_static_scratch(B, heads, n, ks):
    """Room for the partial Gram matrices that the call's workgroups can leave, and no more: at least 8 tiles of 64 rows
    a workgroup, and a partial for every head and workgroup."""
    p = B._Params(heads // 8, 8, 128, ks, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    reqs = (B._Request * 1)(_req(B, n=n))
    assert _accepts(B, p, reqs, B.STATIC_SCRATCH_BYTES)


def _size(B, p, reqs):
    nbytes = C.c_size_t(0)
    assert B._lib.compactor_workspace_size(C.byref(p), reqs, len(reqs), C.byref(nbytes)) == 0
    return nbytes.value


@pytest.mark.parametrize("heads,ks", [(1, 48), (1, 0), (3, 16), (8, 48), (64, 64), (128, 16), (160, 48), (256, 48), (300, 32), (700, 0)])
@pytest.mark.parametrize("scope", [0, 1])
def test_a_workspace_for_the_longest_context_takes_shorter_ones(B, heads, ks, scope):
    """Half runs, the number of Gram workgroups and of their runs, parts of shares and score workgroups change with the length,
    some of them downwards: no length may need more than is asked for at a greater one."""
    p = B._Params(heads, 1, 128, ks, 0x2000, 1e-4, 0.3, 0, 0, 0, scope, None)
    tiles = sorted(set(list(range(1, 20)) + [int(20 * 1.07 ** i) for i in range(80)] + [255, 256, 257, 511, 512, 513, 2047, 2048, 2049]))
    shortest = []
    for t in reversed(tiles):
        n = 64 * t - (t % 5)
        req = _req(B, n=n)
        req.attn = 0x8000
        reqs = (B._Request * 1)(req)
        size = _size(B, p, reqs)
        shortest.append(min([size] + shortest[-1:]))
        for fused in (True, False):
            assert _accepts(B, p, reqs, shortest[-1], fused), n


@pytest.mark.parametrize("heads,n,ks", [(1, 64, 16), (8, 4096, 48), (1, 32768, 48), (256, 500, 48), (128, 256, 64)])
def test_room_for_half_runs_is_not_demanded(B, heads, n, ks):
    """Runs of 8 tiles, a partial Gram matrix of 10 blocks of 32 x 32 floats for every run and head, two bf16 planes of W^T, a
    histogram of 4096 ints and the scores are enough."""
    p = B._Params(1, heads, 128, ks, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    runs = -(-heads * -(-n // 64) // 8)
    nbytes = 40960 * (runs + heads) + heads * (2 * 2 * 128 * ks + 4 * 4096 + 4 * n)
    assert _accepts(B, p, (B._Request * 1)(_req(B, n=n)), nbytes + 256)
    assert not _accepts(B, p, (B._Request * 1)(_req(B, n=n)), nbytes - 256)


def _pieces(lengths, run):
    """(workgroup, head) pairs that share a tile, runs of `run` tiles."""
    at, pieces = 0, 0
    for t in (-(-n // 64) for n in lengths):
        pieces += (at + t - 1) // run - at // run + 1
        at += t
    return pieces


@pytest.mark.parametrize("lengths,heads", [([500], 304), ([300], 512), ([1000], 256), ([1000], 1024), ([200], 768), ([4096], 384), ([5000], 300),
                                           ([600, 130, 2000], 160), ([64, 900, 64, 1500, 320], 96), ([5000, 65], 256)])
def test_two_gram_workgroups_a_unit_where_they_leave_no_more_partials(B, lengths, heads):
    """From a head a unit on, more than 8 and less than 112 tiles a unit.  What a call demands tells how many workgroups it has."""
    p = B._Params(1, heads, 128, 16, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    reqs = (B._Request * len(lengths))(*[_req(B, n=n) for n in lengths])
    per_head = [n for n in lengths for _ in range(heads)]
    total = sum(-(-n // 64) for n in per_head)
    assert len(per_head) >= 256 and 8 * 256 < total < 112 * 256
    one, two = (max(8, -(-total // w)) for w in (256, 512))
    run = two if _pieces(per_head, two) <= _pieces(per_head, one) else one
    nbytes = 40960 * (-(-total // run) + len(per_head)) + len(per_head) * (2 * 2 * 128 * 16 + 4 * 4096) + 4 * sum(per_head)
    assert _accepts(B, p, reqs, nbytes + 256 * len(lengths)) and not _accepts(B, p, reqs, nbytes - 256)


@pytest.mark.parametrize("heads,n,ks", [(256, 1000, 48), (129, 2000, 64), (240, 1000, 48)])
def test_no_shares_are_asked_for_where_none_are_used(B, heads, n, ks):
    """Above 128 heads whose partials are few at any length up to n: partials of one run or two a unit, or of shorter calls' runs
    and half runs, W^T, histograms and scores."""
    p = B._Params(1, heads, 128, ks, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    tiles = heads * -(-n // 64)
    partials = max(min(-(-tiles // 8), 256 if tiles < 112 * 256 and heads < 256 else 512) + heads, 64 + 128 + 2 * heads)
    assert _size(B, p, (B._Request * 1)(_req(B, n=n))) <= 40960 * partials + heads * (2 * 2 * 128 * ks + 4 * 4096 + 4 * n) + 1024


def test_widened_entry_points_check_their_arguments_on_the_host(B):
    good = B._Params(2, 2, 128, 48, 0x2000, 0.0, 0.3, 0, 0, 0, 0, None)
    reqs = (B._Request * 1)(_req(B, n=100, ratio=0.5))

    # paged compaction: the pool's geometry and the length of each page table
    def paged(pool, tab_len, in_place=0, kept_idx=0x3000):
        tabs = (B._PageTable * 1)(B._PageTable(0x7000, tab_len))
        return B._lib.compactor_compact_paged(C.byref(good), reqs, 1, kept_idx, 0x4000, C.byref(pool),
                                              tabs, in_place, None)

    def pool(k=0x100000, v=0x200000, page_stride=4 * 16 * 128, layer_stride=2 * 16 * 128,
             head_stride=128, slot_stride=2 * 128, page_size=16, num_pages=64):
        return B._PagePool(k, v, page_stride, layer_stride, head_stride, slot_stride, page_size, num_pages)

    assert paged(pool(), 3) == B.EINVAL          # 50 kept rows need 4 pages of 16
    assert paged(pool(), 4, in_place=1) == B.EINVAL  # read in place: all 100 tokens, 7 pages
    assert paged(pool(k=0), 4) == B.EINVAL
    assert paged(pool(page_size=0), 4) == B.EINVAL
    assert paged(pool(num_pages=0), 4) == B.EINVAL
    assert paged(pool(slot_stride=64), 4) == B.EINVAL
    assert paged(pool(page_stride=-8), 4) == B.EINVAL
    assert paged(pool(k=0x100008), 4) == B.EALIGN
    assert paged(pool(head_stride=132), 4) == B.EALIGN
    assert paged(pool(), 4, kept_idx=0) == B.EINVAL
    layer = B._Params(2, 2, 128, 48, 0x2000, 0.0, 0.3, 0, 0, 0, 1, None)
    tabs = (B._PageTable * 1)(B._PageTable(0x7000, 4))       # a head may take 2 * 50 rows: 7 pages
    assert B._lib.compactor_compact_paged(C.byref(layer), reqs, 1, 0x3000, 0x4000, C.byref(pool()),
                                          tabs, 0, None) == B.EINVAL

    # the SRHT builder reads its column list on the host
    signs = (C.c_uint8 * 128)(*([1, 0] * 64))
    cols_t = C.c_int32 * 48

    def srht(ks, cols, phi=0x8000, sg=signs):
        return B._lib.compactor_srht_phi(ks, sg, cols, phi, None)

    ok_cols = cols_t(*range(48))
    assert srht(40, ok_cols) == B.EUNSUPPORTED
    assert srht(48, ok_cols, phi=0) == B.EINVAL
    assert srht(48, ok_cols, phi=0x8004) == B.EALIGN
    assert srht(48, cols_t(*([5] + list(range(1, 48))))) == B.EINVAL     # column 5 twice
    assert srht(48, cols_t(*([128] + list(range(1, 48))))) == B.EINVAL   # out of range
    assert srht(48, cols_t(*([-1] + list(range(1, 48))))) == B.EINVAL
    assert srht(48, None) == B.EINVAL

    # attention scores
    def attn(p, r, out=0x3000, ws=0x10000, wsb=1 << 40):
        return B._lib.compactor_attention_scores(C.byref(p), (B._AttnRequest * 1)(r), 1, out, ws, wsb, None)

    def areq(q=0x1000, k=0x2000, qst=128, kst=128, n=300):
        return B._AttnRequest(q, k, 8 * n * qst, n * qst, qst, 2 * n * kst, n * kst, kst, n)

    def apar(layers=2, kv=2, qh=8, d=128, chunk=256, pool_=7, scale=0.088):
        return B._AttnParams(layers, kv, qh, d, chunk, pool_, scale)

    need = C.c_size_t(0)
    assert B._lib.compactor_attention_workspace_size(C.byref(apar()), (B._AttnRequest * 1)(areq()), 1,
                                                     C.byref(need)) == 0
    assert need.value >= 2 * 2 * 300 * 4 and need.value % 256 == 0
    assert attn(apar(qh=3), areq()) == B.EINVAL           # query heads not a multiple of KV heads
    assert attn(apar(qh=1), areq()) == B.EINVAL
    assert attn(apar(d=64), areq()) == B.EUNSUPPORTED
    assert attn(apar(chunk=128), areq()) == B.EUNSUPPORTED
    assert attn(apar(pool_=4), areq()) == B.EINVAL        # pooling windows are odd
    assert attn(apar(pool_=65), areq()) == B.EINVAL
    assert attn(apar(scale=-1.0), areq()) == B.EINVAL
    assert attn(apar(), areq(n=0)) == B.EINVAL
    assert attn(apar(), areq(q=0)) == B.EINVAL
    assert attn(apar(), areq(qst=64)) == B.EINVAL
    assert attn(apar(), areq(kst=132)) == B.EALIGN
    assert attn(apar(), areq(k=0x2008)) == B.EALIGN
    assert attn(apar(), areq(), out=0) == B.EINVAL
    assert attn(apar(), areq(), ws=0) == B.EWORKSPACE
    assert attn(apar(), areq(), wsb=256) == B.EWORKSPACE
    assert attn(apar(), areq(), ws=0x10010) == B.EALIGN


def test_default_params(B):
    p = B.compactor_default_params(32, 8)
    assert (p.layers, p.kv_heads, p.head_dim, p.sketch_dim) == (32, 8, 128, 48)
    assert abs(p.lambda_blend - 0.3) < 1e-7 and p.ridge_rel == 0.0 and p.group_bytes == 0


def test_binding_checks_what_the_pointers_cannot_say(B):
    """Sizes, types and devices of tensors are invisible to the C boundary: the binding refuses a
    wrong one with a ValueError before any library call (CPU tensors suffice to show it)."""
    import torch
    L, H, n = 2, 2, 64
    k = torch.zeros(L, H, n, 128, dtype=torch.bfloat16)
    v = torch.zeros_like(k)
    phi = torch.zeros(128, 48)
    p = B.Params(L, H, phi=phi)
    ok = [B.Request(k_score=k, v_cache=v, ratio=0.5)]
    so, ko, kk = B.compactor_layout(p, ok)                 # host helpers take CPU tensors
    assert (so, ko, kk) == ([0, L * H * n], [0, L * H * 32], [32])
    assert B.compactor_workspace_size(p, ok) > 0

    def refused(fn, needle):
        with pytest.raises(ValueError) as e:
            fn()
        assert needle in str(e.value), str(e.value)

    refused(lambda: B.compactor_layout(p, []), "at least one request")
    refused(lambda: B.compactor_layout(p, [B.Request(k.float(), v, 0.5)]), "bfloat16")
    refused(lambda: B.compactor_layout(p, [B.Request(k, v[:, :, :32], 0.5)]), "v_cache")
    refused(lambda: B.compactor_layout(p, [B.Request(k[:1], v[:1], 0.5)]), "the parameters say")
    refused(lambda: B.compactor_layout(p, [B.Request(k.transpose(2, 3), v.transpose(2, 3), 0.5)]), "d contiguous")
    refused(lambda: B.compactor_layout(B.Params(L, H, phi=torch.zeros(128, 32)), ok), "phi must have shape")
    refused(lambda: B.compactor_layout(p, [B.Request(k, v, 0.5, attn=torch.zeros(L * H * n - 1))]), "attn")
    # entry points that launch refuse CPU tensors and short or mistyped outputs
    refused(lambda: B.compactor_compress(p, ok, kept_idx=torch.zeros(5, dtype=torch.int32)), "GPU")
    refused(lambda: B.compactor_select(p, ok, torch.zeros(L * H * n), kept_idx=torch.zeros(3, dtype=torch.int32),
                                       kept_cnt=torch.zeros(L * H, dtype=torch.int32),
                                       workspace=torch.zeros(256, dtype=torch.uint8)), "GPU")
    aq = torch.zeros(L, 4 * H, n, 128, dtype=torch.bfloat16)
    ap = B.AttnParams(L, H, 4 * H)
    refused(lambda: B.compactor_attention_workspace_size(ap, [B.AttnRequest(aq[:, :3], k)]), "do not match")
    refused(lambda: B.compactor_attention_workspace_size(ap, [B.AttnRequest(aq[:, :, :10], k)]), "same tokens")
