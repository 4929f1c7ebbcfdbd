"""Host-side checks that need no GPU: the library loads, exports what the
header declares, and rejects bad arguments before anything is launched."""
import ctypes
import os
import re

import pytest

import paper_2605_14844_amd as xfp
from paper_2605_14844_amd.binding import xfp_weights

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x10000          # a non-NULL, 16-byte aligned "device pointer" that is never dereferenced


def declared_functions():
    text = open(os.path.join(ROOT, "include", "xfp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(xfp_[a-z0-9_]+)\s*\(", text)))


def desc(**kw):
    d = xfp_weights()
    d.struct_size = ctypes.sizeof(xfp_weights)
    d.mode, d.bits, d.group, d.N, d.K, d.L, d.E = 0, 4, 128, 64, 256, 0, 1
    d.indices = d.codebooks = d.out_row_ptr = d.out_col = d.out_val = FAKE
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def gemv(d, x=FAKE, M=1, ldx=256, y=FAKE, dt=0, ldy=64):
    return xfp.load_library().xfp_gemv(ctypes.byref(d), x, M, ldx, y, dt, ldy, None)


def moe(d, ids=FAKE, T=2, x=FAKE, xs=0, y=FAKE, dt=0, ldy=64):
    return xfp.load_library().xfp_gemv_moe(ctypes.byref(d), ids, T, x, xs, y, dt, ldy, None)


def test_library_exports_every_declared_symbol():
    lib = xfp.load_library()
    names = declared_functions()
    assert {"xfp_gemv", "xfp_gemv_moe", "xfp_gemv_moe_silu_mul", "xfp_gemv_moe_combine", "xfp_check_contents", "xfp_convert_bf16_to_f16", "xfp_repack_word10", "xfp_unpack_indices", "xfp_dequant_bulk", "xfp_strerror",
            "xfp_version", "xfp_probe_read", "xfp_probe_copy"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    assert xfp.xfp_version() >= 0x100
    assert ctypes.sizeof(xfp_weights) == 104


def test_strerror_texts():
    assert xfp.xfp_strerror(0) == "ok"
    for s in (-1, -2, -3, -4):
        assert xfp.xfp_strerror(s) not in ("ok", "unknown status")
    assert xfp.xfp_strerror(-99) == "unknown status"


def test_null_pointers():
    assert xfp.load_library().xfp_gemv(None, FAKE, 1, 256, FAKE, 0, 64, None) == -1
    assert gemv(desc(indices=None)) == -1
    assert gemv(desc(codebooks=None)) == -1
    assert gemv(desc(out_row_ptr=None)) == -1
    assert gemv(desc(), x=None) == -1
    assert gemv(desc(), y=None) == -1
    assert gemv(desc(mode=1, L=32)) == -1                     # V2a without group ids
    assert moe(desc(E=4), ids=None) == -1
    lib = xfp.load_library()
    assert lib.xfp_unpack_indices(ctypes.byref(desc()), None, None) == -1
    assert lib.xfp_dequant_bulk(ctypes.byref(desc()), None, None) == -1


def test_shape_errors():
    assert gemv(desc(K=200)) == -2                             # K % 128
    assert gemv(desc(N=0)) == -2
    assert gemv(desc(K=0)) == -2
    assert gemv(desc(), M=0) == -2
    assert gemv(desc(), M=-3) == -2
    assert gemv(desc(), ldx=128) == -2                         # ldx < K
    assert gemv(desc(), ldy=10) == -2                          # ldy < N
    assert gemv(desc(E=2)) == -2                               # xfp_gemv takes one matrix
    assert moe(desc(E=4), T=-1) == -2
    assert moe(desc(E=4), xs=64) == -2                         # 0 < stride < K


def test_unsupported_format():
    for bits in (0, 1, 7, 8):
        assert gemv(desc(bits=bits)) == -3
    assert gemv(desc(mode=2)) == -3
    assert gemv(desc(group=64)) == -3
    assert gemv(desc(flags=1)) == -3                           # a scale and mid-point per group: V2a only
    assert gemv(desc(flags=2)) == -3 and gemv(desc(mode=1, L=32, group_ids=FAKE, flags=3, group_scale=FAKE, group_mid=FAKE)) == -3
    assert gemv(desc(mode=1, L=32, group_ids=FAKE, flags=1)) == -1                      # announced but not given
    assert gemv(desc(mode=1, L=32, group_ids=FAKE, flags=1, group_scale=FAKE)) == -1
    assert gemv(desc(mode=1, L=32, group_ids=FAKE, group_scale=FAKE, group_mid=FAKE)) == -3   # given but not announced
    assert gemv(desc(mode=1, L=32, group_ids=FAKE, flags=1, group_scale=FAKE + 1, group_mid=FAKE)) == -4
    assert gemv(desc(struct_size=80)) == -3
    assert gemv(desc(mode=1, L=0, group_ids=FAKE)) == -3
    assert gemv(desc(mode=1, L=300, group_ids=FAKE)) == -3
    assert gemv(desc(L=32)) == -3                              # L given for V2
    assert gemv(desc(), dt=3) == -3                            # bad y dtype (0 fp16, 1 fp32, 2 bf16)
    assert gemv(desc(), dt=0x200) == -3                        # unknown flag (0x100: x is bf16)


def test_rows_no_kernel_can_take_are_rejected_up_front():
    """Longer than the streaming kernel holds, no split into equal slices (a prime number of groups),
    and too long for the general kernel to stage in LDS: refused before anything is launched."""
    assert gemv(desc(K=128 * 1009, bits=3), ldx=128 * 1009) == -3
    assert gemv(desc(K=128 * 1009, bits=2), ldx=128 * 1009) == -3
    assert moe(desc(E=4, K=128 * 1009, bits=3), xs=128 * 1009) == -3
    # the same row at 4 bits (V2) is the tile kernel's, which takes any number of groups
    assert xfp.xfp_route(desc(K=128 * 1009), 1) == (xfp.XFP_ROUTE_TILE, 1)
    assert "too long" in xfp.xfp_strerror(-3) and "bf16" in xfp.xfp_strerror(-3)


def test_ring_slot_arithmetic():
    """Eager calls cycle through slots 0..3, calls recorded into a graph through 4..7; the two never meet,
    and a call takes one slot however many planes it uses (the ticket counter advances once per call)."""
    lib = xfp.load_library()
    lib.xfp_ring_slot.argtypes = [ctypes.c_uint, ctypes.c_int]
    eager = [lib.xfp_ring_slot(t, 0) for t in range(16)]
    rec = [lib.xfp_ring_slot(t, 1) for t in range(16)]
    assert eager == [0, 1, 2, 3] * 4 and rec == [4, 5, 6, 7] * 4
    assert lib.xfp_ring_slot(0xFFFFFFFF, 0) == 3 and lib.xfp_ring_slot(0xFFFFFFFF, 1) == 7     # wrap-around stays in range
    assert not set(eager) & set(rec)


def test_noalloc_entry_point_refuses_what_its_static_array_cannot_hold():
    """Checked on the host before anything is launched (the pointers are fakes)."""
    lib = xfp.load_library()
    call = lambda d, M, ldx: lib.xfp_gemv_noalloc(ctypes.byref(d), FAKE, M, ldx, FAKE, 0, d.N, None)
    assert call(desc(K=65536, bits=2), 2, 65536) == -6             # M >= 2: the re-laid activations hold K <= 32768
    assert call(desc(K=32768, N=300000, bits=3), 1, 32768) == -6   # M = 1 split-K (3 bits): 4 * N floats of partial sums > 2^20
    assert "scratch" in xfp.xfp_strerror(-6)
    assert call(desc(K=200), 1, 256) == -2 and call(desc(bits=9), 1, 256) == -3      # the usual validation comes first
    assert call(desc(E=2), 1, 256) == -2


def test_kernel_selection_takes_only_its_three_values():
    lib = xfp.load_library()
    assert lib.xfp_select_kernel(2) == 0 and lib.xfp_select_kernel(1) == 0 and lib.xfp_select_kernel(0) == 0
    assert lib.xfp_select_kernel(3) == -3 and lib.xfp_select_kernel(-1) == -3


def test_alignment_errors():
    assert gemv(desc(indices=FAKE + 4)) == -4
    assert gemv(desc(codebooks=FAKE + 2)) == -4
    assert gemv(desc(out_row_ptr=FAKE + 2)) == -4
    assert gemv(desc(), x=FAKE + 2) == -4
    assert gemv(desc(), y=FAKE + 8) == -4
    assert gemv(desc(), M=2, ldx=260) == -4
    assert moe(desc(E=4), xs=260) == -4


def test_moe_zero_slots_is_a_no_op():
    assert moe(desc(E=4), T=0, ids=None, x=None, y=None) == 0


def test_binding_rejects_bad_y_dtype_without_touching_the_gpu():
    import torch
    with pytest.raises(xfp.XfpError):
        xfp.binding._y_code(torch.float64)
    with pytest.raises(xfp.XfpError):
        xfp.binding._y_code(torch.float16, torch.zeros(4, dtype=torch.float32))     # x must be fp16 or bf16
    assert xfp.binding._y_code(torch.bfloat16) == xfp.XFP_BF16
    assert xfp.binding._y_code(torch.float32, torch.zeros(4, dtype=torch.bfloat16)) == xfp.XFP_F32 | xfp.XFP_X_BF16


def test_new_entry_points_reject_bad_arguments():
    """Every call below fails validation, so nothing is launched (the pointers are fakes)."""
    lib = xfp.load_library()
    d = desc(E=4)
    silu = lambda dd=d, ids=FAKE, T=2, x=FAKE, xs=0, h=FAKE, dt=0, ldh=32: lib.xfp_gemv_moe_silu_mul(
        ctypes.byref(dd), ids, T, x, xs, h, dt, ldh, None)
    assert silu(dd=desc(E=4, N=63)) == -2                      # N must be even
    assert silu(ldh=31) == -2                                  # ldh < N / 2
    assert silu(ids=None) == -1                                # ids required for a bank of several matrices
    assert silu(h=None) == -1 and silu(x=None) == -1
    assert silu(dt=7) == -3
    assert silu(T=0, ids=None, x=None, h=None) == 0
    comb = lambda ids=FAKE, T=2, x=FAKE, xs=256, w=FAKE, y=FAKE, dt=0: lib.xfp_gemv_moe_combine(
        ctypes.byref(d), ids, T, x, xs, w, y, dt, None)
    assert comb(T=0) == -2 and comb(xs=64) == -2
    assert comb(w=None) == -1 and comb(ids=None) == -1 and comb(y=None) == -1
    assert comb(w=FAKE + 2) == -4 and comb(dt=9) == -3
    cvt = lambda src=FAKE, ld=256, dst=FAKE, rows=2, cols=256: lib.xfp_convert_bf16_to_f16(src, ld, dst, rows, cols, None)
    assert cvt(src=None) == -1 and cvt(dst=None) == -1
    assert cvt(cols=100) == -2 and cvt(ld=128) == -2 and cvt(rows=-1) == -2
    assert cvt(src=FAKE + 2) == -4 and cvt(ld=260) == -4
    assert cvt(rows=0) == 0
    rpw = lambda src=FAKE, rows=4, K=256, bits=5, dst=FAKE: lib.xfp_repack_words(src, rows, K, bits, dst, None)
    assert rpw(bits=7) == -3 and rpw(bits=1) == -3 and rpw(src=None) == -1 and rpw(K=100) == -2 and rpw(rows=0) == 0
    assert rpw(src=FAKE + 2, bits=6) == -4 and rpw(src=FAKE + 1, bits=5) == -4
    rpk = lambda src=FAKE, rows=4, K=256, dst=FAKE: lib.xfp_repack_word10(src, rows, K, dst, None)
    assert rpk(src=None) == -1 and rpk(dst=None) == -1
    assert rpk(K=100) == -2 and rpk(K=0) == -2 and rpk(rows=-1) == -2 and rpk(rows=1 << 40) == -2
    assert rpk(src=FAKE + 2) == -4 and rpk(dst=FAKE + 1) == -4
    assert rpk(rows=0) == 0
    chk = lambda dd=d, cap=10, ids=None, T=0, rep=FAKE: lib.xfp_check_contents(ctypes.byref(dd), cap, ids, T, rep, None)
    assert chk(rep=None) == -1 and chk(cap=-1) == -2 and chk(rep=FAKE + 4) == -4
    assert chk(dd=desc(out_col=None)) == -1                   # entries claimed but no column array


def route(d, M, moe=False):
    return xfp.xfp_route(d, M, moe)


def test_dispatch_rule_on_the_host():
    """xfp_route reports the families by format and size, which is what the decode calls run but where another kernel stands in
    (test_the_launches_of_a_call_are_reported_as_they_run): the five workloads and the configurations bench.py times land on the
    families the design notes name, and the size limits sit where the header says."""
    R = xfp
    v2a = dict(mode=1, L=32, group_ids=FAKE)
    # the five workloads
    assert route(desc(N=512, K=1024), 1) == (R.XFP_ROUTE_STREAM, 1)                       # C1
    assert route(desc(N=8192, K=4096), 1) == (R.XFP_ROUTE_STREAM, 1)                      # C2: 2^25 weights
    assert route(desc(N=4096, K=4096, bits=3, **v2a), 1) == (R.XFP_ROUTE_STREAM, 1)       # C3
    assert route(desc(N=2048, K=4096, bits=3, E=256), 8, moe=True) == (R.XFP_ROUTE_STREAM, 8)   # C4 gate_up
    assert route(desc(N=28672, K=8192), 16) == (R.XFP_ROUTE_BATCH, 16)                    # C5
    # M = 1: the tile kernel from 2^26 weights per call on and for rows beyond 16384 columns (4-bit V2 only)
    assert route(desc(N=16384, K=4096), 1) == (R.XFP_ROUTE_TILE, 1)
    assert route(desc(N=8192, K=28672), 1) == (R.XFP_ROUTE_TILE, 1)
    # 2 .. 16 tokens on rows the 16-token kernel would cut into slices: the wide kernel once its tiles fill the chip
    assert route(desc(N=8192, K=28672), 16) == (R.XFP_ROUTE_WIDE, 16)
    assert route(desc(N=8192, K=28672, bits=3), 5) == (R.XFP_ROUTE_WIDE, 5)
    assert route(desc(N=8160, K=28672), 16) == (R.XFP_ROUTE_BATCH, 16)
    assert route(desc(N=4096, K=16384), 16) == (R.XFP_ROUTE_BATCH, 16)
    assert route(desc(N=64, K=16384 + 128), 1) == (R.XFP_ROUTE_TILE, 1)
    assert route(desc(N=16384, K=4096, bits=3), 1) == (R.XFP_ROUTE_STREAM, 1)
    assert route(desc(N=8192, K=28672, bits=3), 1) == (R.XFP_ROUTE_SPLIT_K, 1)
    assert route(desc(N=2048, K=4096, E=16), 8, moe=True) == (R.XFP_ROUTE_TILE, 8)        # 8 slots x 2^23 weights
    # tokens: 2 .. 16 the batched kernel; more: as many as the wide kernel's copies hold, then the rest
    assert route(desc(N=64, K=8192), 2) == (R.XFP_ROUTE_BATCH, 2)
    assert route(desc(N=64, K=8192), 17) == (R.XFP_ROUTE_WIDE, 17)
    assert route(desc(N=64, K=8192), 64) == (R.XFP_ROUTE_WIDE, 64)
    assert route(desc(N=64, K=8192), 200) == (R.XFP_ROUTE_WIDE, 64)
    assert route(desc(N=64, K=8192 + 128), 64) == (R.XFP_ROUTE_WIDE, 48)                  # 16 * 3 * K <= 2^19 < 16 * 4 * K
    assert route(desc(N=64, K=16384), 64) == (R.XFP_ROUTE_WIDE, 32)
    assert route(desc(N=64, K=16384 + 128), 64) == (R.XFP_ROUTE_BATCH, 16)                # one chunk only: chunks of 16
    assert route(desc(N=64, K=8192, bits=3), 40) == (R.XFP_ROUTE_WIDE, 40)
    assert route(desc(N=64, K=8192, bits=3, **v2a), 40) == (R.XFP_ROUTE_WIDE, 40)
    assert route(desc(N=64, K=8192, bits=2, **v2a), 40) == (R.XFP_ROUTE_WIDE, 40)
    # widths 5 and 6 and tensors with a scale and a mid-point per group: the general kernel, token by token
    assert route(desc(N=64, K=4096, bits=5), 3) == (R.XFP_ROUTE_GENERAL, 3)
    # a scale and a mid-point per group: the streaming kernel's own mode for rows it holds, token by token; else general
    assert route(desc(N=64, K=4096, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 1) == (R.XFP_ROUTE_STREAM, 1)
    assert route(desc(N=64, K=4096, bits=3, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 40) == (R.XFP_ROUTE_STREAM, 40)
    # ... and from 2^27 weights x tokens on through the wide kernel's mode for them, 16 tokens per launch
    assert route(desc(N=4096, K=4096, bits=3, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 8) == (R.XFP_ROUTE_WIDE, 8)
    assert route(desc(N=4096, K=4096, bits=3, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 4) == (R.XFP_ROUTE_STREAM, 4)
    assert route(desc(N=28672, K=8192, bits=3, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 40) == (R.XFP_ROUTE_WIDE, 16)
    assert route(desc(N=28672, K=8192, bits=3, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 1) == (R.XFP_ROUTE_STREAM, 1)
    assert route(desc(N=64, K=20480, flags=1, group_scale=FAKE, group_mid=FAKE, **v2a), 1) == (R.XFP_ROUTE_GENERAL, 1)
    # what xfp_select_kernel changes, xfp_route reports
    xfp.xfp_select_kernel(xfp.XFP_KERNEL_TILE)
    try:
        assert route(desc(N=512, K=1024), 1) == (R.XFP_ROUTE_TILE, 1)
    finally:
        xfp.xfp_select_kernel(xfp.XFP_KERNEL_AUTO)
    # errors come back as the decode calls would raise them
    with pytest.raises(xfp.XfpError) as ei:
        route(desc(K=128 * 1009, bits=3), 1)
    assert ei.value.status == -3
    with pytest.raises(xfp.XfpError):
        route(desc(K=200), 1)


def test_dispatch_invariants_over_random_descriptors():
    """Whatever the descriptor, every launch takes between 1 and the remaining tokens: 2 .. 16 on the batched route,
    2 .. 64 on the wide one, all of them on the M = 1 routes; and walking a call launch by launch terminates."""
    import random
    rnd = random.Random(2605)
    R = xfp
    names = {getattr(R, n) for n in dir(R) if n.startswith("XFP_ROUTE_")}
    for _ in range(3000):
        mode = rnd.choice([0, 0, 1])
        bits = rnd.choice([2, 3, 4, 5, 6]) if mode == 0 else rnd.choice([2, 3, 4])
        kw = dict(N=rnd.choice([1, 31, 32, 33, 4096, 8160, 8161, 8192, 28672, 70000]), K=128 * rnd.choice([1, 2, 7, 8, 63, 64, 65, 128, 129, 224, 256, 257, 512]),
                  bits=bits)
        if mode == 1:
            kw.update(mode=1, L=rnd.choice([1, 32, 64, 65, 256]), group_ids=FAKE)
        d = desc(**kw)
        M = rnd.choice([1, 2, 15, 16, 17, 33, 63, 64, 65, 200])
        left, launches = M, 0
        while left:
            try:
                r, n = xfp.xfp_route(d, left)
            except xfp.XfpError as e:
                assert e.status == -3                         # a row no kernel takes
                break
            assert r in names and 1 <= n <= left, (kw, M, left, r, n)
            if r == R.XFP_ROUTE_BATCH:
                assert 2 <= n <= 16, (kw, M, left, r, n)
            elif r == R.XFP_ROUTE_WIDE:
                assert 2 <= n <= 64, (kw, M, left, r, n)
            else:
                assert n == left, (kw, M, left, r, n)         # the M = 1 kernels take every remaining token as a slot
            left -= n
            launches += 1
            assert launches <= M


def test_prompts_take_the_product_where_it_is_the_faster_one():
    v2a = dict(mode=1, group_ids=FAKE)
    G, Wd = xfp.XFP_ROUTE_GEMM, xfp.XFP_ROUTE_WIDE
    for kw, M, want in [(dict(N=4096, K=4096), 192, (Wd, 64)), (dict(N=4096, K=4096), 193, (G, 193)), (dict(N=127, K=4096), 193, (Wd, 64)),
                        (dict(N=8192, K=8192), 256, (G, 256)), (dict(N=8192, K=8192), 257, (Wd, 64)), (dict(N=8192, K=8192), 512, (G, 512)),
                        (dict(N=28672, K=8192), 383, (Wd, 64)), (dict(N=28672, K=8192), 384, (G, 384)),
                        (dict(N=2048, K=28672), 127, (xfp.XFP_ROUTE_BATCH, 16)), (dict(N=2048, K=28672), 128, (G, 128)),
                        (dict(N=4096, K=4096, L=256, **v2a), 65, (G, 65)), (dict(N=512, K=512, L=32, bits=3, **v2a), 65, (Wd, 64)),
                        (dict(N=4096, K=4096, bits=5), 500, (xfp.XFP_ROUTE_GENERAL, 500))]:
        assert xfp.xfp_route(desc(**kw), M) == want, (kw, M)
    assert xfp.xfp_route(desc(N=130, K=65536, bits=2), 256)[0] == G       # an outlier's column is kept in 16 bits
    assert xfp.xfp_route(desc(N=130, K=65536 + 128, bits=2), 256)[0] != G


def test_a_prompt_launch_takes_what_its_copies_hold():
    """Both copies of the activations hold 2^24 halves: [K][tokens rounded up to 8] and [tokens][K rounded up to 256]."""
    for K in range(128, 65536 + 1, 128):
        most = 2**24 // (-(-K // 256) * 256)
        for M in [m for m in range(most - 9, most + 10) if 512 <= m <= 65535] + [min(65535, 2 * most + 3)]:
            left = M
            while left:
                route, n = xfp.xfp_route(desc(N=16384, K=K, bits=2), left)
                if left == M:
                    assert route == xfp.XFP_ROUTE_GEMM or M < 512, (K, M)
                if route == xfp.XFP_ROUTE_GEMM:
                    assert K * (-(-n // 8) * 8) <= 2**24 and n * (-(-K // 256) * 256) <= 2**24, (K, M, n)
                left -= n


def test_tokens_left_over_by_prompt_launches():
    """What a launch leaves over is planned like a call of its own (also behind passes: a prompt that is one round of tiles and
    a little more is passes, then one round); where no other matrix-core kernel takes it, launches share the tokens."""
    G, Wd, R = xfp.XFP_ROUTE_GEMM, xfp.XFP_ROUTE_WIDE, xfp
    for kw, M, want in [(dict(N=28672, K=8192), 2049, [(G, 2048), (R.XFP_ROUTE_TILE, 1)]),
                        (dict(N=28672, K=8192), 2100, [(G, 2048), (Wd, 52)]),
                        (dict(N=8192, K=8192), 2048 + 300, [(G, 2048), (Wd, 64), (G, 236)]),
                        (dict(N=8192, K=8192), 257, [(Wd, 64), (G, 193)]), (dict(N=8192, K=8192), 320, [(Wd, 64), (G, 256)]),
                        (dict(N=8192, K=8192), 448, [(Wd, 64)] * 3 + [(G, 256)]), (dict(N=28672, K=8192), 257, [(Wd, 64)] * 4 + [(R.XFP_ROUTE_TILE, 1)]),
                        (dict(N=2048, K=28672), 585, [(G, 512), (R.XFP_ROUTE_BATCH, 16)]),
                        (dict(N=130, K=65536, bits=2), 300, [(G, 152), (G, 148)]),
                        (dict(N=4096, K=4096, L=256, mode=1, group_ids=FAKE), 2 * 4096 + 3, [(G, 4096), (G, 2056), (G, 2043)])]:
        left = M
        for step in want:
            assert xfp.xfp_route(desc(**kw), left) == step, (kw, M, left)
            left -= step[1]


def test_more_than_two_dimensions_are_not_tokens():
    """x [2, 1, K] is no matrix of two tokens: one row of two columns, which the library refuses."""
    import torch
    W = type("W", (), {"desc": desc(), "N": 64})
    with pytest.raises(xfp.XfpError) as e:
        xfp.xfp_gemv(W, torch.zeros((2, 1, 256), dtype=torch.float16), stream=0)
    assert e.value.status == -2


@pytest.mark.parametrize("torch_there", [False, True])
def test_the_library_is_built_without_the_extension(torch_there, monkeypatch, tmp_path):
    """A C program's build: no torch, or no compiler or headers for the binding's native half."""
    from paper_2605_14844_amd import build as b

    def run(cmd, verbose, remarks_to=None):
        if b.EXT_SRC in cmd:
            raise RuntimeError("no extension here")
        open(cmd[cmd.index("-o") + 1], "w").close()

    find = b.importlib.util.find_spec
    monkeypatch.setattr(b.importlib.util, "find_spec", lambda name: find(name) if torch_there else None)
    monkeypatch.setattr(b, "sources", lambda: [])
    monkeypatch.setattr(b, "_run", run)
    for name in ("LIB", "EXT", "RESOURCES"):
        monkeypatch.setattr(b, name, str(tmp_path / name))
    if torch_there:
        with pytest.raises(RuntimeError, match="no extension here"):
            b.build()
    else:
        b.build()
    assert os.path.exists(b.LIB) and not os.path.exists(b.EXT)


@pytest.mark.parametrize("other", [bytes(104), (ctypes.c_char * 104)(), None])
def test_only_a_descriptor_is_one(other):
    import torch
    x, ids = torch.zeros((1, 256), dtype=torch.float16), torch.zeros(1, dtype=torch.int32)
    W = type("W", (), {"desc": other, "N": 64})
    for f in (lambda: xfp.xfp_gemv(W, x, stream=0), lambda: xfp.xfp_gemv_moe(W, ids, x, stream=0),
              lambda: xfp.xfp_gemv_moe_silu_mul(W, ids, x, stream=0),
              lambda: xfp.xfp_gemv_moe_combine(W, ids, x, torch.ones(1), stream=0)):
        with pytest.raises(TypeError):
            f()


def test_the_output_type_may_be_left_to_torch():
    """y_dtype=None is torch's default dtype, as in torch.empty: the call gets as far as the library's own refusal."""
    import torch
    W = type("W", (), {"desc": desc(), "N": 64})
    for dtype, status in ((torch.float32, -2), (torch.float64, -3)):      # a row too short; an output of 64 bits
        before = torch.get_default_dtype()
        torch.set_default_dtype(dtype)
        try:
            with pytest.raises(xfp.XfpError) as e:
                xfp.xfp_gemv(W, torch.zeros((1, 128), dtype=torch.float16), y_dtype=None, stream=0)
        finally:
            torch.set_default_dtype(before)
        assert e.value.status == status
    with pytest.raises(TypeError):
        xfp.xfp_gemv_noalloc(W, torch.zeros((1, 128), dtype=torch.float16), None, stream=0)


def launches(kw, M, moe=False):
    """[(route, tokens)] of every launch of a call, as xfp_launch_route reports them."""
    out = []
    while M:
        out.append(xfp.xfp_launch_route(desc(**kw), M, moe))
        M -= out[-1][1]
    return out


def test_the_launches_of_a_call_are_reported_as_they_run():
    """decode() executes the function that xfp_launch_route reports: the resident kernel and the tiled product where they stand in
    for a family of xfp_route, at the limits of either, and for nothing else."""
    R, lib = xfp, dict(mode=1, L=32, group_ids=FAKE)
    record = dict(flags=1, group_scale=FAKE, group_mid=FAKE, **lib)
    Res, G, Wd, B = R.XFP_ROUTE_RESIDENT, R.XFP_ROUTE_GEMM, R.XFP_ROUTE_WIDE, R.XFP_ROUTE_BATCH
    for kw, M, want in [
            # a few tokens: the resident kernel, the others where it would take too many slices of the activations
            (dict(N=7001, K=5504, bits=2), 5, [(Res, 5)]), (dict(N=28672, K=8192), 16, [(B, 16)]), (dict(N=4096, K=4096, **record), 24, [(Res, 24)]),
            (dict(N=28672, K=8192, bits=3, **record), 16, [(Wd, 16)]),
            # 5 and 6 bits: as many as fit in one slice
            (dict(N=8192, K=4096, bits=5), 16, [(Res, 8), (Res, 8)]), (dict(N=617, K=14208, bits=5), 2, [(R.XFP_ROUTE_GENERAL, 2)]),
            # a token of long rows
            (dict(N=8192, K=28672, bits=3, **lib), 1, [(Res, 1)]), (dict(N=8192, K=28672, bits=3), 1, [(R.XFP_ROUTE_SPLIT_K, 1)]),
            # the tiled product: from 80 tokens on, 65 for long rows, 128 for few long rows, not for two passes more than a round
            (dict(N=4096, K=4096), 79, [(Wd, 64), (Res, 15)]), (dict(N=4096, K=4096), 80, [(G, 80)]), (dict(N=4096, K=4096), 96, [(G, 96)]),
            (dict(N=8192, K=8192), 65, [(Wd, 64), (R.XFP_ROUTE_TILE, 1)]), (dict(N=4096, K=14336), 64, [(Wd, 32), (Wd, 32)]),
            (dict(N=4096, K=14336), 65, [(G, 65)]), (dict(N=512, K=8192), 127, [(Res, 64), (Res, 63)]), (dict(N=512, K=8192), 128, [(G, 128)]),
            (dict(N=8192, K=8192), 320, [(Wd, 64), (G, 256)]), (dict(N=40, K=4096), 130, [(Res, 64), (Res, 64), (Res, 2)])]:
        assert launches(kw, M) == want, (kw, M)
    assert launches(dict(N=2048, K=4096, bits=3, E=16), 8, moe=True) == [(R.XFP_ROUTE_STREAM, 8)]


def test_what_stands_in_for_a_planned_launch():
    """Over random descriptors: the resident kernel takes up to 64 tokens of the call, of a row it can hold; the product more
    than 64; every other launch is the planned one; expert-indexed calls are as planned."""
    import random
    rnd = random.Random(14844)
    R, seen = xfp, set()
    for _ in range(3000):
        kw = dict(N=rnd.choice([1, 33, 640, 1100, 4096, 8160, 8161, 28672, 70000]), K=128 * rnd.choice([1, 9, 32, 64, 65, 85, 128, 129, 167, 224, 512, 520]),
                  bits=rnd.choice([2, 3, 4]))
        kw.update(rnd.choice([{}, dict(mode=1, L=32, group_ids=FAKE), dict(mode=1, L=32, group_ids=FAKE, flags=1, group_scale=FAKE, group_mid=FAKE),
                              dict(bits=5), dict(bits=6)]))
        M = rnd.choice([1, 2, 5, 16, 17, 40, 64, 65, 79, 80, 128, 192, 321])
        try:
            planned = xfp.xfp_route(desc(**kw), M)
        except xfp.XfpError as e:
            with pytest.raises(xfp.XfpError) as ei:
                xfp.xfp_launch_route(desc(**kw), M)
            assert ei.value.status == e.status == -3
            continue
        r, n = xfp.xfp_launch_route(desc(**kw), M)
        seen.add(r)
        assert 1 <= n <= M, (kw, M, r, n)
        if r == R.XFP_ROUTE_RESIDENT:
            assert n <= 64 and kw["K"] <= 65536 and planned[0] in (R.XFP_ROUTE_STREAM, R.XFP_ROUTE_SPLIT_K, R.XFP_ROUTE_BATCH, R.XFP_ROUTE_WIDE,
                                                                   R.XFP_ROUTE_GENERAL), (kw, M, n)
        elif (r, n) != planned:
            assert r == R.XFP_ROUTE_GEMM and n > 64 and planned[0] in (R.XFP_ROUTE_BATCH, R.XFP_ROUTE_WIDE), (kw, M, n)
        assert xfp.xfp_launch_route(desc(**kw), M, True) == xfp.xfp_route(desc(**kw), M, True)
    assert seen == set(range(8))


def test_the_tile_of_a_wide_launch_is_reported():
    """Two kernels run XFP_ROUTE_WIDE launches; the tile tells them apart: 32 rows and as many chunks of 16 tokens as there are, or
    128 rows and 32 or 64 tokens."""
    R, lib = xfp, dict(mode=1, L=32, group_ids=FAKE)
    record = dict(flags=1, group_scale=FAKE, group_mid=FAKE, **lib)
    tile = lambda M, **kw: R.xfp_wide_tile(desc(**kw), M)
    for kw in (dict(), dict(bits=3), dict(bits=2, **lib)):
        assert [tile(M, N=28672, K=8192, **kw) for M in (16, 17, 32, 33, 64)] == [(32, 16), (128, 32), (128, 32), (128, 64), (128, 64)]
        assert [tile(M, N=14336, K=8192, **kw) for M in (2, 17, 33, 49, 64)] == [(32, 16), (32, 32), (32, 48), (32, 64), (32, 64)]
    assert tile(16, N=28672, K=8192, **record) == (32, 16)
    assert tile(2, N=8192, K=28672) == (32, 16)
    for M, kw, status in [(33, dict(N=28672, K=16384), -3), (17, dict(N=28672, K=8192, **record), -3), (20, dict(N=28672, K=4096, bits=5), -3),
                          (20, dict(N=28672, K=4096, mode=1, L=65, group_ids=FAKE), -3), (65, dict(N=28672, K=4096), -2), (0, dict(N=28672, K=4096), -2),
                          (20, dict(N=28672, K=4096, E=2), -2), (20, dict(N=28672, K=100), -2)]:
        with pytest.raises(R.XfpError) as e:
            tile(M, **kw)
        assert e.value.status == status, (M, kw)
    assert R.load_library().xfp_wide_tile(ctypes.byref(desc(N=28672, K=4096)), 20, None) == -1


@pytest.mark.parametrize("lib", [False, True])
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_the_lines_of_the_tall_matrix_rule(bits, lib):
    """Tiles of 128 rows where they fill more of the last round of 256 than the 64-token kernel is the faster one at: the first matrix above
    a line, the last below it."""
    fmt = dict(mode=1, L=32, group_ids=FAKE) if lib else {}
    rows = lambda M, N, K: xfp.xfp_wide_tile(desc(N=N, K=K, bits=bits, **fmt), M)[0]
    lib3 = lib and bits == 3
    for M, K, one, many in [(17, 4096, 12, 15 if bits == 4 else 14), (32, 128, 12, 15 if bits == 4 else 14), (33, 512, 8, 11), (64, 128, 8, 11),
                            (33, 640, 12 if lib3 else 8, 14 if lib else 12), (64, 1024, 12 if lib3 else 8, 14 if lib else 12),
                            (33, 1152, 12, 16 if lib3 else 15 if bits == 3 or (lib and bits == 4) else 14),
                            (48, 8192, 12, 16 if lib3 else 15 if bits == 3 or (lib and bits == 4) else 14),
                            (49, 1152, 12 if lib and bits >= 3 else 10, 14 if lib else 13), (64, 8192, 12 if lib and bits >= 3 else 10, 14 if lib else 13)]:
        for rounds, line in ((1, one), (2, many), (3, many)):
            last = 128 * 16 * line * rounds                           # rows of the tiles at the line
            assert rows(M, last, K) == 32, (M, K, rounds)
            if line < 16:
                assert rows(M, last + 1, K) == 128 and rows(M, 128 * 256 * rounds, K) == 128, (M, K, rounds)
        assert rows(M, 128 * 256 + 1, K) == 32
    assert rows(16, 28672, 4096) == 32


def shares(M, **kw):
    """(slices, blocks of 16 rows of a workgroup, waves per block, workgroups) of a launch of the resident kernel"""
    out = (ctypes.c_uint * 4)()
    status = xfp.load_library().xfp_resident_shares(ctypes.byref(desc(**kw)), M, out)
    assert status in (0, -3), (kw, M, status)
    return tuple(out) if status == 0 else None


def resident_formats():
    lib = dict(mode=1, L=32, group_ids=FAKE)
    return [dict(bits=b, **f) for b in (2, 3, 4) for f in ({}, lib, dict(lib, flags=1, group_scale=FAKE, group_mid=FAKE))] + [dict(bits=5), dict(bits=6)]


def test_the_resident_kernel_fills_one_round_of_the_cus():
    """One workgroup runs on a CU: one more than the 256 is a second round for nothing, unless workgroups of as many blocks as they
    have waves are still more than 256."""
    for kw in resident_formats():
        for N in (16, 300, 1100, 2048, 4096, 5200, 6000, 8160, 28672):
            for K in (128, 4096, 8192, 8320, 14336, 20480, 28672):
                for M in (1, 2, 6, 8, 12, 16, 30, 40, 64):
                    s = shares(M, N=N, K=K, **kw)
                    if s is None:
                        continue
                    most = 16 if M <= 32 and kw["bits"] <= 4 else 8
                    assert s[1] * s[2] <= most and 16 * s[1] * (s[3] // s[0]) >= N, (kw, N, K, M, s)
                    assert s[3] <= 256 or s[1] == most, (kw, N, K, M, s)
    assert shares(8, N=4096, K=14336) == (3, 4, 4, 192)


def test_slices_are_taken_where_a_workgroup_fills_its_cu():
    """More than two slices only for the rows that take three launches elsewhere, in workgroups of up to eight blocks."""
    R, kw = xfp, dict(N=4096, K=28672)
    assert shares(12, **kw)[:2] == (8, 8) and launches(kw, 12) == [(R.XFP_ROUTE_RESIDENT, 12)]
    assert shares(16, **kw)[:2] == (9, 10) and launches(kw, 16) == [(R.XFP_ROUTE_BATCH, 16)]
    assert launches(dict(N=3000, K=28672), 16) == [(R.XFP_ROUTE_BATCH, 16)]
    assert launches(dict(N=300, K=28672), 16) == [(R.XFP_ROUTE_RESIDENT, 16)] and launches(dict(N=4096, K=8192), 16) == [(R.XFP_ROUTE_BATCH, 16)]
    for kw in resident_formats()[:9]:
        for N in (100, 2048, 4096, 6000, 8160, 8161):
            for K in (4096, 5120, 8192, 8320, 14336, 28672):
                for M in (2, 5, 9, 16):
                    if launches(dict(kw, N=N, K=K), M)[0][0] == R.XFP_ROUTE_RESIDENT:
                        s = shares(M, N=N, K=K, **kw)
                        assert s[0] <= 2 or (s[1] <= 8 and K > 8192 and N <= 8160), (kw, N, K, M, s)


def test_short_rows_are_staged_by_more_waves_than_they_have_units():
    """A unit is 128 columns (256 at 2 bits): with one to three of them a wave per unit left the staging of up to 64 tokens, the
    outliers and the sums to one to three waves."""
    for kw in resident_formats():
        unit = 256 if kw["bits"] == 2 else 128
        for N in (16, 1000, 4096, 4112, 8000):
            for units in (1, 2, 3, 4, 6):
                for M in (2, 16, 17, 32, 33, 64):
                    s = shares(M, N=N, K=unit * units, **kw)
                    most = 16 if M <= 32 and kw["bits"] <= 4 else 8
                    if s[0] > 1:
                        continue
                    want = units if units >= 4 or (N > 4096 and M <= 16) else max(units, 8)
                    assert s[2] == min(most // s[1], want), (kw, N, units, M, s)
    assert shares(30, N=335, K=256, bits=2) == (1, 1, 8, 21)


def test_few_rows_with_records_stay_token_by_token():
    """A scale and a mid-point per group: with up to 640 rows (1008 for 2 to 8 tokens and for more than 32 of rows that are not
    short, more for 2 to 5) the streaming kernel runs all tokens side by side in less time than the resident kernel stages them."""
    R, record = xfp, dict(mode=1, L=32, group_ids=FAKE, flags=1, group_scale=FAKE, group_mid=FAKE)
    stream, res = R.XFP_ROUTE_STREAM, R.XFP_ROUTE_RESIDENT
    for bits, N, K, M, want in [(2, 73, 256, 45, stream), (3, 640, 2048, 20, stream), (3, 641, 2048, 20, res), (3, 641, 2048, 40, stream), (3, 641, 1152, 40, res),
                                (3, 1008, 2048, 8, stream), (3, 1009, 2048, 8, res), (3, 1024, 1024, 5, stream), (3, 3072, 1024, 2, stream),
                                (3, 3073, 1024, 2, res), (4, 2048, 1024, 2, stream), (4, 2049, 1024, 2, res), (4, 1008, 128, 2, stream)]:
        assert launches(dict(record, bits=bits, N=N, K=K), M)[0][0] == want, (bits, N, K, M)
    # rows that the streaming kernel does not hold: sixteen tokens at a time or one wave per row and token elsewhere
    assert launches(dict(record, bits=3, N=600, K=20480), 16) == [(res, 16)]


def test_few_long_rows_at_5_and_6_bits_stay_token_by_token():
    """In one slice the resident kernel takes a few tokens of long rows per launch, on as many CUs as there are blocks of 16 rows:
    few rows are faster in the general kernel, which runs all tokens side by side."""
    R = xfp
    for bits in (5, 6):
        for N, K, M, want in [(1024, 23424, 42, R.XFP_ROUTE_GENERAL), (2048, 8320, 64, R.XFP_ROUTE_GENERAL), (2049, 8320, 64, R.XFP_ROUTE_RESIDENT),
                              (1280, 5632, 20, R.XFP_ROUTE_GENERAL), (1281, 5632, 20, R.XFP_ROUTE_RESIDENT), (1280, 5504, 20, R.XFP_ROUTE_RESIDENT),
                              (896, 3072, 64, R.XFP_ROUTE_GENERAL), (897, 3072, 64, R.XFP_ROUTE_RESIDENT), (896, 2944, 64, R.XFP_ROUTE_RESIDENT)]:
            assert launches(dict(bits=bits, N=N, K=K), M)[0][0] == want, (bits, N, K, M)


def test_a_little_more_than_a_round_of_tiles_is_passes_first():
    """Up to 192 tokens in 257 to 384 tiles of 128 x 64: a second round that is mostly empty costs more than a pass of 64 tokens."""
    R, lib = xfp, dict(mode=1, L=32, group_ids=FAKE)
    G, Wd = R.XFP_ROUTE_GEMM, R.XFP_ROUTE_WIDE
    first = lambda M, **kw: launches(kw, M)[0]
    # 3 and 4 bits, 3072 to 8192 columns: whatever is left behind the passes
    for kw in (dict(bits=4), dict(bits=3), dict(bits=3, **lib)):
        assert first(128, N=128 * 128, K=4096, **kw) == (G, 128) and first(128, N=128 * 128 + 1, K=4096, **kw) == (Wd, 64)
        assert first(128, N=192 * 128, K=4096, **kw) == (Wd, 64) and first(128, N=192 * 128 + 1, K=4096, **kw) == (G, 128)
        assert first(128, N=20000, K=2944, **kw) == (G, 128) and first(128, N=20000, K=8320, **kw) == (G, 128)
    # all widths: where no more than 32 tokens are left, rows that are not short
    for bits in (2, 3, 4):
        assert first(96, N=20000, K=640, bits=bits) == (Wd, 64) and first(96, N=20000, K=512, bits=bits) == (G, 96)
        assert first(97, N=20000, K=640, bits=bits) == (G, 97)
        assert first(160, N=12000, K=1536, bits=bits) == (Wd, 64) and first(160, N=12000, K=1408, bits=bits) == (G, 160)
        assert (first(65, N=21000, K=9344, bits=bits)[0] == G) == (bits == 2)
    # more than 192 tokens: as before
    assert first(193, N=11000, K=4096) == (G, 193)


def test_the_16_token_kernel_has_every_row_length_that_reaches_it():
    """It is built for rows of more than 2048 columns and, in slices, of more than 10240: shorter ones are the resident kernel's at
    any number of rows and tokens, whatever room the library takes."""
    rows = [1, 16, 500, 1009, 2049, 4096, 4097, 6000, 8160, 8161, 12288, 16384, 20480, 24576, 28672, 32768, 32769, 45056, 61440, 65536, 128256, 1000000]
    for bits in (2, 3, 4):
        for L in (0, 1, 32, 64, 128, 256):
            fmt = dict(mode=1, L=L, group_ids=FAKE) if L else {}
            for G in list(range(1, 17)) + list(range(65, 81)):
                for N in rows:
                    for M in (2, 5, 8, 12, 15, 16, 17, 33, 64, 70):
                        r, _ = xfp.xfp_launch_route(desc(bits=bits, N=N, K=128 * G, **fmt), M)
                        assert r != xfp.XFP_ROUTE_BATCH, (bits, L, G, N, M)


def test_one_token_of_long_library_rows():
    """Rows that the streaming kernel takes in slices are the resident kernel's where the matrix keeps all CUs busy in one round of blocks
    or nearly: fewer rows the fewer bits an index has."""
    R, lib = xfp, dict(mode=1, L=32, group_ids=FAKE)
    record = dict(lib, flags=1, group_scale=FAKE, group_mid=FAKE)
    for kw, N in [(dict(lib, bits=4), 5632), (dict(lib, bits=3), 4864), (dict(lib, bits=2), 4096)]:
        assert launches(dict(kw, N=N, K=21504), 1) == [(R.XFP_ROUTE_RESIDENT, 1)] and launches(dict(kw, N=N - 1, K=21504), 1) == [(R.XFP_ROUTE_SPLIT_K, 1)], kw
    # with records, and rows without equal slices: one wave per row of the general kernel otherwise
    for kw in (dict(record, bits=4), dict(lib, bits=4, K=21376)):
        assert launches(dict(dict(K=21504), N=2048, **kw), 1) == [(R.XFP_ROUTE_RESIDENT, 1)] and launches(dict(dict(K=21504), N=2047, **kw), 1) == [(R.XFP_ROUTE_GENERAL, 1)], kw
