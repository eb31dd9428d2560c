"""Host-side checks of the C ABI that need no GPU: exported symbols, argument validation, planning."""
import ctypes as C
import os
import re

import pytest

from paper_2509_11254_amd import psgd

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    return psgd.load_library()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "psgd.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(psgd_[a-z_]+)\s*\(", header))
    assert declared, "no declarations found"
    assert declared == set(psgd.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def _init(lib, layers, n_workers=1, opt=None):
    descs = (psgd.LayerDesc * max(1, len(layers)))()
    for i, l in enumerate(layers):
        descs[i].rows, descs[i].cols, descs[i].ld, descs[i].r, descs[i].grad_dtype = l
    ctx = C.c_void_p()
    rc = lib.psgd_init(C.byref(ctx), len(layers), descs, n_workers, opt)
    return rc, ctx


def test_init_rejects_bad_arguments(lib):
    ok = (256, 128, 0, 4, psgd.PSGD_F32)
    rc, ctx = _init(lib, [ok])
    assert rc == psgd.PSGD_OK and ctx
    lib.psgd_destroy(ctx)
    assert _init(lib, [ok], n_workers=0)[0] == psgd.PSGD_E_INVALID_ARG
    assert _init(lib, [])[0] == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_init(None, 1, None, 1, None) == psgd.PSGD_E_INVALID_ARG
    assert _init(lib, [(256, 128, 0, 0, psgd.PSGD_F32)])[0] == psgd.PSGD_E_SHAPE       # r < 1
    assert _init(lib, [(256, 128, 0, 129, psgd.PSGD_F32)])[0] == psgd.PSGD_E_SHAPE     # r > n
    assert _init(lib, [(128, 256, 0, 129, psgd.PSGD_F32)])[0] == psgd.PSGD_E_SHAPE     # r > n (transposed)
    assert _init(lib, [(0, 128, 0, 4, psgd.PSGD_F32)])[0] == psgd.PSGD_E_SHAPE         # empty matrix
    assert _init(lib, [(256, 128, 0, 4, 7)])[0] == psgd.PSGD_E_INVALID_ARG             # dtype
    assert _init(lib, [(256, 128, 120, 4, psgd.PSGD_F32)])[0] == psgd.PSGD_E_ALIGN     # ld < cols
    assert _init(lib, [(256, 130, 0, 4, psgd.PSGD_F32)])[0] == psgd.PSGD_E_ALIGN       # ld = cols not multiple of 8
    assert _init(lib, [(256, 130, 136, 4, psgd.PSGD_F32)])[0] == psgd.PSGD_OK          # padded ld is fine
    assert _init(lib, [(4096, 4096, 0, 190, psgd.PSGD_F32)])[0] == psgd.PSGD_E_SHAPE   # block wider than supported
    # leading dimensions beyond what the kernels' 32-bit lane offsets cover (127 rows * ld * 4 bytes < 2^32)
    assert _init(lib, [(256, 128, (1 << 23) + 8, 4, psgd.PSGD_F32)])[0] == psgd.PSGD_E_SHAPE
    assert _init(lib, [(256, 128, 1 << 23, 4, psgd.PSGD_F32)])[0] == psgd.PSGD_OK
    # the refresh's iteration budget has eight bits in the launches' gate word
    for iters, want in ((255, psgd.PSGD_OK), (256, psgd.PSGD_E_INVALID_ARG), (-1, psgd.PSGD_E_INVALID_ARG)):
        opt = psgd.Options(iters, -1, 1, 1, 0.0, 0, 0, 0, 0, 0)
        rc, ctx = _init(lib, [ok], opt=C.byref(opt))
        assert rc == want, iters
        if rc == psgd.PSGD_OK:
            lib.psgd_destroy(ctx)
    for code in (0, -1, -2, -3, -4, -5, -6, -7, -99):
        assert lib.psgd_strerror(code)


def test_compute_calls_reject_null_without_touching_a_gpu(lib):
    rc, ctx = _init(lib, [(256, 128, 0, 4, psgd.PSGD_F32)])
    assert rc == 0
    assert lib.psgd_compress(ctx, None, None, None, None, None, None) == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_compress_static(ctx, None, None, None, None, None) == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_compress_refresh(ctx, None, None, None, None, None, None) == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_refresh(ctx, None, None, 0, None, None, None, None) == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_decompress(ctx, None, None, None, None, None, 0) == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_status(ctx, None, None, 0, None) == psgd.PSGD_E_INVALID_ARG
    assert lib.psgd_copy_bytes(None, None, None, 16) == psgd.PSGD_E_INVALID_ARG
    lib.psgd_destroy(ctx)


def test_workspace_and_algorithmic_bytes(lib):
    rc, ctx = _init(lib, [(4096, 4096, 0, 8, psgd.PSGD_F32)], n_workers=8)
    assert rc == 0
    ws = lib.psgd_workspace_bytes(ctx)
    assert 0 < ws < 1 << 30
    # 8 fp32 gradients + E read, M written and read, E written: 48 bytes per element (+ thin matrices)
    elems = 4096 * 4096
    thin = 16 * (4096 + 4096) * 8
    assert lib.psgd_algorithmic_bytes(ctx) == pytest.approx(elems * 48 + thin)
    lib.psgd_destroy(ctx)
    # one bf16 gradient: forming M twice (2*2 + 12 = 16 bytes) beats storing it (2 + 16)
    rc, ctx = _init(lib, [(11008, 4096, 0, 64, psgd.PSGD_BF16)], n_workers=1)
    assert rc == 0
    assert lib.psgd_algorithmic_bytes(ctx) == pytest.approx(11008 * 4096 * 16 + 16 * (11008 + 4096) * 64)
    lib.psgd_destroy(ctx)
    rc1, c1 = _init(lib, [(512, 512, 0, 8, 0)])
    rc2, c2 = _init(lib, [(512, 512, 0, 8, 0)] * 3)
    assert lib.psgd_workspace_bytes(c2) > lib.psgd_workspace_bytes(c1)
    lib.psgd_destroy(c1)
    lib.psgd_destroy(c2)


# (layers, workers, oversample, m_policy, lazy_residual): contexts that psgd_compress_static takes with one split of the
# reductions per kind of product
@pytest.mark.parametrize("layers,n,over,policy,lazy", [
    ([(2048, 2048, 0, 48, 1)], 1, -1, 0, 0), ([(4096, 1024, 0, 48, 1)], 1, -1, 0, 0), ([(1024, 2048, 0, 64, 0)], 1, -1, 0, 0),
    ([(1024, 4096, 0, 48, 0)], 1, -1, 0, 0), ([(410, 6794, 6800, 37, 1)], 2, -1, 0, 0), ([(122, 8007, 8008, 47, 0)], 1, 0, 0, 1),
    ([(2246, 2505, 2512, 60, 1)], 4, 0, 2, 0), ([(153, 306, 312, 9, 1), (507, 14397, 14400, 9, 1)], 1, -1, 0, 1),
    ([(1334, 1608, 0, 53, 0)] * 3, 4, -1, 2, 0), ([(222, 1476, 1480, 103, 1)] * 3, 4, -1, 0, 0),
    ([(271, 160, 160, 33, 1), (3450, 3313, 3320, 5, 1)], 1, -1, 0, 1), ([(1195, 3371, 3376, 38, 0)] * 2, 1, -1, 0, 0),
    ([(376, 578, 584, 35, 0), (1051, 5177, 5184, 35, 0), (1051, 5177, 5184, 35, 0)], 1, -1, 2, 0)])
def test_static_workspace_takes(lib, layers, n, over, policy, lazy):
    opt = psgd.Options(0, over, 1, 1, 0.0, 0, policy, 0, lazy, 0)
    rc, ctx = _init(lib, layers, n_workers=n, opt=C.byref(opt))
    assert rc == psgd.PSGD_OK
    assert lib.psgd_workspace_bytes(ctx) <= psgd.STATIC_WORKSPACE_BYTES
    lib.psgd_destroy(ctx)


@pytest.mark.parametrize("r", [24, 64, 192])
def test_a_small_layer_does_not_shrink_the_others_regions(lib, r):
    """Block widths of the subspace iteration are capped by the matrix; a layer's partial sums, Gram and factor matrices have
    to hold its own rank whatever the smallest matrix of the context is."""
    def ws(layers):
        opt = psgd.Options(0, 0, 1, 1, 0.0, 0, 0, 0, 0, 0)
        rc, ctx = _init(lib, layers, opt=C.byref(opt))
        assert rc == psgd.PSGD_OK
        b = lib.psgd_workspace_bytes(ctx)
        lib.psgd_destroy(ctx)
        return b

    big, small = (1024, 512, 0, r, psgd.PSGD_F32), (64, 8, 0, 4, psgd.PSGD_F32)
    assert ws([big, small]) >= ws([big])


def test_struct_layouts_match_the_header(tmp_path):
    """The ctypes mirrors of the ABI structs against the C compiler's view of include/psgd.h: sizes and the offset
    of every field, and the error codes the binding names."""
    import subprocess
    fields = {"psgd_layer_desc": [f[0] for f in psgd.LayerDesc._fields_],
              "psgd_options": [f[0] for f in psgd.Options._fields_],
              "psgd_layer_status": [f[0] for f in psgd.LayerStatus._fields_]}
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "psgd.h"', 'int main(void) {']
    for s, fs in fields.items():
        lines.append('printf("%s %%zu\\n", sizeof(%s));' % (s, s))
        for f in fs:
            lines.append('printf("%s.%s %%zu\\n", offsetof(%s, %s));' % (s, f, s, f))
    lines.append('printf("codes %d %d %d %d %d %d %d\\n", PSGD_E_INVALID_ARG, PSGD_E_SHAPE, PSGD_E_ALIGN, PSGD_E_HIP, '
                 'PSGD_E_NOMEM, PSGD_E_CAPTURE, PSGD_E_TOO_LARGE);')
    lines.append('printf("static_ws %u\\n", (unsigned)PSGD_STATIC_WORKSPACE_BYTES);')
    lines += ['return 0; }']
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    out = dict(l.split(" ", 1) for l in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines())
    mirrors = {"psgd_layer_desc": psgd.LayerDesc, "psgd_options": psgd.Options, "psgd_layer_status": psgd.LayerStatus}
    for s, cls in mirrors.items():
        assert int(out[s]) == C.sizeof(cls), s
        for f in fields[s]:
            assert int(out["%s.%s" % (s, f)]) == getattr(cls, f).offset, (s, f)
    assert [int(x) for x in out["codes"].split()] == [psgd.PSGD_E_INVALID_ARG, psgd.PSGD_E_SHAPE, psgd.PSGD_E_ALIGN,
                                                      psgd.PSGD_E_HIP, psgd.PSGD_E_NOMEM, psgd.PSGD_E_CAPTURE,
                                                      psgd.PSGD_E_TOO_LARGE]
    assert int(out["static_ws"]) == psgd.STATIC_WORKSPACE_BYTES


def test_kernel_bytes_of_a_one_launch_step():
    """256 x 128 fp32, r = 4, four workers: the step's one launch reads four gradients, E and Q and writes E, P~, Q and their operand
    copies (three planes, 32 columns, lengths padded to 128); the same layer with a deferred residual has its passes."""
    comp = psgd.Compressor([(256, 128, 4, psgd.PSGD_F32)], 4, allocate=False)
    matrix, thin, copies = 4 * 256 * 128, 4 * 4, 3 * 2 * 32 * (256 + 128)
    assert comp.kernel_bytes("sweep1") == 6 * matrix + thin * (128 + 256 + 128) + copies
    lazy = psgd.Compressor([(256, 128, 4, psgd.PSGD_F32)], 4, lazy_residual=True, allocate=False)
    assert lazy.kernel_bytes("sweep1") > 6 * matrix and lazy.kernel_bytes("residual") == 0


# M and the thin matrices in 160 KB of LDS to the last bytes: 16 columns of whole 16-byte pieces take up to 384 bytes more than their rows
@pytest.mark.parametrize("rows,cols", [(175, 192), (199, 170), (199, 172), (209, 157), (219, 154), (4, 1905), (1, 2242), (12, 1358)])
def test_the_largest_layers_of_one_launch(rows, cols):
    r = min(4, rows)
    comp = psgd.Compressor([(rows, cols, r, psgd.PSGD_F32, (cols + 7) // 8 * 8)], 1, allocate=False)
    m, n = max(rows, cols), min(rows, cols)
    copies = 3 * 2 * 32 * sum((x + 127) // 128 * 128 for x in (rows, cols))
    assert comp.kernel_bytes("sweep1") == 3 * 4 * rows * cols + 4 * r * (m + 2 * n) + copies
