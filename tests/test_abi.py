"""CPU-only checks of the C-ABI library: it loads and exports every symbol the header declares, and the
pure host functions behave (no GPU compute is called)."""
import os
import re

import pytest

from paper_2007_00784_amd import kfac as K

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    src = open(os.path.join(ROOT, "include", "kfac.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(kfac_[a-z_]+)\s*\(", src)))


def test_header_symbols_all_exported():
    if not os.path.exists(K.LIB_PATH):
        from paper_2007_00784_amd import build
        build.build()
    L = K.lib()
    syms = declared_symbols()
    assert set(syms) == set(K.EXPORTS)
    for s in syms:
        assert hasattr(L, s), s


def test_host_functions():
    assert K.kfac_strerror(0) == "success"
    assert "workspace" in K.kfac_strerror(K.KFAC_EWORKSPACE)
    assert K.kfac_schedule_due(0, 10, 100) == (True, True)
    assert K.kfac_schedule_due(10, 10, 100) == (True, False)
    assert K.kfac_schedule_due(11, 10, 100) == (False, False)
    nf = ne = 0
    for k in range(200):
        f, e = K.kfac_schedule_due(k, 10, 100)
        nf += f
        ne += e
    assert (nf, ne) == (20, 2)
    with pytest.raises(K.KfacError):
        K.kfac_schedule_due(-1, 10, 100)
    # workspace queries are monotone and cover the exact eig requirement
    a = K.kfac_workspace_bytes(577, 4, 131072)
    b = K.kfac_workspace_bytes(4609, 4, 131072)
    assert 0 < a < b
    assert K.kfac_eig_workspace_bytes([577, 64, 577, 16]) <= a
    assert K.kfac_eig_workspace_bytes([0]) == 0
    assert K.kfac_workspace_bytes(100000, 1, 1) == 0


def test_workspace_query_covers_every_operand_form():
    """kfac_workspace_bytes(max_d, 1, max_R) suffices for one factor update of that size whatever the layout and
    element type of its samples (the split plans differ between the operand forms)."""
    for d in (64, 257, 1153, 4609):
        for R in (1568, 25088, 401408):
            cap = K.kfac_workspace_bytes(d, 1, R)
            assert cap > 0
            for dtype in (K.KFAC_F32, K.KFAC_BF16):
                for T in (1, 4, 5, 8, 9, 49, 196, R):
                    N = max(1, R // T)
                    for layout in (K.KFAC_LAYOUT_RD, K.KFAC_LAYOUT_NDT):
                        it = dict(X=None, dtype=dtype, layout=layout, N=N, d=d - 1, T=T, append_ones=1, scale=1.0, decay=0.0, F=None)
                        need = K.kfac_update_factors_workspace_bytes([it])
                        assert 0 < need <= cap, (d, R, dtype, T, layout, need, cap)


def test_eig_workspace_of_many_small_factors():
    """What small factors take in the workspace follows their size: about 16 n^2 bytes of matrices and some vectors, not
    the tiles that the wide ones are cut into (which was half a megabyte for a factor of 8 as for one of 128)."""
    for n in (1, 8, 16, 33, 64):
        one = K.kfac_eig_workspace_bytes([n])
        assert one <= 16 * (n + 16) ** 2 + 1700 * n + 8192, (n, one)
        assert K.kfac_eig_workspace_bytes([n] * 1000) <= 1000 * one


def test_eig_workspace_that_was_sized_before_still_holds_a_direct_decomposition():
    """A program may keep the size of its workspace, and a call that is 256 bytes short is served by Jacobi sweeps, several times slower: the
    sizes as they were when the direct decomposition came (lists where a few bytes more in a factor's descriptor showed)."""
    assert K.kfac_eig_workspace_bytes([577, 64] * 9) <= 79068416
    assert K.kfac_eig_workspace_bytes([4, 52, 9, 4, 118, 71, 16, 1, 16, 9, 94, 5, 1, 1915, 15, 46, 2, 95, 1, 886, 98, 116, 71, 8, 1, 242, 13, 288, 239, 71]) <= 91162368


@pytest.mark.parametrize("bf16", [False, True])
def test_factor_workspace_does_not_depend_on_the_order_of_the_list(bf16):
    """Nor does the plan: convolutions and a Linear layer as backward hooks deliver them (last layer first) and as the forward pass does, and
    convolutions of both types in one list."""
    dtype = K.KFAC_BF16 if bf16 else K.KFAC_F32
    conv = lambda d, T, t=dtype: dict(X=None, dtype=t, layout=K.KFAC_LAYOUT_NDT, N=32, d=d, T=T, append_ones=1, F=None)
    fc = dict(X=None, dtype=dtype, layout=K.KFAC_LAYOUT_RD, N=32, d=2048, T=1, append_ones=1, F=None)
    convs = [conv(64, 3136), conv(576, 3136), conv(256, 3136), conv(1152, 784), conv(512, 784), conv(2304, 196), conv(4608, 49)]
    for items in (convs + [fc], convs[:2] + [conv(128, 784, K.KFAC_F32), conv(128, 784, K.KFAC_BF16)] + convs[2:] + [fc]):
        want = K.kfac_update_factors_workspace_bytes(items)
        for k in range(len(items)):
            assert K.kfac_update_factors_workspace_bytes(items[k:] + items[:k]) == want
            assert K.kfac_update_factors_workspace_bytes((items[k:] + items[:k])[::-1]) == want


def test_precondition_workspace_follows_from_the_dimensions():
    """kfac_precondition_workspace_bytes() reads dA and dG only: whatever stands in the other fields, the answer is the same."""
    for dims in ([(145, 16)], [(1153, 128), (577, 64)], [(2401, 2400)], [(4609, 512)] * 8):
        arr = (K.kfac_precond_item * len(dims))()
        for j, (dA, dG) in enumerate(dims):
            arr[j].dA, arr[j].dG = dA, dG
        want = K.kfac_precondition_workspace_bytes(dims)
        for split, dtype in ((1, 0), (0x55555555, -1)):
            arr[-1].split_f16 = arr[-1].factored_damping = split
            arr[-1].grad_dtype = dtype
            assert K.lib().kfac_precondition_workspace_bytes(len(dims), arr) == want, dims


@pytest.mark.parametrize("n,dA,dG,edge", [(1, 145, 16, 64), (1, 3025, 314, 64), (12, 1153, 128, 64), (24, 1153, 128, 128), (26, 384, 384, 128), (20, 496, 280, 128),
                                          (2, 1024, 1024, 64), (3, 1280, 1280, 64), (60, 256, 256, 128), (75, 256, 256, 128), (1, 2401, 2400, 64), (440, 100, 100, 128)])
def test_preconditioning_takes_small_tiles_where_they_are_faster(n, dA, dG, edge):
    """The tables in the workspace have 32 bytes a tile (up to three roundings to 256 of them); with one layer 1 x 1 in the place of each there is one tile each."""
    elements = lambda a, g: 8 * n * ((a * g + 63) // 64 * 64)
    tables = K.kfac_precondition_workspace_bytes([(dA, dG)] * n) - elements(dA, dG)
    ones = K.kfac_precondition_workspace_bytes([(1, 1)] * n) - elements(1, 1)
    tiles = n * ((dA + edge - 1) // edge) * ((dG + edge - 1) // edge)
    assert abs(tables - ones - 32 * (tiles - n)) <= 768, (tables, ones, tiles)
