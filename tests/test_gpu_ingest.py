"""The handle's copy and check of the caller's CSR at its edges (entries in
fours and their remainder, arrays off 16-byte alignment, row starts where the
columns do and do not descend), and the feature pass on groups of rows around
the length from which whole workgroups run a row."""
import numpy as np
import pytest

from helpers import say
from synth import matrices as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ck():
    import paper_2411_10143_amd as ck
    return ck


def _rows(lengths, ncols, seed):
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    col = np.concatenate([np.sort(rng.choice(ncols, r, replace=False)) for r in lengths]
                         + [np.zeros(0)]).astype(np.int32)
    val = rng.integers(1, 9, rp[-1]).astype(np.float64)
    return M.CSR(len(lengths), ncols, rp, col, val, "edge").check()


def _shifted(a, off):
    """The array on the device, `off` entries past an allocation's start."""
    import torch
    t = torch.zeros(len(a) + off, dtype=torch.from_numpy(a[:0]).dtype, device="cuda")
    t[off:] = torch.from_numpy(a).cuda()
    return t[off:]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("offs", [(0, 0, 0), (1, 1, 1), (0, 4, 1), (3, 0, 2)])
@pytest.mark.parametrize("lengths", [[1], [0, 0, 3, 0], [2, 2, 0], [1] * 5, [7] * 40 + [0, 3],
                                     [0] * 300 + [1500, 0, 1], [33] * 997],
                         ids=["1", "3", "4", "5", "283", "1501", "32901"])
def test_copy_is_exact(ck, lengths, offs, fp32):
    """Whole numbers: every product is exact, in FP64 and in FP32."""
    import torch
    A = _rows(lengths, 2000, 3)
    say(f"copy nnz {len(A.col)} offsets {offs} fp32 {fp32}")
    rp, col, val = (_shifted(a, o) for a, o in zip((A.rp, A.col, A.val), offs))
    Mx = ck.Matrix(rp, col, val, ncols=A.ncols, keep_fp32=fp32)
    rp.zero_()
    col.zero_()
    val.zero_()                       # the handle holds its own copy
    x = np.arange(1, A.ncols + 1, dtype=np.float64) % 7
    want = np.zeros(A.n)
    np.add.at(want, np.repeat(np.arange(A.n), np.diff(A.rp)), A.val * x[A.col])
    for dt in [torch.float64] + [torch.float32] * fp32:
        y = torch.empty(A.n, dtype=dt, device="cuda")
        apply = ck.spmv_apply if dt == torch.float64 else ck.spmv_apply_f32
        apply(Mx.handle, torch.from_numpy(x).to("cuda", dt), y, 1.0, 0.0, ck.config_from_id(3))
        assert np.array_equal(y.cpu().double().numpy(), want), dt
    Mx.close()


@pytest.mark.parametrize("off", [0, 1])
def test_descents_are_row_starts(ck, off):
    """A column may fail to increase at a row's first entry and nowhere else,
    on both sides of each place in a group of four."""
    import torch
    for k in range(1, 9):
        say(f"descent at {k}")
        col = np.concatenate([np.arange(k) + 3, np.arange(9 - k) + 1]).astype(np.int32)
        val = np.ones(9)
        for cut in range(0, 10):
            rp = np.array([0, 0, cut, cut, 9], np.int32)
            args = [_shifted(a, o) for a, o in zip((rp, col, val), (0, off, off))]
            ok = cut == k
            if ok:
                ck.Matrix(*args, ncols=20).close()
            else:
                with pytest.raises(ck.CkError) as e:
                    ck.spmv_create(*args, ncols=20)
                assert e.value.status == ck.CK_E_INVALID
    # equal columns on both sides of a row start are sound, inside a row not
    col = torch.tensor([4, 4], dtype=torch.int32, device="cuda")
    val = torch.ones(2, dtype=torch.float64, device="cuda")
    ck.Matrix(torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda"), col, val, ncols=5).close()
    with pytest.raises(ck.CkError):
        ck.spmv_create(torch.tensor([0, 2, 2], dtype=torch.int32, device="cuda"), col, val, ncols=5)


@pytest.mark.parametrize("where", [0, 3, 4, 7, 8])
def test_range_is_checked_everywhere(ck, where):
    import torch
    rp = torch.arange(10, dtype=torch.int32, device="cuda")
    val = torch.ones(9, dtype=torch.float64, device="cuda")
    for bad in (-1, 5):
        col = torch.zeros(9, dtype=torch.int32, device="cuda")
        ck.Matrix(rp, col, val, ncols=5).close()
        col[where] = bad
        with pytest.raises(ck.CkError) as e:
            ck.spmv_create(rp, col, val, ncols=5)
        assert e.value.status == ck.CK_E_INVALID


@pytest.mark.parametrize("lengths", [[511, 512, 513] * 40, [600] * 70, [513] + [3] * 200 + [2000] * 3,
                                     [0, 513, 0, 1024, 1025, 255, 256, 257] * 9],
                         ids=["around", "every", "scattered", "mixed"])
def test_features_of_long_rows(ck, orc, lengths):
    A = _rows(lengths, 2600, 11)
    say(f"features of {A.n} rows, longest {max(lengths)}")
    Mx = ck.Matrix.from_csr(A)
    F = ck.spmv_features(Mx.handle)
    assert F.ints() == [int(v) for v in orc.features(A)[0]]
    Mx.close()
