"""The slot copy of a small matrix is an option: a CG solve whose handle cannot
have the memory for it runs from the CSR arrays, with the same bits."""
import numpy as np
import pytest

from helpers import say, upload
from synth import matrices as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True])
def test_refused_copy(orc, mixed):
    import torch
    import paper_2411_10143_amd as ck
    A = M.diagonally_dominant(M.laplacian_2d(70))   # n = 4,900: above the FP64 kernel of its own
    b = M.vector(A.n, 2)
    db = torch.from_numpy(b).cuda()
    most = {"bytes": 1 << 40}
    live, refused = {}, []

    def alloc(nbytes, stream):
        if nbytes > most["bytes"]:
            refused.append(nbytes)
            return 0
        p = torch.cuda.caching_allocator_alloc(nbytes, torch.cuda.current_device(), stream)
        live[p] = nbytes
        return p

    def free(p, stream):
        del live[p]
        torch.cuda.caching_allocator_delete(p)

    got = []
    for limit in (1 << 40, (4 if mixed else 8) * 4 * (A.n + 64)):   # any; the vectors at most
        most["bytes"] = 1 << 40
        Mx = ck.Matrix(*upload(A), keep_fp32=True, allocator=ck.CallbackAllocator(alloc, free))
        most["bytes"] = limit
        say(f"slot copy mixed={mixed} blocks of at most {limit} bytes")
        x = torch.zeros_like(db)
        r = ck.cg_solve(Mx.handle, db, x, tol=1e-10,
                        precision=ck.CK_PREC_MIXED if mixed else ck.CK_PREC_FP64)
        assert r["status"] == ck.CK_OK, r
        got.append(x.cpu().numpy())
        Mx.close()
    assert refused and not live
    assert orc.relres(A, b, got[0]) <= 1e-10
    assert np.array_equal(got[0].view(np.int64), got[1].view(np.int64))
