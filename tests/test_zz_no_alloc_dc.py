"""mg_solve_dgp_noalloc in every precision that it admits: the static workspace
holds the largest layout, and the defect-correction solve (MG_MIXED_DC, the
largest) agrees to the bit with mg_solve_dgp."""
import ctypes as C
import re

import pytest
import torch

import inputs
import paper_2110_00566_amd as mg


def test_static_workspace_holds_every_precision():
    # the size that the header and the message state, against the layouts (256 bytes
    # of a query's answer are for the alignment of the caller's workspace)
    doc = re.sub(r"\s*\n \*", "", open(mg.HEADER).read())
    mib = int(re.search(r"workspace is a static device array of (\d+) MiB", doc).group(1))
    for precision in (mg.MG_FP64, mg.MG_MIXED, mg.MG_FP32, mg.MG_MIXED_DC):
        assert mg.lib().mg_workspace_bytes(128, precision, mg.MODEL_DGP, 0) - 256 <= mib << 20
    o, st, d = mg.make_opts(256), mg.Stats(), C.c_void_p(0x1000)
    assert mg.lib().mg_solve_dgp_noalloc(C.byref(o), C.byref(mg.dgp_params()), d, d, None,
                                         C.byref(st)) == mg.MG_ERR_ARG
    assert b"%d MiB" % mib in mg.lib().mg_last_error()


@pytest.mark.gpu
def test_noalloc_defect_correction():
    delta = torch.from_numpy(inputs.lognormal_delta(128, 21)).to("cuda")
    kw = dict(tol=1e-8, max_cycles=30, precision=mg.MG_MIXED_DC)
    ref, st_ref = mg.solve_dgp(delta, **kw)
    got, st = mg.solve_dgp_noalloc(delta, **kw)
    assert st["status"] == st_ref["status"] == mg.MG_OK
    assert st["eps_hist"] == st_ref["eps_hist"]
    assert torch.equal(got, ref)
