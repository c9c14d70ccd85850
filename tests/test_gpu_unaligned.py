"""The decay gradient takes dY at any address (the other convolution calls ask
for 16-byte alignment): where a view does not start on 16 bytes, no load of the
tile pass is wider than an element, and no fused kernel reads it."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("c,n_decays,dtype", [
    (20, 2, "f32"),   # tile pass, whole 16-byte pieces but for the base
    (64, 3, "f32"),
    (24, 2, "bf16"),
    (40, 4, "bf16"),
    (32, 2, "f32"),   # the shape of the fused kernel
])
@pytest.mark.parametrize("with_csc", [False, True])
def test_decay_gradient_of_an_unaligned_view(c, n_decays, dtype, with_csc):
    print(f"[unaligned dY] C {c} decays {n_decays} {dtype} csc {with_csc}", flush=True)
    w = workloads.small_events(seed=80, n=1300, c=c, n_decays=n_decays, dtype=dtype)
    rp, ci = oracle.events_csr(w["px"], w["py"], w["t"], w["window"], 1, w["width"], w["height"])
    t = G.to_device(w)
    csr = G.search(w, t)
    csc = G.sbc.csr_transpose(csr) if with_csc else None
    vd = oracle.basis.event_decay_basis(w["px"], w["py"], w["t"], rp, ci, w["decays"],
                                        derivative=True)
    ref = oracle.conv.decay_backward(rp, ci, vd, w["F"], w["W"], w["dY"])
    buf = torch.zeros(t["dY"].numel() + 1, dtype=t["dY"].dtype, device=G.DEV)
    dY = buf[1:].view(t["dY"].shape)
    dY.copy_(t["dY"])
    assert dY.data_ptr() % 16 != 0 and dY.is_contiguous()
    dl = G.sbc.conv_decay_gradient(csr, t["F"], t["W"], dY, G.geometry(w, t), csc=csc)
    tol = G.TOL_BF16 if dtype == "bf16" else G.TOL_F32
    assert G.norm_error(dl.cpu().numpy(), ref) < tol
