"""The Z-resident up projection at the edges of its tiles: 256-row bands (one row, a band less one, whole,
one more), one to several 64-column tiles of d per block (odd counts, whose last sum of squares has one
half), and several blocks per row band. It forms the products and the row sums of squares of the tiled
kernel in the same order, so M_l * gamma_l, K and V must agree to the bit."""
import pytest
import torch

import paper_2609_34972_amd as dvl
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [256, 512])
@pytest.mark.parametrize("T,d,L", [(1, 64, 1), (31, 128, 3), (255, 192, 2), (256, 1024, 1), (257, 960, 2),
                                   (513, 2048, 5)])
def test_resident_up_matches_tiled(T, d, L, r):
    say(f"[resident up T {T} d {d} L {L} r {r}]")
    g = torch.Generator().manual_seed(T * 7 + d + r)
    mk = lambda *s, std=1.0: (torch.randn(*s, generator=g) * std).bfloat16().cuda()
    E, Z, Uw = mk(T, d), mk(L, T, r), mk(L, d, r, std=r ** -0.5)
    gamma, Wk, Wv = mk(L, d), mk(L, 256, d, std=d ** -0.5), mk(L, 256, d, std=d ** -0.5)
    nbytes = dvl.project_visual_kv_workspace(T, d, L, torch.bfloat16)
    out = []
    try:
        for mode in (1, 2, 2):
            dvl.set_up_kernel(mode)
            assert dvl.project_visual_kv_up_kernel(T, d, r, L, torch.bfloat16) == mode
            ws = torch.full((nbytes,), 0x7F, dtype=torch.uint8, device="cuda:0")
            Kv = torch.empty(L, 1, 2, T, 128, dtype=torch.bfloat16, device="cuda:0")
            Vv = torch.empty_like(Kv)
            dvl.project_visual_kv(E, Z, Uw, gamma, Wk, Wv, Kv, Vv, eps=1e-5, ws=ws)
            torch.cuda.synchronize()
            out.append((ws[: L * T * d * 2].clone(), Kv, Vv))
    finally:
        dvl.set_up_kernel(0)
    for mode, got in zip(("resident", "resident again"), out[1:]):
        for name, x, y in zip(("M * gamma", "Kv", "Vv"), out[0], got):
            assert torch.equal(x, y), f"{name} differs between the kernels ({mode})"
