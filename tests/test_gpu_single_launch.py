"""The single cooperative launch of the batched build at line lengths whose
tables leave fewer work-groups resident than the LDS bytes alone would allow
(LDS is handed out in pieces of 1280 bytes): every work-group of the grid must
be resident, or the grid barriers are never complete.  Against the x pass
followed by pdm_distance_yz."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [170, 192, 196, 197, 199, 210, 214, 217, 218, 225, 232, 236, 239, 256])
def test_single_launch_line_lengths(m):
    import paper_2407_21552_amd as pdm
    items, want = [], []
    for k, s in enumerate([(4 * m, 9, 21), (6, 4 * m - 1, 40)]):  # the longest lines along z and along y
        g = torch.Generator(device="cuda").manual_seed(m + k)
        vol = torch.zeros(s, dtype=torch.uint8, device="cuda")
        at = torch.randint(0, vol.numel(), (30,), generator=g, device="cuda")
        vol.view(-1)[at] = torch.randint(0, 256, (30,), generator=g, device="cuda").to(torch.uint8)
        bounds = np.array([0, 90, 170, 256], np.int32)
        v = pdm.Volume(vol, 256, bounds)
        pdms = torch.empty_like(v.pdms)
        pdm.build_bricks(v.desc, vol, v.bmin, v.bmax)
        pdm.pom_distance_x(v.desc, v.bmin, v.bmax, bounds, pdms)
        pdm.distance_yz(v.desc, pdms, 3)
        want.append(pdms)
        v.pdms.fill_(7)
        items.append((v.desc, v.volume, v.bmin, v.bmax, v.bounds, v.pdms))
    ws = torch.zeros(pdm.batch_workspace_bytes(len(items)), dtype=torch.uint8, device="cuda")
    pdm.batch_build(items, ws, dict(single_launch=1))
    assert pdm.batch_error(ws) == 0
    for it, w in zip(items, want):
        assert torch.equal(it[5], w)
