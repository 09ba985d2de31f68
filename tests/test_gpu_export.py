"""mst_layer_export_dense against the arrays that the layer was loaded from: rows shorter and longer than the run of positions a
workgroup owns (4096), layers of so many rows that it owns several, row lengths that are no multiple of four, empty and full rows, either output alone."""
import pytest
import torch

from paper_2408_11746_amd import binding as mst

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("O,I", [(1, 1), (5, 7), (64, 64), (3, 4095), (3, 4096), (3, 4097), (2, 8201), (1283, 515), (4, 12288), (3073, 515), (2051, 768),
                                 (9000, 7), (65535, 1)])
@pytest.mark.parametrize("density", [0.0, 0.03, 1.0])
def test_export(O, I, density):
    gen = torch.Generator().manual_seed(O * 131 + I)
    W = torch.randn(O, I, generator=gen)
    M = torch.rand(O, I, generator=gen) < density
    if density == 0.03 and O > 1:
        M[0], M[O - 1] = False, True
    count = int(M.sum())
    layer = mst.Layer(O, I, max(count, 1), "cuda")
    ws = torch.empty(mst.mst_workspace_bytes(O, I, max(count, 1), 64), dtype=torch.uint8, device="cuda")
    layer.load_dense(W.cuda(), M.to(torch.uint8).cuda(), ws)
    expect_W, expect_M = torch.where(M, W, torch.zeros(())), M.to(torch.uint8)
    for with_W, with_M in ((True, True), (True, False), (False, True)):
        oW = torch.full((O * I + 64,), 7.0, device="cuda")
        oM = torch.full((O * I + 64,), 9, dtype=torch.uint8, device="cuda")
        layer.export_dense(oW if with_W else None, oM if with_M else None)
        oW, oM = oW.cpu(), oM.cpu()
        if with_W:
            assert torch.equal(oW[:O * I].view(O, I), expect_W)
        if with_M:
            assert torch.equal(oM[:O * I].view(O, I), expect_M)
        assert (oW[O * I if with_W else 0:] == 7.0).all() and (oM[O * I if with_M else 0:] == 9).all()   # nothing past the end


@pytest.mark.parametrize("O,I,density", [(2, 4100, 0.26), (3, 8193, 0.2), (2, 16381, 0.5), (1, 65535, 1.0), (2, 65533, 0.016), (2, 65534, 0.9)])
def test_parts_of_long_rows(O, I, density):
    """Rows of several parts with more than 1024 active positions, whose parts find theirs by samples: even ones, and rows whose
    positions all lie at one end."""
    gen = torch.Generator().manual_seed(I)
    W = torch.randn(O, I, generator=gen)
    M = torch.rand(O, I, generator=gen) < density
    if O > 1:
        at = I - int(density * I) if I % 2 else 0
        M[1] = False
        M[1, at:at + int(density * I)] = True
    count = int(M.sum())
    layer = mst.Layer(O, I, count, "cuda")
    ws = torch.empty(mst.mst_workspace_bytes(O, I, count, 64), dtype=torch.uint8, device="cuda")
    layer.load_dense(W.cuda(), M.to(torch.uint8).cuda(), ws)
    out = torch.full((O * I + 64,), 7.0, device="cuda")
    layer.export_dense(out, None)
    out = out.cpu()
    assert torch.equal(out[:O * I].view(O, I), torch.where(M, W, torch.zeros(()))) and (out[O * I:] == 7.0).all()
