"""Which products go to the sparse matrix instructions, and when their packed weights are made again: the choice follows the mask
that the layer has now, the packing follows what products read.  Nothing is pinned but where a test says so; every product is compared with
the double-precision product of the exported weights (two bfloat16 parts per fp32 operand: see test_gpu_pairs.py)."""
import pytest

import paper_2408_11746_amd as mst

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from gpu_util import DEV, rel_err  # noqa: E402

PARTS = 2e-5
PAIRS = 24
T, I, O = 16384, 1024, 4096


def _mask(density, kind, gen):
    """uniform: every position alike.  rows: a twentieth of the rows full, so that most of the steps of Y go a second time.  crossed: full rows and
    full columns, so that those of dX do as well."""
    M = torch.rand((O, I), generator=gen, device=DEV) < (density if kind == "uniform" else density - 0.05)
    if kind != "uniform":
        M[torch.randperm(O, generator=gen, device=DEV)[:O // (20 if kind == "rows" else 40)]] = True
    if kind == "crossed":
        M[:, torch.randperm(I, generator=gen, device=DEV)[:I // 40]] = True
    return M.to(torch.uint8)


class Layer:
    def __init__(self, density, mask="uniform", dtype="f32"):
        self.act = mst.MST_BF16 if dtype == "bf16" else mst.MST_F32
        self.gen = torch.Generator(device=DEV).manual_seed(9)
        self.L = mst.Layer(O, I, O * I, DEV)
        self.ws = torch.empty(mst.mst_workspace_bytes(O, I, O * I, T), dtype=torch.uint8, device=DEV)
        self.load(density, mask)
        kind = torch.bfloat16 if dtype == "bf16" else torch.float32
        self.X = torch.randn((T, I), generator=self.gen, device=DEV).to(kind)
        self.dY = torch.randn((T, O), generator=self.gen, device=DEV).to(kind)
        self.Y = torch.empty((T, O), dtype=torch.float32, device=DEV)
        self.dX = torch.empty((T, I), dtype=torch.float32, device=DEV)

    def load(self, density, mask):
        W = 0.02 * torch.randn((O, I), generator=self.gen, device=DEV)
        self.L.load_dense(W, _mask(density, mask, self.gen), self.ws)

    def weights(self):
        W = torch.empty((O, I), dtype=torch.float32, device=DEV)
        self.L.export_dense(W, None)
        return W.double()

    def update(self, density, zeta=0.3, rand_ratio=0.25):
        G = torch.randn((O, I), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV)
        mst.mst_mask_update_from_scores(self.L, G, density, zeta, rand_ratio, 7, self.ws)
        self.L.values().add_(0.01)
        self.L.sync_values()
        torch.cuda.synchronize()

    def fwd(self, tokens=T, stream=None):
        self.Y.fill_(float("nan"))
        mst.mst_sparse_fc_fwd(self.L, self.X, self.Y, tokens, self.act, stream)
        return mst.mst_gemm_last_tile() == PAIRS

    def bwd(self, stream=None):
        self.dX.fill_(float("nan"))
        mst.mst_sparse_fc_bwd_input(self.L, self.dY, self.dX, T, self.act, stream)
        return mst.mst_gemm_last_tile() == PAIRS

    def right(self, scale=1.0, tokens=T):
        """the last Y, of the weights handed over last (scale: theirs against the values now)"""
        torch.cuda.synchronize()
        W = self.weights() * scale
        at = torch.arange(0, tokens, max(1, tokens // 64), device=DEV)
        assert rel_err(self.Y[at].cpu().numpy(), (self.X[at].double() @ W.T).cpu().numpy()) <= PARTS

    def right_dx(self, scale=1.0):
        torch.cuda.synchronize()
        W = self.weights() * scale
        at = torch.arange(0, T, T // 64, device=DEV)
        assert rel_err(self.dX[at].cpu().numpy(), (self.dY[at].double() @ W).cpu().numpy()) <= PARTS

    def packed(self):
        """the packed weights of dX, in front of the two planes at the end of the layer's buffer"""
        end = self.L.buf.numel() - 8 * O * I
        return self.L.buf[end - -(-I // 256) * (O // 64) * 2 * 34816:end]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_the_choice_follows_the_loaded_mask(dtype):
    l = Layer(0.1, "uniform", dtype)
    assert l.fwd()
    l.right()
    for mask, want in (("rows", False), ("uniform", True), ("rows", False)):
        l.load(0.1, mask)
        assert l.fwd() == want, mask
        l.right()


def test_a_recorded_first_product_leaves_the_measurement_to_an_eager_one():
    l, side, graph = Layer(0.1, "rows"), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    l.L.set_path(mst.MST_PATH_DENSE)
    mst.mst_gemm_force_fp32_mfma(128)
    try:
        l.fwd()                                              # the dense copy alone
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        l.fwd(stream=side)
    graph.replay()
    l.right()
    assert not l.fwd()
    l.right()


def test_the_choice_follows_updates():
    """An uneven mask that an update replaces by a random one: measured again where products have come between."""
    l = Layer(0.1, "rows")
    for _ in range(70):
        assert not l.fwd()
    l.update(0.1, zeta=1.0, rand_ratio=1.0)
    assert l.fwd()
    l.right()


def _untouched(l, what):
    torch.cuda.synchronize()
    assert bool((l.packed() == 0xFF).all()), what


def test_nothing_is_packed_for_a_mask_that_was_turned_down():
    l = Layer(0.1, "crossed")
    assert not l.fwd()
    assert not l.bwd()
    torch.cuda.synchronize()
    l.packed().fill_(0xFF)
    l.L.values().mul_(2.0)
    l.L.sync_values()
    _untouched(l, "handed over")
    assert not l.fwd()
    l.right()
    l.update(0.1)
    _untouched(l, "updated")
    assert not l.fwd()
    l.right()


def test_nothing_is_packed_at_a_density_at_which_the_dense_kernels_are_ahead():
    l = Layer(0.1)
    assert l.fwd() and l.bwd()
    l.update(0.09)
    assert l.fwd() and l.bwd()
    l.right()
    l.right_dx()
    torch.cuda.synchronize()
    l.packed().fill_(0xFF)
    l.update(0.119)
    _untouched(l, "updated")
    assert not l.fwd()
    l.right()
    l.update(0.1)
    assert l.fwd() and l.bwd()
    l.right()
    l.right_dx()


def test_the_packing_stops_where_no_product_reads_it():
    l = Layer(0.1)
    assert l.fwd()
    for k in range(12):                                      # (short batches: other kernels)
        l.L.values().mul_(1.1)
        l.L.sync_values()
        l.fwd(tokens=100)
        if k == 9:
            torch.cuda.synchronize()
            l.packed().fill_(0xFF)
    _untouched(l, "twelve hand-overs")
    assert l.fwd()
    l.right()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_handover_recorded_at_half_density_does_not_bar_the_packed_pairs(dtype):
    l, side, graph = Layer(0.5, "uniform", dtype), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    assert not l.fwd()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        l.L.sync_values(side)
    l.update(0.1)
    for _ in range(3):
        assert l.fwd() and l.bwd()
        l.right()
        l.right_dx()
        l.L.values().mul_(2.0)
        l.L.sync_values()
    torch.cuda.synchronize()
    step = torch.cuda.CUDAGraph()
    with torch.cuda.graph(step, stream=side):
        assert l.fwd(stream=side) and l.bwd(stream=side)
        l.L.values().mul_(2.0)
        l.L.sync_values(side)
    for _ in range(3):
        step.replay()
        l.right(0.5)
        l.right_dx(0.5)
        assert l.fwd() and l.bwd()
        l.right()
        l.right_dx()
        l.L.values().mul_(0.25)
        l.L.sync_values()


def test_a_handover_recorded_before_the_first_packed_product():
    """Its replays leave packed weights behind that products read between them."""
    l, side, graph, product = Layer(0.1), torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    mst.mst_gemm_force_fp32_mfma(128)
    try:
        assert not l.fwd()                                   # the dense copy alone
    finally:
        mst.mst_gemm_force_fp32_mfma(0)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        l.L.values().mul_(2.0)
        l.L.sync_values(side)
    assert l.fwd()
    l.right()
    with torch.cuda.graph(product, stream=side):
        l.fwd(stream=side)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert l.fwd()
        l.right()
        graph.replay()
        torch.cuda.synchronize()
        product.replay()
        l.right()
        assert l.bwd()
        l.right_dx()


def test_a_recorded_product_outlives_the_densities_of_the_packed_pairs():
    l, side, graph = Layer(0.1), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    assert l.fwd()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        assert l.fwd(stream=side)
    for density in (0.2, 0.5, 0.1):
        l.update(density)                                    # (keeps the dense copy)
        graph.replay()
        l.right()
        for _ in range(12):                                  # hand-overs that nothing but the recording reads
            l.L.values().mul_(1.1)
            l.L.sync_values()
        graph.replay()
        l.right()


def test_a_recorded_handover_leaves_out_planes_that_the_packed_pairs_stand_for():
    l, side, graph = Layer(0.1, "uniform", "bf16"), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    assert l.fwd() and l.bwd()
    planes = l.L.buf[-8 * O * I:]
    torch.cuda.synchronize()
    planes.fill_(0xFF)
    with torch.cuda.graph(graph, stream=side):
        l.L.values().mul_(2.0)
        l.L.sync_values(side)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((planes == 0xFF).all())
        assert l.fwd() and l.bwd()
        l.right()
        l.right_dx()
    mst.mst_gemm_force_fp32_mfma(256)                        # products that read the planes after all
    try:
        for _ in range(2):
            graph.replay()
            torch.cuda.synchronize()
            l.fwd()
            assert mst.mst_gemm_last_tile() == 256
            l.right()
    finally:
        mst.mst_gemm_force_fp32_mfma(0)


@pytest.mark.parametrize("tokens", [2048, 5120, 9216])
def test_full_rows_go_to_the_dense_kernels(tokens):
    """Where every step goes a second time and the dense kernel takes 1.85 to 2.1 times as long as the steps of the first kind."""
    l = Layer(0.1, "rows")
    assert not l.fwd(tokens)
    l.right(tokens=tokens)
    l.load(0.1, "uniform")
    assert l.fwd(tokens)
    l.right(tokens=tokens)
