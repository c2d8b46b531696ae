"""GPU parity of the MoE layer (dispatch, GEMM0 + SiLU*up, GEMM1, combine)
against the CPU oracle, in the three execution modes and under forced plans.

Bar: max|y_gpu - y_ref| <= 2e-2 * max|y_ref| over the checked rows (bf16
inputs, fp32 accumulation, bf16 intermediates).  The dispatched rows are
checked bit for bit.  Every plan computes each output element with the same
operations in the same order, so y must also be bit-identical across modes
and plans."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2609_21483_amd import workloads as W
from tests.cases import bf16_to_f64, check_plan, make_case, oracle_rows, pick_rows, plain_reading, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21483_amd import binding
    return binding


def run_modes(B, layer, c, idx, w, modes=("dynamic", "static", "serial"), forced=()):
    shape = c.shape
    x = c.x.cuda()
    idx_d = torch.from_numpy(np.ascontiguousarray(idx, np.int32)).cuda()
    w_d = torch.from_numpy(np.ascontiguousarray(w, np.float32)).cuda()
    B.moe_build_tables(layer.h, idx_d)
    outs = {}
    for m in modes:
        y = torch.full((shape.T, shape.hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
        layer.forward(x, idx_d, w_d, y, m)
        st = B.moe_sync_status(layer.h)
        assert st == B.MOE_OK, (m, B.moe_last_error())
        outs[m] = y
    for p in forced:
        y = torch.full((shape.T, shape.hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
        layer.forward(x, idx_d, w_d, y, "dynamic", forced=B.moe_plan(*p, 0.0))
        st = B.moe_sync_status(layer.h)
        assert st == B.MOE_OK, (p, B.moe_last_error())
        outs[p] = y
    return outs


def check_case(B, c, rows=None, forced=(), check_A=False, gemm1_split=0):
    shape = c.shape
    idx, w = c.oracle_route()
    layer = B.MoeLayer(shape, c.w1, c.w3, c.w2, c.ws1, c.ws3, c.ws2, gemm1_split=gemm1_split)
    try:
        outs = run_modes(B, layer, c, idx, w, forced=forced)
        rows = np.arange(shape.T) if rows is None else rows
        y_ref = oracle_rows(c, idx, w, rows)
        first = None
        for key, y in outs.items():
            yg = bf16_to_f64(y[torch.from_numpy(rows).cuda()])
            assert np.all(np.isfinite(yg)), key
            err = rel_err(yg, y_ref)
            assert err <= TOL, (key, err)
            if first is None:
                first = y
            else:
                assert torch.equal(y.view(torch.int16), first.view(torch.int16)), f"{key} differs from dynamic"
        if check_A:
            check_dispatched_rows(B, layer, c, idx, w)
        return err
    finally:
        layer.close()


def check_dispatched_rows(B, layer, c, idx, w):
    """After a forward at each chunk count K, A holds the oracle's dispatched
    rows (slot order) at the rows of the row map of moe.h, and the row map is
    the segment-major prefix of the (segment, chunk) row counts, each rounded
    up to 32 rows."""
    shape = c.shape
    El, S, Tr, T, H = shape.n_local_experts, shape.n_shared_experts, shape.tokens_per_rank, shape.T, shape.hidden
    tab = O.route_tables(idx, shape.n_src_ranks, Tr, 0, El)
    ref = O.dispatch(c.xu, tab, shape.top_k)
    x = c.x.cuda()
    idx_d = torch.from_numpy(np.ascontiguousarray(idx, np.int32)).cuda()
    w_d = torch.from_numpy(np.ascontiguousarray(w, np.float32)).cuda()
    B.moe_build_tables(layer.h, idx_d)
    y = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    nseg = El + S
    rof = layer.ws_view("row_off", torch.int32, 4 * nseg * 9).cpu().numpy().reshape(4, nseg, 9)
    for ki, K in enumerate((1, 2, 4, 8)):
        sub = O.chunk_offsets(tab, T, shape.top_k, K)
        bnd = [(q * T + K - 1) // K for q in range(K + 1)]
        rows = [[int(sub[le][q + 1] - sub[le][q]) for q in range(K)] for le in range(El)]
        rows += [[max(0, min(bnd[q + 1], Tr) - bnd[q]) for q in range(K)] for _ in range(S)]
        start, at = np.zeros((nseg, K), np.int64), 0
        for seg in range(nseg):
            for q in range(K):
                start[seg, q] = at
                at += -(-rows[seg][q] // 32) * 32
        assert np.array_equal(rof[ki, :, :K], start), K
        assert not rof[ki, :, K:].any()
        layer.forward(x, idx_d, w_d, y, "dynamic", forced=B.moe_plan(8, K, 3, 1, 0.0))
        assert B.moe_sync_status(layer.h) == B.MOE_OK
        # 32-row groups, each group's 32-column k-steps one 32 x 32 block after the other
        G = -(-int(at) // 32)
        A = layer.ws_view("A", torch.int16, G * 32 * H).cpu().numpy().view(np.uint16)
        A = A.reshape(G, H // 32, 32, 32).transpose(0, 2, 1, 3).reshape(G * 32, H)
        for le in range(El):
            for q in range(K):
                n, s0, r0 = rows[le][q], int(sub[le][q]), int(start[le, q])
                assert np.array_equal(A[r0:r0 + n], ref[s0:s0 + n]), (K, le, q)


FORCED_SMALL = [(1, 1, 0, 1), (8, 2, 3, 1), (64, 4, 0, 0), (255, 8, 1000, 1), (40, 1, 0, 0), (128, 8, 2, 0)]


def test_tiny_all_rows_all_plans(B):
    c = make_case(W.TINY)
    check_case(B, c, forced=FORCED_SMALL, check_A=True)


@pytest.mark.parametrize("shape", [
    W.MoeShape("ragged", 98, 3, 45, 192, 320, 10, 3, 4, n_shared_experts=1),
    W.MoeShape("one_token", 97, 1, 1, 128, 128, 8, 2, 8),
    W.MoeShape("all_local", 96, 2, 150, 256, 192, 4, 4, 4),
    W.MoeShape("skew_empty", 95, 4, 77, 128, 256, 32, 8, 5, zipf_s=3.0),
    W.MoeShape("wide_tail", 94, 2, 200, 320, 576, 12, 2, 3, n_shared_experts=2),
], ids=lambda s: s.name)
def test_edge_shapes(B, shape):
    c = make_case(shape.with_(w_std=0.05))
    check_case(B, c, forced=FORCED_SMALL, check_A=True)


@pytest.mark.parametrize("split", [1, 2, 4, 8])
def test_gemm1_split_factors(B, split):
    """GEMM1 split 1, 2, 4 or 8 ways over F (the last split of a tile adds
    the fp32 partials in split order); shared experts and a ragged row tail
    included."""
    shape = W.MoeShape("split", 92, 3, 70, 128, 512, 8, 2, 4, n_shared_experts=1)
    c = make_case(shape.with_(w_std=0.05))
    check_case(B, c, forced=[(8, 2, 3, 1), (100, 4, 0, 0)], gemm1_split=split)


@pytest.mark.parametrize("shape,skew,split", [
    # GEMM0 in whole slabs, GEMM1 in narrow tiles
    (W.MoeShape("few32", 90, 2, 40, 192, 192, 16, 2, 4), 0, 1),           # one row block, ragged columns
    (W.MoeShape("few64", 89, 3, 64, 128, 192, 8, 2, 8, n_shared_experts=1), 0, 2),  # two; rank 0 fills a shared one
    (W.MoeShape("few_skew", 88, 2, 192, 128, 320, 32, 4, 6), 1, 1),      # one expert takes every token: 256 rows + 128
    (W.MoeShape("few_wide", 87, 1, 64, 128, 512, 48, 8, 40), 0, 4),      # both in whole slabs
    (W.MoeShape("few_wide_skew", 86, 1, 384, 320, 512, 64, 8, 48), 1, 1),  # GEMM1 in narrow tiles, two of them tall
    # GEMM0 deep enough for narrow tiles
    (W.MoeShape("few_deep32", 69, 2, 40, 1536, 192, 16, 2, 8), 0, 1),
    (W.MoeShape("few_deep64", 68, 3, 64, 1600, 192, 8, 2, 8, n_shared_experts=1), 0, 2),
    (W.MoeShape("few_deep_skew", 67, 2, 192, 1536, 320, 32, 4, 6), 1, 1),
    (W.MoeShape("few_deep_two", 66, 1, 16, 4096, 512, 24, 2, 24), 0, 1),  # more of them than workers
], ids=lambda v: getattr(v, "name", None))
def test_few_rows(B, shape, skew, split):
    """Layers of at most 48 routed rows per expert gather their rows and run
    phases of few tiles in narrow ones (GEMM0 where it is deep): y matches the oracle and has the bits
    of the general path, which a layer of the same tokens and routing several
    times over takes (a token's y does not depend on the other tokens)."""
    shape = shape.with_(w_std=0.05)
    c = make_case(shape)
    R, Tr, H, E, k = shape.n_src_ranks, shape.tokens_per_rank, shape.hidden, shape.n_experts, shape.top_k
    idx, w = W.random_routing(shape.T, E - skew, k - skew, seed=7)
    if skew:
        idx = np.concatenate([np.zeros((shape.T, 1), np.int64), idx + 1], axis=1)
        w = np.concatenate([np.full((shape.T, 1), 0.5), w * 0.5], axis=1)
    idx, w = idx.astype(np.int32), w.astype(np.float32)
    rep = 48 * E // (shape.T * k) + 1
    assert shape.T * k <= 48 * E < rep * shape.T * k
    big = shape.with_(tokens_per_rank=Tr * rep)

    def again(a):  # each rank's tokens rep times
        return np.tile(a.reshape(R, Tr, -1), (1, rep, 1)).reshape(R * Tr * rep, -1)

    layers = [B.MoeLayer(s, c.w1, c.w3, c.w2, c.ws1, c.ws3, c.ws2, gemm1_split=split) for s in (shape, big)]
    try:
        outs = run_modes(B, layers[0], c, idx, w, forced=[(8, 2, 3, 1), (100, 4, 0, 0)])
        y = outs["dynamic"]
        for key, o in outs.items():
            assert torch.equal(o.view(torch.int16), y.view(torch.int16)), key
        assert rel_err(bf16_to_f64(y), oracle_rows(c, idx, w.astype(np.float64), np.arange(shape.T))) <= TOL
        x2 = c.x.view(R, Tr, H).repeat(1, rep, 1).reshape(-1, H).contiguous().cuda()
        idx2, w2 = torch.from_numpy(again(idx)).cuda(), torch.from_numpy(again(w)).cuda()
        y2 = torch.empty((big.T, H), dtype=torch.bfloat16, device="cuda")
        B.moe_build_tables(layers[1].h, idx2)
        layers[1].forward(x2, idx2, w2, y2, "dynamic")
        assert B.moe_sync_status(layers[1].h) == B.MOE_OK
        y2 = y2.view(R, Tr * rep, H)[:, :Tr].reshape(-1, H)
        assert torch.equal(y2.contiguous().view(torch.int16), y.view(torch.int16))
    finally:
        for layer in layers:
            layer.close()


@pytest.mark.parametrize("shape,spread,split", [
    (W.MoeShape("few_units3", 81, 1, 770, 128, 1088, 17, 1, 8), 8, 1),     # tall row tiles, GEMM0 in whole slabs
    (W.MoeShape("few_units3n", 80, 1, 770, 128, 960, 17, 1, 8), 8, 2),     # and GEMM1 in two splits
    (W.MoeShape("few_units3d", 62, 1, 770, 1536, 960, 17, 1, 8), 8, 1),    # tall row tiles, narrow in both
    (W.MoeShape("few_units4", 79, 2, 513, 192, 192, 86, 4, 20), 86, 1),    # dispatch units of 8 tokens, the last of 2
    (W.MoeShape("few_units3t", 61, 2, 83, 192, 192, 24, 4, 20), 24, 1),    # of 3 tokens, the last of 1
    (W.MoeShape("few_units8", 78, 1, 4096, 64, 128, 86, 1, 3), 3, 1),      # the most tokens that gather, all local
    (W.MoeShape("beyond_few", 77, 1, 4097, 64, 128, 86, 1, 3), 3, 1),      # one more
], ids=lambda v: getattr(v, "name", None))
def test_few_rows_under_skewed_routing(B, shape, spread, split):
    """Layers of few rows on average whose routing takes `spread` experts: row
    tiles taller than a narrow tile's fast range, dispatch units of several
    tokens, and the bounds of the rule."""
    c = make_case(shape.with_(w_std=0.05))
    idx, w = W.random_routing(shape.T, spread, shape.top_k, seed=13)
    idx, w = idx.astype(np.int32), w.astype(np.float32)
    layer = B.MoeLayer(shape, c.w1, c.w3, c.w2, gemm1_split=split)
    try:
        outs = run_modes(B, layer, c, idx, w, forced=[(8, 2, 3, 1), (100, 4, 0, 0), (1, 1, 0, 1)])
        for key, o in outs.items():
            assert torch.equal(o.view(torch.int16), outs["serial"].view(torch.int16)), key
        y_ref = oracle_rows(c, idx, w.astype(np.float64), np.arange(shape.T))
        assert rel_err(bf16_to_f64(outs["serial"]), y_ref) <= TOL
    finally:
        layer.close()


@pytest.mark.parametrize("shape", [W.MoeShape("view_few", 76, 2, 40, 192, 192, 16, 2, 4),
                                   W.MoeShape("view_few_wide", 75, 1, 64, 128, 512, 48, 8, 40),
                                   W.MoeShape("view_few_deep", 63, 2, 40, 1536, 192, 16, 2, 8),
                                   W.MoeShape("view_general", 74, 2, 300, 128, 192, 4, 2, 2)], ids=lambda s: s.name)
@pytest.mark.parametrize("off", [1, 4])
def test_tokens_off_a_16_byte_boundary(B, shape, off):
    """x as a view that starts anywhere in a larger buffer: y has the bits of
    its aligned copy's, in layers that gather their rows from x too."""
    c = make_case(shape.with_(w_std=0.05))
    idx, w = W.random_routing(shape.T, shape.n_experts, shape.top_k, seed=3)
    ml = B.MoeLayer(shape, c.w1, c.w3, c.w2)
    try:
        x = c.x.cuda()
        buf = torch.zeros(x.numel() + off, dtype=torch.bfloat16, device="cuda")
        view = buf[off:].view(x.shape)
        view.copy_(x)
        idx_d, w_d = torch.from_numpy(idx.astype(np.int32)).cuda(), torch.from_numpy(w.astype(np.float32)).cuda()
        B.moe_build_tables(ml.h, idx_d)
        ys = []
        for xv, mode in ((x, "dynamic"), (view, "dynamic"), (view, "static"), (view, "serial")):
            y = torch.full((shape.T, shape.hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
            ml.forward(xv, idx_d, w_d, y, mode)
            assert B.moe_sync_status(ml.h) == B.MOE_OK
            ys.append(y)
        y = torch.empty_like(ys[0])
        B.moe_forward_stack([ml.h], view, [idx_d], [w_d], [ml.packed], [y])
        assert B.moe_sync_status(ml.h) == B.MOE_OK
        for o in ys[1:] + [y]:
            assert torch.equal(o.view(torch.int16), ys[0].view(torch.int16))
    finally:
        ml.close()


def test_no_local_pairs(B):
    """Every token routed off this GPU: y must be all zeros (no shared experts),
    or only the shared output on rank 0."""
    for S in (0, 1):
        shape = W.MoeShape("nolocal", 93, 2, 64, 128, 128, 16, 2, 4, n_shared_experts=S)
        c = make_case(shape.with_(w_std=0.05))
        idx, w = W.random_routing(shape.T, 12, 2, seed=5)
        idx = (idx + 4).astype(np.int32)  # experts 4..15, all remote
        layer = B.MoeLayer(shape, c.w1, c.w3, c.w2, c.ws1, c.ws3, c.ws2)
        try:
            outs = run_modes(B, layer, c, idx, w.astype(np.float64))
            y_ref = oracle_rows(c, idx, w.astype(np.float64), np.arange(shape.T))
            for y in outs.values():
                yg = bf16_to_f64(y)
                if S == 0:
                    assert np.all(yg == 0.0)
                else:
                    assert np.all(yg[shape.tokens_per_rank:] == 0.0)
                    assert rel_err(yg, y_ref) <= TOL
        finally:
            layer.close()


FULL = [("mixtral_ep4", 0), ("fine_zipf", 0), ("shared_routed", 0)] + [("large_stack", l) for l in range(8)]


@pytest.mark.parametrize("name,layer", FULL, ids=[f"{n}-L{l}" for n, l in FULL])
def test_full_size_sampled_rows(B, name, layer):
    """A whole layer share at full size, y checked on sampled rows (rows are
    independent, so a sample is exact) in every mode, under forced chunked
    plans, and under the cost model's plans on the built-in table, the
    committed measured table and the plain reading of the printed equations;
    each plan against the oracle's cost model on the oracle's tables."""
    from paper_2609_21483_amd.calibrate import load_calib
    shape = W.WORKLOADS[name]
    c = make_case(shape, layer)
    idx, w = c.oracle_route()
    rows = pick_rows(shape, idx, per_rank=16, seed=100 + layer)
    forced = [(8, 8, 4, 1), (120, 2, 0, 1)] if name == "fine_zipf" else [(40, 2, 4, 1), (64, 4, 2, 1)]
    ml = B.MoeLayer(shape, c.w1, c.w3, c.w2, c.ws1, c.ws3, c.ws2)
    try:
        x = c.x.cuda()
        idx_d = torch.from_numpy(np.ascontiguousarray(idx, np.int32)).cuda()
        w_d = torch.from_numpy(np.ascontiguousarray(w, np.float32)).cuda()
        B.moe_build_tables(ml.h, idx_d)

        def fwd(mode, plan=None):
            y = torch.full((shape.T, shape.hidden), float("nan"), dtype=torch.bfloat16, device="cuda")
            ml.forward(x, idx_d, w_d, y, mode, forced=None if plan is None else B.moe_plan(*plan, 0.0))
            assert B.moe_sync_status(ml.h) == B.MOE_OK, (mode, plan, B.moe_last_error())
            return y

        outs = {"dynamic": fwd("dynamic")}
        check_plan(B, ml.h, shape, idx)
        outs["static"] = fwd("static")
        outs["serial"] = fwd("serial")
        for p in forced:
            outs[p] = fwd("dynamic", p)
        measured = load_calib(name, torch.cuda.get_device_properties(0).multi_processor_count)
        if measured is not None:
            B.moe_set_calib(ml.h, measured)
            outs["measured"] = fwd("dynamic")
            check_plan(B, ml.h, shape, idx)
            B.moe_set_calib(ml.h, plain_reading(B.moe_calib.from_buffer_copy(measured)))
            outs["plain"] = fwd("dynamic")
            check_plan(B, ml.h, shape, idx)
        y_ref = oracle_rows(c, idx, w, rows)
        first = outs["dynamic"]
        sel = torch.from_numpy(rows).cuda()
        for key, y in outs.items():
            yg = bf16_to_f64(y[sel])
            assert np.all(np.isfinite(yg)), key
            assert rel_err(yg, y_ref) <= TOL, key
            assert torch.equal(y.view(torch.int16), first.view(torch.int16)), f"{key} differs from dynamic"
    finally:
        ml.close()


@pytest.mark.parametrize("K", [1, 2, 4])
def test_run_stages_reproduces_forward(B, K):
    """moe_run_stages (the stages as separate kernels on n workers, used by
    the calibration) with every stage gives the forward's y bit for bit."""
    shape = W.SHARED_ROUTED.with_(tokens_per_rank=512)
    c = make_case(shape)
    idx, w = c.oracle_route()
    ml = B.MoeLayer(shape, c.w1, c.w3, c.w2, c.ws1, c.ws3, c.ws2)
    try:
        x = c.x.cuda()
        idx_d = torch.from_numpy(idx).cuda()
        w_d = torch.from_numpy(w.astype(np.float32)).cuda()
        B.moe_build_tables(ml.h, idx_d)
        y0 = torch.empty((shape.T, shape.hidden), dtype=torch.bfloat16, device="cuda")
        ml.forward(x, idx_d, w_d, y0, "dynamic")
        assert B.moe_sync_status(ml.h) == B.MOE_OK
        rows = pick_rows(shape, idx, per_rank=24, seed=3)
        assert rel_err(bf16_to_f64(y0[torch.from_numpy(rows).cuda()]), oracle_rows(c, idx, w, rows)) <= TOL
        for n in (torch.cuda.get_device_properties(0).multi_processor_count, 37):
            y = torch.full_like(y0, float("nan"))
            B.moe_run_stages(ml.h, x, idx_d, w_d, ml.packed, y, 15, n, K)
            assert B.moe_sync_status(ml.h) == B.MOE_OK
            assert torch.equal(y.view(torch.int16), y0.view(torch.int16)), (K, n)
    finally:
        ml.close()


@pytest.mark.parametrize("shape", [
    W.MoeShape("few_stages", 85, 2, 40, 192, 192, 16, 2, 4),          # GEMM1 in narrow tiles of one row block
    W.MoeShape("few_stages_wide", 84, 1, 64, 128, 512, 48, 8, 40),    # whole slabs
    W.MoeShape("few_stages_tall", 83, 2, 192, 128, 320, 16, 1, 1),    # one expert of many rows: one k-step a stage
    W.MoeShape("few_deep", 65, 2, 40, 1536, 192, 16, 2, 8),           # GEMM0 in narrow tiles too
    W.MoeShape("few_deep_tall", 64, 2, 192, 1536, 704, 16, 1, 1),
    W.MoeShape("general_stages", 82, 2, 300, 128, 192, 4, 2, 2),
], ids=lambda s: s.name)
@pytest.mark.parametrize("K", [1, 4])
def test_run_stages_read_what_earlier_stages_wrote(B, shape, K):
    """Stages called one by one, x overwritten once its rows are dispatched:
    GEMM0 reads the dispatched rows, also in layers of few rows."""
    c = make_case(shape.with_(w_std=0.05))
    idx, w = W.random_routing(shape.T, shape.n_experts, shape.top_k, seed=11)
    if shape.name.endswith("tall"):
        idx[:] = 0
    idx, w = idx.astype(np.int32), w.astype(np.float32)
    ml = B.MoeLayer(shape, c.w1, c.w3, c.w2)
    try:
        x, idx_d, w_d = c.x.cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda()
        B.moe_build_tables(ml.h, idx_d)
        y0 = torch.empty((shape.T, shape.hidden), dtype=torch.bfloat16, device="cuda")
        ml.forward(x, idx_d, w_d, y0, "dynamic")
        assert rel_err(bf16_to_f64(y0), oracle_rows(c, idx, w.astype(np.float64), np.arange(shape.T))) <= TOL
        n = torch.cuda.get_device_properties(0).multi_processor_count
        y = torch.full_like(y0, float("nan"))
        for stage in (1, 2, 4, 8):
            B.moe_run_stages(ml.h, x, idx_d, w_d, ml.packed, y, stage, n, K)
            if stage == 1:
                x.zero_()
        assert B.moe_sync_status(ml.h) == B.MOE_OK
        assert torch.equal(y.view(torch.int16), y0.view(torch.int16))
    finally:
        ml.close()


def test_route_then_forward_end_to_end(B):
    """moe_route output fed straight into moe_forward."""
    shape = W.FINE_ZIPF.with_(tokens_per_rank=256)
    c = make_case(shape)
    idx_ref, w_ref = c.oracle_route()
    layer = B.MoeLayer(shape, c.w1, c.w3, c.w2)
    try:
        x = c.x.cuda()
        idx = torch.empty((shape.T, shape.top_k), dtype=torch.int32, device="cuda")
        w = torch.empty((shape.T, shape.top_k), dtype=torch.float32, device="cuda")
        layer.route(x, c.wg.cuda(), c.bias.cuda(), idx, w)
        y = torch.empty((shape.T, shape.hidden), dtype=torch.bfloat16, device="cuda")
        layer.forward(x, idx, w, y, "dynamic")
        assert B.moe_sync_status(layer.h) == B.MOE_OK
        assert np.array_equal(idx.cpu().numpy(), idx_ref)
        y_ref = oracle_rows(c, idx_ref, w_ref, np.arange(shape.T))
        assert rel_err(bf16_to_f64(y), y_ref) <= TOL
        # forward refuses routing the tables were not built from
        other = idx.clone()
        with pytest.raises(B.MoeError) as ei:
            layer.forward(x, other, w, y, "dynamic")
        assert ei.value.status == B.MOE_ERR_STATE
    finally:
        layer.close()


def test_repeat_launches_deterministic(B):
    c = make_case(W.FINE_ZIPF.with_(tokens_per_rank=512))
    idx, w = c.oracle_route()
    layer = B.MoeLayer(c.shape, c.w1, c.w3, c.w2)
    try:
        x = c.x.cuda()
        idx_d = torch.from_numpy(idx).cuda()
        w_d = torch.from_numpy(w.astype(np.float32)).cuda()
        B.moe_build_tables(layer.h, idx_d)
        ys = []
        for i in range(6):
            y = torch.empty((c.shape.T, c.shape.hidden), dtype=torch.bfloat16, device="cuda")
            layer.forward(x, idx_d, w_d, y, ("dynamic", "static", "serial")[i % 3])
            ys.append(y)
        assert B.moe_sync_status(layer.h) == B.MOE_OK
        for y in ys[1:]:
            assert torch.equal(y.view(torch.int16), ys[0].view(torch.int16))
    finally:
        layer.close()


def test_relaunch_with_new_inputs(B):
    """The same workspace and control sets serve launches whose tokens and
    routing change: each result matches the oracle for its own inputs (no
    stale rows from the previous launch)."""
    shape = W.FINE_ZIPF.with_(tokens_per_rank=384)
    c1 = make_case(shape)
    c2 = make_case(shape.with_(wid=shape.wid + 50))
    layer = B.MoeLayer(shape, c1.w1, c1.w3, c1.w2)
    try:
        for c in (c1, c2, c1):
            idx, w = c.oracle_route()
            outs = run_modes(B, layer, c, idx, w, modes=("dynamic", "serial"))
            rows = pick_rows(shape, idx, per_rank=24, seed=7)
            # c2 shares c1's expert weights (the layer packs them once)
            y_ref = oracle_rows(c1.with_tokens(c), idx, w, rows)
            for y in outs.values():
                assert rel_err(bf16_to_f64(y[torch.from_numpy(rows).cuda()]), y_ref) <= TOL
    finally:
        layer.close()


def test_more_workers_than_the_gpu_holds_is_refused(B):
    """The megakernel's workgroups wait on each other, so all of them must be
    resident at once: a worker count beyond what the GPU holds is refused
    before any launch (one workgroup fits a CU)."""
    c = make_case(W.TINY)
    idx, w = c.oracle_route()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    layer = B.MoeLayer(c.shape, c.w1, c.w3, c.w2, n_workers=2 * cus)
    try:
        x = c.x.cuda()
        idx_d = torch.from_numpy(idx).cuda()
        w_d = torch.from_numpy(w.astype(np.float32)).cuda()
        B.moe_build_tables(layer.h, idx_d)
        y = torch.zeros((c.shape.T, c.shape.hidden), dtype=torch.bfloat16, device="cuda")
        with pytest.raises(B.MoeError) as ei:
            layer.forward(x, idx_d, w_d, y, "dynamic")
        assert ei.value.status == B.MOE_ERR_UNSUPPORTED
        assert "holds at once" in B.moe_last_error()
        # the serial kernels have no such constraint
        layer.forward(x, idx_d, w_d, y, "serial")
        assert B.moe_sync_status(layer.h) == B.MOE_OK
        assert rel_err(bf16_to_f64(y), oracle_rows(c, idx, w, np.arange(c.shape.T))) <= TOL
    finally:
        layer.close()


def test_timeout_path_recovers(B):
    """Host-forced stall: every wait targets an unreachable value, so the
    launch times out on its own bounded waits, reports MOE_ERR_TIMEOUT, and the
    next launch (other control set) is correct again."""
    c = make_case(W.TINY)
    idx, w = c.oracle_route()
    layer = B.MoeLayer(c.shape, c.w1, c.w3, c.w2)
    try:
        x = c.x.cuda()
        idx_d = torch.from_numpy(idx).cuda()
        w_d = torch.from_numpy(w.astype(np.float32)).cuda()
        B.moe_build_tables(layer.h, idx_d)
        y = torch.empty((c.shape.T, c.shape.hidden), dtype=torch.bfloat16, device="cuda")
        B.moe_set_timeout_ms(layer.h, 20.0, 1)
        layer.forward(x, idx_d, w_d, y, "dynamic")
        assert B.moe_sync_status(layer.h) == B.MOE_ERR_TIMEOUT
        B.moe_set_timeout_ms(layer.h, 2000.0, 0)
        for _ in range(2):
            layer.forward(x, idx_d, w_d, y, "dynamic")
            assert B.moe_sync_status(layer.h) == B.MOE_OK
            y_ref = oracle_rows(c, idx, w, np.arange(c.shape.T))
            assert rel_err(bf16_to_f64(y), y_ref) <= TOL
    finally:
        layer.close()
