"""GPU parity of routing (gate logits, softmax, top-k, renormalise) and of the
routing tables, against the CPU oracle.  Expert ids, counts, offsets, slots,
inverse permutation, first slots, chunk offsets and stats must match bit for
bit; the renormalised weights within 1e-6 absolute."""
import functools

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2609_21483_amd import workloads as W
from tests.cases import gate_filtered, make_case, oracle_logits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_21483_amd import binding
    return binding


@functools.lru_cache(maxsize=2)
def _tokens(name):
    return W.tokens(W.WORKLOADS[name])


class Handle:
    def __init__(self, B, shape):
        self.B = B
        self.h = B.moe_init(B.make_config(shape))
        self.ws = torch.empty(B.moe_workspace_size(self.h), dtype=torch.uint8, device="cuda")
        B.moe_set_workspace(self.h, self.ws)
        self.L = B.moe_workspace_layout(self.h)

    def view(self, name, n):
        off = getattr(self.L, name)
        return self.ws[off:off + 4 * n].view(torch.int32).cpu().numpy()

    def close(self):
        self.B.moe_destroy(self.h)


def check_tables(hd: Handle, shape, idx_ref):
    T, k, R, Tr, El = shape.T, shape.top_k, shape.n_src_ranks, shape.tokens_per_rank, shape.n_local_experts
    tab = O.route_tables(idx_ref, R, Tr, 0, El)
    assert np.array_equal(hd.view("slot", T * k).reshape(T, k), tab.slot)
    assert np.array_equal(hd.view("inv", tab.X), tab.inv)
    assert np.array_equal(hd.view("first_slot", T), tab.first_slot)
    assert np.array_equal(hd.view("off", El + 1), tab.off)
    assert np.array_equal(hd.view("cnt_rank", El * R).reshape(El, R), tab.cnt_rank)
    assert np.array_equal(hd.view("uniq", R), tab.uniq)
    st = hd.view("stats", 16)
    X_local = int(tab.cnt_rank[:, 0].sum())
    assert list(st[:6]) == [tab.X, X_local, tab.X - X_local, int(tab.uniq[0]), int(tab.uniq[1:].sum()), 0]
    sub = hd.view("sub_off", 4 * El * 9).reshape(4, El, 9)
    for ki, K in enumerate((1, 2, 4, 8)):
        assert np.array_equal(sub[ki, :, :K + 1], O.chunk_offsets(tab, T, k, K)), K
    return tab


ROUTE_CASES = [("tiny", 0), ("mixtral_ep4", 0), ("fine_zipf", 0), ("shared_routed", 0)] + \
    [("large_stack", l) for l in range(8)]


@pytest.mark.parametrize("name,layer", ROUTE_CASES, ids=[f"{n}-L{l}" for n, l in ROUTE_CASES])
def test_route_parity(B, name, layer):
    shape = W.WORKLOADS[name]
    c = make_case(shape, layer, weights=False) if name != "large_stack" else None
    if c is None:
        from tests.cases import Case
        c = Case(shape, layer, _tokens(name), W.gate(shape, layer), W.zipf_log_prior(shape, layer))
    idx_ref, w_ref = c.oracle_route()
    hd = Handle(B, shape)
    try:
        x = c.x.cuda()
        wg = c.wg.cuda()
        bias = None if c.bias is None else c.bias.cuda()
        idx = torch.full((shape.T, shape.top_k), -7, dtype=torch.int32, device="cuda")
        w = torch.zeros((shape.T, shape.top_k), dtype=torch.float32, device="cuda")
        B.moe_route(hd.h, x, wg, bias, shape.top_k, idx, w)
        assert B.moe_sync_status(hd.h) == B.MOE_OK, B.moe_last_error()
        idx_g = idx.cpu().numpy()
        mism = np.nonzero((idx_g != idx_ref).any(axis=1))[0]
        assert mism.size == 0, f"{mism.size} tokens differ, first {mism[:5]}"
        assert np.max(np.abs(w.cpu().numpy() - w_ref)) <= 1e-6
        check_tables(hd, shape, idx_ref)
        # the certified filter evaluated the defined logit of few experts per token
        cands = int(hd.view("stats", 16)[8])
        assert shape.T * shape.top_k <= cands <= min(shape.T * shape.n_experts, 3 * shape.T * shape.top_k), cands
    finally:
        hd.close()


def test_route_layers_on_several_streams(B):
    """Independent layers routed concurrently on three streams (as the bench
    routes the layers of a step), each with its own handle: ids, weights and
    routing tables are those of the oracle, as when routed one at a time."""
    shape = W.FINE_ZIPF
    layers = range(6)
    cases = [make_case(shape, l, weights=False) for l in layers]
    hds = [Handle(B, shape) for _ in layers]
    streams = [torch.cuda.Stream() for _ in range(3)]
    try:
        x = cases[0].x.cuda()
        args = []
        for c in cases:
            idx = torch.full((shape.T, shape.top_k), -7, dtype=torch.int32, device="cuda")
            w = torch.zeros((shape.T, shape.top_k), dtype=torch.float32, device="cuda")
            args.append((c.wg.cuda(), None if c.bias is None else c.bias.cuda(), idx, w))
        torch.cuda.synchronize()
        for rep in range(2):
            for l, (hd, (wg, bias, idx, w)) in enumerate(zip(hds, args)):
                B.moe_route(hd.h, x, wg, bias, shape.top_k, idx, w, stream=streams[l % 3])
            torch.cuda.synchronize()
            for l, (c, hd, (_, _, idx, w)) in enumerate(zip(cases, hds, args)):
                assert B.moe_sync_status(hd.h) == B.MOE_OK, B.moe_last_error()
                idx_ref, w_ref = c.oracle_route()
                assert np.array_equal(idx.cpu().numpy(), idx_ref), (rep, l)
                assert np.max(np.abs(w.cpu().numpy() - w_ref)) <= 1e-6, (rep, l)
                check_tables(hd, shape, idx_ref)
    finally:
        for hd in hds:
            hd.close()


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("Tr,H", [(40, 128), (4100, 1216)], ids=["gate", "filter"])
def test_route_ties_and_candidate_overflow(B, Tr, H, bias):
    """Exact ties on either gate: zero token rows tie every expert (all of them
    are the filter's candidates), duplicated gate columns tie expert pairs;
    equal logits go to the smaller id."""
    shape = W.MoeShape("ties", 98, 2, Tr, H, 64, 128, 8, 8)
    assert gate_filtered(shape.T, H, 128, 8) == (Tr == 4100)
    rng = np.random.default_rng(11)
    x = torch.from_numpy(rng.standard_normal((shape.T, shape.hidden)).astype(np.float32)).to(torch.bfloat16)
    x[[0, 7, 41]] = 0
    wg = torch.from_numpy(0.05 * rng.standard_normal((shape.hidden, shape.n_experts)).astype(np.float32)).to(torch.bfloat16)
    wg[:, 5] = wg[:, 3]
    wg[:, 40] = wg[:, 2]
    wg[:, 100] = wg[:, 99]
    b = torch.from_numpy((-0.1 * np.log(np.arange(1, shape.n_experts + 1))).astype(np.float32)) if bias else None
    bu = None if b is None else b.numpy()
    lg = oracle_logits(W.as_u16_numpy(x), W.as_u16_numpy(wg), bu)
    idx_ref, w_ref = O.softmax_topk(lg, shape.top_k)
    hd = Handle(B, shape)
    try:
        idx = torch.full((shape.T, shape.top_k), -7, dtype=torch.int32, device="cuda")
        w = torch.zeros((shape.T, shape.top_k), dtype=torch.float32, device="cuda")
        B.moe_route(hd.h, x.cuda(), wg.cuda(), None if b is None else b.cuda(), shape.top_k, idx, w)
        assert B.moe_sync_status(hd.h) == B.MOE_OK, B.moe_last_error()
        assert np.array_equal(idx.cpu().numpy(), idx_ref)
        assert np.max(np.abs(w.cpu().numpy() - w_ref)) <= 1e-6
        if not bias:
            assert list(idx_ref[0]) == list(range(8))
    finally:
        hd.close()


@pytest.mark.parametrize("R,Tr,E,k,El,skew", [
    (3, 45, 10, 3, 4, 0.0),      # ragged token count
    (1, 1, 8, 2, 8, 0.0),        # a single token
    (2, 300, 16, 4, 16, 0.0),    # every expert local
    (4, 77, 32, 8, 5, 2.5),      # heavy skew: empty local experts
    (2, 513, 64, 6, 16, 1.0),    # three table workgroups, the last of 2 tokens
    (4, 10000, 8, 8, 8, 0.0),    # 320000 pairs: every token has every expert
])
def test_build_tables_supplied_routing(B, R, Tr, E, k, El, skew):
    shape = W.MoeShape("t", 99, R, Tr, 64, 64, E, k, El)
    idx_ref, _ = W.random_routing(shape.T, E, k, seed=R * 1000 + Tr, skew=skew)
    hd = Handle(B, shape)
    try:
        idx = torch.from_numpy(idx_ref).cuda()
        B.moe_build_tables(hd.h, idx)
        assert B.moe_sync_status(hd.h) == B.MOE_OK
        check_tables(hd, shape, idx_ref)
    finally:
        hd.close()


# one table workgroup, of 512 and of 960 tokens; four of them, whose bad ids the counting step adds up
@pytest.mark.parametrize("Tr,rows", [(40, (5, 9, 11)), (300, (5, 290, 580)), (800, (5, 700, 1599))])
def test_bad_routing_ids_are_flagged(B, Tr, rows):
    shape = W.MoeShape("t", 99, 2, Tr, 64, 64, 8, 2, 4)
    idx_ref, _ = W.random_routing(shape.T, 8, 2, seed=3)
    bad = idx_ref.copy()
    r0, r1, r2 = rows
    bad[r0, 1] = 8           # out of range
    bad[r1, 1] = bad[r1, 0]  # repeated in a row
    bad[r2, 0] = -1
    hd = Handle(B, shape)
    try:
        B.moe_build_tables(hd.h, torch.from_numpy(bad).cuda())
        assert B.moe_sync_status(hd.h) == B.MOE_ERR_ROUTING
        # the flagged pairs are treated as not local; everything else is intact
        clean = bad.copy()
        clean[r0, 1] = 100
        clean[r1, 1] = 100
        clean[r2, 0] = 100
        tab = O.route_tables(clean, 2, Tr, 0, 4)
        assert np.array_equal(hd.view("slot", shape.T * 2).reshape(-1, 2), tab.slot)
        assert hd.view("stats", 16)[5] == 3
        assert B.moe_sync_status(hd.h) == B.MOE_OK  # the error word was cleared
    finally:
        hd.close()


@pytest.mark.parametrize("R,Tr,E,k,El,S", [
    (1, 256, 16, 2, 8, 1),       # the 512-token workgroup, half full
    (1, 257, 16, 2, 8, 0),       # a wavefront with one token
    (2, 256, 16, 2, 8, 1),       # full
    (3, 171, 16, 2, 8, 0),       # 513 tokens: the first size of the 960-token workgroup
    (4, 240, 128, 8, 64, 2),     # its last
    (31, 31, 128, 8, 64, 0),     # 961 tokens: the first size of several workgroups
    (4, 256, 128, 8, 64, 2),     # two full ones
    (5, 205, 128, 8, 64, 0),     # 1025 tokens: the last of three has one
    (2, 2048, 64, 8, 1, 0),      # one local expert
    (64, 1040, 64, 1, 64, 0),    # more count words than the table blocks sum themselves; 64 ranks
])
def test_build_tables_workgroup_edges(B, R, Tr, E, k, El, S):
    """Sizes where the table builder changes its launch; twice in a row on one
    workspace, so that the accumulators are seen to be zero again."""
    shape = W.MoeShape("t", 99, R, Tr, 64, 64, E, k, El, n_shared_experts=S)
    hd = Handle(B, shape)
    try:
        for rep in range(2):
            idx_ref, _ = W.random_routing(shape.T, E, k, seed=17 + rep, skew=0.8)
            idx = torch.from_numpy(idx_ref).cuda()
            B.moe_build_tables(hd.h, idx)
            assert B.moe_sync_status(hd.h) == B.MOE_OK
            tab = check_tables(hd, shape, idx_ref)
        # the row maps and tile counts over them
        bm, nt0, nt1 = B.moe_tile_geometry(hd.h)
        rof = hd.view("row_off", 4 * (El + S) * 9).reshape(4, El + S, 9)
        st = hd.view("stats", 16)
        for ki, K in enumerate((1, 2, 4, 8)):
            sub = O.chunk_offsets(tab, shape.T, k, K)
            bnd = [min((q * shape.T + K - 1) // K, Tr) for q in range(K + 1)]
            rows = np.array([np.diff(sub[le]) for le in range(El)] + [np.diff(bnd)] * S, np.int64)
            up = -(-rows // 32) * 32
            start = np.concatenate([[0], np.cumsum(up.reshape(-1))[:-1]]).reshape(El + S, K)
            assert np.array_equal(rof[ki, :, :K], start) and not rof[ki, :, K:].any(), K
            assert st[10 + ki] == int((-(-rows // bm)).sum()) * (nt0 + nt1), K
    finally:
        hd.close()


# gate classes and launch shapes: (T, H, E, k, bias)
GATES = [
    (1, 64, 1, 1, False), (17, 64, 8, 8, True), (5, 192, 3, 2, True),       # one stage of h; padded rows
    (4097, 128, 16, 4, False), (40000, 64, 7, 3, True),                     # 16 experts: small shape, large shape
    (2049, 128, 32, 5, True), (20000, 64, 30, 4, False),                    # 32
    (1025, 192, 33, 6, False), (9000, 64, 64, 8, True),                     # 64
    (31, 320, 65, 8, True), (1030, 128, 128, 3, False), (5000, 64, 126, 8, True),  # 128
    (300, 128, 129, 8, True), (1100, 64, 256, 1, False), (3000, 96 * 2, 200, 7, True),  # 256
    (67, 128, 257, 4, False), (1500, 64, 512, 8, True),                     # 512
    # the classes up to 64 experts with one token wavefront a workgroup or with several, and 16 in the large shape
    (5000, 128, 8, 2, True), (100, 128, 12, 3, False), (33000, 64, 16, 4, True), (500, 128, 24, 4, True), (300, 128, 48, 6, False),
    (32768, 64, 66, 2, True), (16384, 1536, 72, 4, False), (32768, 4096, 130, 1, False),  # many tokens (two by the filter)
]


@pytest.mark.parametrize("T,H,E,k,bias", GATES)
def test_gate_classes(B, T, H, E, k, bias):
    """Every expert class and launch shape of the gate, ragged token counts and
    expert counts, a row of zeros and tied experts: ids bit for bit."""
    rng = torch.Generator().manual_seed(T * 1000 + E)
    x = torch.randn(T, H, generator=rng).to(torch.bfloat16)
    wg = (0.05 * torch.randn(H, E, generator=rng)).to(torch.bfloat16)
    x[T // 2] = 0
    if E > 2:
        wg[:, E - 1] = wg[:, 1]
    b = torch.randn(E, generator=rng) if bias else None
    lg = oracle_logits(W.as_u16_numpy(x), W.as_u16_numpy(wg), None if b is None else b.numpy())
    idx_ref, w_ref = O.softmax_topk(lg, k)
    idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k), dtype=torch.float32, device="cuda")
    B.moe_route_topk_static(T, H, E, k, x.cuda(), wg.cuda(), None if b is None else b.cuda(), idx, w)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    assert np.max(np.abs(w.cpu().numpy() - w_ref)) <= 1e-6


# one problem for each kernel of the filter: logit tiles of 64 and of 128
# tokens, E <= 128 and above, and chains k < 4, k < 8, k = 8
FILTER_GATES = [(8200, 832, 66, 1, False), (8300, 1088, 100, 6, True), (8200, 1216, 66, 8, True),
                (33000, 512, 66, 1, True), (32800, 384, 66, 4, False), (33000, 448, 66, 8, False),
                (8200, 2880, 34, 1, True), (16600, 1728, 48, 4, False), (16700, 1920, 64, 4, True),  # 33 to 64 experts
                (4100, 1472, 257, 2, True), (8300, 2048, 300, 8, False), (41000, 1600, 129, 1, True)]


@pytest.mark.parametrize("T,H,E,k,bias", FILTER_GATES)
def test_gate_filter_classes(B, T, H, E, k, bias):
    assert gate_filtered(T, H, E, k)
    test_gate_classes(B, T, H, E, k, bias)


def test_gate_masked_experts(B):
    """A bias of -inf or of the lowest float takes an expert out unless too few
    are left, when the masked ones follow by id with weight 0; a NaN logit is
    never chosen."""
    T, H, E, k = 40, 128, 12, 4
    rng = torch.Generator().manual_seed(5)
    x = torch.randn(T, H, generator=rng).to(torch.bfloat16)
    wg = (0.05 * torch.randn(H, E, generator=rng)).to(torch.bfloat16)
    for keep, low in ((6, float("-inf")), (6, torch.finfo(torch.float32).min), (2, float("-inf"))):
        b = torch.zeros(E)
        b[keep:] = low
        lg = O.gate_logits(W.as_u16_numpy(x), W.as_u16_numpy(wg), b.numpy())
        order = np.argsort(-lg.astype(np.float64), axis=1, kind="stable")[:, :k]
        idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
        w = torch.zeros((T, k), dtype=torch.float32, device="cuda")
        B.moe_route_topk_static(T, H, E, k, x.cuda(), wg.cuda(), b.cuda(), idx, w)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), order), (keep, low)
        wn = w.cpu().numpy()
        assert np.all(wn[:, keep:] == 0) and np.allclose(wn.sum(axis=1), 1, atol=1e-6)
    b = torch.zeros(E)
    b[3] = float("nan")
    idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
    B.moe_route_topk_static(T, H, E, k, x.cuda(), wg.cuda(), b.cuda(), idx, torch.zeros((T, k), device="cuda"))
    torch.cuda.synchronize()
    got = idx.cpu().numpy()
    assert not np.any(got == 3) and got.min() >= 0 and got.max() < E


@pytest.mark.parametrize("T,H,E,k", [
    (100, 832, 66, 4), (300, 320, 257, 3),                            # the gate that evaluates every logit
    (8200, 960, 66, 3), (8300, 1088, 100, 6), (8200, 1216, 66, 8),    # the filter, E <= 128
    (4100, 1472, 257, 2), (8300, 2048, 300, 8),                       # the filter above 128 experts
])
def test_gate_infinities_and_nans(B, T, H, E, k):
    """Masked experts (bias -inf or the lowest float), too few of them left,
    biases of +inf and NaN, and tokens with infinite, NaN, huge and zero values:
    the ids of the defined logits from either gate, ties to the smaller id, NaN
    never chosen (no id left: 1 << 30)."""
    assert gate_filtered(T, H, E, k) == (T > 4000)
    rng = torch.Generator().manual_seed(T + E)
    x = torch.randn(T, H, generator=rng).to(torch.bfloat16)
    wg = (0.05 * torch.randn(H, E, generator=rng)).to(torch.bfloat16)
    x[3, 5] = float("inf")
    x[4, 7] = float("-inf")
    x[5, 0] = float("nan")
    x[6] *= 1e30
    x[7] *= 3e37
    x[8] = 0
    base = oracle_logits(W.as_u16_numpy(x), W.as_u16_numpy(wg), None)
    inf, low = float("inf"), torch.finfo(torch.float32).min
    left, cut = torch.arange(E) % (E // (k + 2)) == 1, torch.arange(E) >= max(k - 2, 1)
    biases = {"none": None, "masked": torch.where(left, 0.0, -inf), "lowest": torch.where(left, 0.0, low),
              "few": torch.where(cut, -inf, 0.0), "few_lowest": torch.where(cut, low, 0.0),
              "plus": torch.where(torch.arange(E) == E - 2, inf, 0.0),
              "nan": torch.where(torch.arange(E) % 3 == 0, float("nan"), 0.0)}
    xd, wd = x.cuda(), wg.cuda()
    for name, b in biases.items():
        with np.errstate(invalid="ignore", over="ignore"):
            lg = (base if b is None else base + b.numpy()).astype(np.float64)
        nan = np.isnan(lg)
        order = np.lexsort((np.broadcast_to(np.arange(E), lg.shape), -np.where(nan, -inf, lg), nan), axis=1)[:, :k]
        ref = np.where(np.take_along_axis(nan, order, 1), 1 << 30, order)
        idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
        w = torch.zeros((T, k), device="cuda")
        B.moe_route_topk_static(T, H, E, k, xd, wd, None if b is None else b.cuda(), idx, w)
        torch.cuda.synchronize()
        bad = np.nonzero((idx.cpu().numpy() != ref).any(axis=1))[0]
        assert bad.size == 0, (name, bad[:5], idx[bad[0]].tolist(), ref[bad[0]], lg[bad[0]][ref[bad[0]] % E])
        if name in ("masked", "few", "lowest", "few_lowest"):
            rows, top = slice(9, None), np.take_along_axis(lg, order, 1)[9:]
            p = np.exp(top - top[:, :1])
            assert np.max(np.abs(w.cpu().numpy()[rows] - p / p.sum(1, keepdims=True))) <= 1e-6, name


@pytest.mark.parametrize("R,Tr,H,E", [(1, 1200, 128, 64), (2, 4150, 1216, 66)])  # the gate; the filter
def test_tokens_without_valid_ids_are_flagged(B, R, Tr, H, E):
    """Tokens whose logits are all NaN get no valid id: moe_route reports and
    counts them, and the other tokens' tables are intact (the gate's own count
    blocks, more than one workgroup of the table builder)."""
    k, El = 8, 8
    shape = W.MoeShape("nan_rows", 97, R, Tr, H, 64, E, k, El)
    T = shape.T
    assert gate_filtered(T, H, E, k) == (T > 4000)
    rng = torch.Generator().manual_seed(5)
    x = torch.randn(T, H, generator=rng).to(torch.bfloat16)
    wg = (0.05 * torch.randn(H, E, generator=rng)).to(torch.bfloat16)
    rows = [0, 511, 512, T - 1]
    x[rows, 1] = float("nan")
    hd = Handle(B, shape)
    try:
        idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
        w = torch.zeros((T, k), device="cuda")
        B.moe_route(hd.h, x.cuda(), wg.cuda(), None, k, idx, w)
        assert B.moe_sync_status(hd.h) == B.MOE_ERR_ROUTING
        got = idx.cpu().numpy()
        assert np.all(got[rows] == 1 << 30)
        tab = O.route_tables(got, R, Tr, 0, El)
        assert np.array_equal(hd.view("slot", T * k).reshape(T, k), tab.slot)
        assert np.array_equal(hd.view("off", El + 1), tab.off)
        assert hd.view("stats", 16)[5] == len(rows)
        assert B.moe_sync_status(hd.h) == B.MOE_OK
    finally:
        hd.close()


def _view_at(t, off):
    """t's values in a contiguous view that starts off values into a buffer."""
    buf = torch.zeros(t.numel() + off, dtype=t.dtype, device="cuda")
    v = buf[off:].view(t.shape)
    v.copy_(t)
    assert v.is_contiguous() and v.data_ptr() % 16 == 2 * off % 16
    return v


@pytest.mark.parametrize("xo,wo", [(0, 1), (0, 4), (1, 0), (4, 3)])
@pytest.mark.parametrize("T,H,E,k", [
    (65, 192, 8, 2), (300, 64, 128, 8), (70, 128, 30, 4),   # rows of a multiple of 4 values, and not
    (8200, 960, 66, 4),                                     # the filter
    (8000, 8192, 8, 2),                                     # more rows than the static scratch holds
])
def test_operands_off_a_16_byte_boundary(B, T, H, E, k, xo, wo):
    """Views that start anywhere in a larger buffer are routed as their aligned
    copies are, by both entry points."""
    rng = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(T, H, device="cuda", generator=rng).to(torch.bfloat16)
    wg = (0.05 * torch.randn(H, E, device="cuda", generator=rng)).to(torch.bfloat16)
    shape = W.MoeShape("views", 96, 1, T, H, 64, E, k, min(4, E))
    hd = Handle(B, shape)
    try:
        out = []
        for xv, wv in ((x, wg), (_view_at(x, xo), _view_at(wg, wo))):
            for route in (lambda *a: B.moe_route(hd.h, xv, wv, None, k, *a),
                          lambda *a: B.moe_route_topk_static(T, H, E, k, xv, wv, None, *a)):
                idx = torch.full((T, k), -7, dtype=torch.int32, device="cuda")
                w = torch.zeros((T, k), device="cuda")
                route(idx, w)
                assert B.moe_sync_status(hd.h) == B.MOE_OK
                out.append((idx, w))
        for idx, w in out[1:]:
            assert torch.equal(idx, out[0][0]) and torch.equal(w, out[0][1])
    finally:
        hd.close()
