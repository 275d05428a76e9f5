"""GPU parity of the pieces around the layer path: attention recall (Section 3.1) and k-means++ seeding
(Sections 4.3 / 5.3), each against the CPU oracle on the same seeded inputs."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2505_18875_amd import workloads as wl
from _util import head_inputs, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def svg2():
    import paper_2505_18875_amd as pkg
    pkg.load_library()
    assert torch.cuda.is_available()
    return pkg


def _dense_lse(svg2, Q, K, V):
    H, N, _ = Q.shape
    one = torch.tensor([[0, N]] * H, dtype=torch.int32, device="cuda")
    rp = torch.tensor([[0, 1]] * H, dtype=torch.int32, device="cuda")
    ci = torch.zeros((H, 1), dtype=torch.int32, device="cuda")
    return svg2.svg2_sparse_attn(Q, K, V, one, one, rp, ci, None, want_lse=True).lse


@pytest.mark.parametrize("name,heads,top_p,sample", [("tiny", [0], 0.9, None), ("small", [2, 19], 0.9, 512),
                                                     ("small", [7], 0.5, 512)])
def test_attention_recall_matches_oracle(svg2, oracle, name, heads, top_p, sample):
    w = wl.replace(wl.WORKLOADS[name], top_p=top_p)
    Q, K, V, cq, ck = head_inputs(w, heads)
    Qd, Kd, Vd = (to_dev(x, w.dtype) for x in (Q, K, V))
    res = svg2.svg2_forward(Qd, Kd, Vd, to_dev(cq), to_dev(ck), w.top_p, w.iters, want_aux=True)
    lse_all = _dense_lse(svg2, Qd, Kd, Vd)
    rec = svg2.svg2_attention_recall(res.aux.lse, lse_all)
    torch.cuda.synchronize()
    a = res.aux
    for i, h in enumerate(heads):
        rows = None if sample is None else np.sort(
            np.random.default_rng(h).choice(w.N, sample, replace=False)).astype(np.int32)
        rp, ci = to_np(a.row_ptr[i]), to_np(a.col_idx[i])
        want = oracle.attention_recall(Q[i], K[i], to_np(a.labels_q[i]), to_np(a.labels_k[i]), w.Cq, w.Ck,
                                       rp, ci[: rp[-1]], rows=rows)
        chk = np.arange(w.N) if rows is None else rows
        got = to_np(rec.recall[i])
        # the two lse values are fp32 results of bf16 / fp32 attention passes: a few 1e-3 absolute on a ratio in [0,1]
        np.testing.assert_allclose(got[chk], want[chk], atol=4e-3, rtol=4e-3)
        np.testing.assert_allclose(float(rec.mean[i]), got.mean(), rtol=1e-5)
        assert got.min() >= 0.0 and got.max() <= 1.0 + 1e-3
    # everything selected: recall is exactly 1
    one = svg2.svg2_attention_recall(lse_all, lse_all)
    torch.cuda.synchronize()
    assert torch.all(one.recall == 1.0) and torch.all(one.mean == 1.0)


@pytest.mark.parametrize("name,heads,C", [("tiny", [0], 32), ("small", [0, 9, 23], 100), ("small", [4], 500)])
def test_kmeans_pp_matches_oracle(svg2, oracle, name, heads, C):
    w = wl.WORKLOADS[name]
    Q, K, V, _, _ = head_inputs(w, heads)
    u = np.random.default_rng(11).random((len(heads), C))
    res = svg2.svg2_kmeans_pp_init(to_dev(K, w.dtype), C, torch.from_numpy(u).cuda())
    torch.cuda.synchronize()
    for i in range(len(heads)):
        picked, centres = oracle.kmeans_pp(K[i], C, u[i])
        np.testing.assert_array_equal(to_np(res.picked[i]), picked)
        np.testing.assert_array_equal(to_np(res.centroids[i]), centres)


def test_kmeans_pp_degenerate_inputs(svg2, oracle):
    # all tokens identical: every D2 is zero and the draw falls back to token floor(u N); duplicates of one token
    X = np.ones((1, 300, 64), dtype=np.float32)
    u = np.array([[0.01, 0.5, 0.999, 0.25]])
    res = svg2.svg2_kmeans_pp_init(to_dev(X), 4, torch.from_numpy(u).cuda())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_np(res.picked[0]), oracle.kmeans_pp(X[0], 4, u[0])[0])
    np.testing.assert_array_equal(to_np(res.picked[0]), [3, 150, 299, 75])
    # ragged N (not a multiple of the 1024-token block), two distinct values
    X = np.zeros((1, 1500, 128), dtype=np.float32)
    X[0, 1100:] = 2.0
    u = np.array([[0.0, 0.3, 0.9]])
    res = svg2.svg2_kmeans_pp_init(to_dev(X, "bf16"), 3, torch.from_numpy(u).cuda())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_np(res.picked[0]), oracle.kmeans_pp(X[0], 3, u[0])[0])


@pytest.mark.parametrize("H,N,d,C,dtype,comps", [
    (1, 1, 64, 1, "bf16", 1), (1, 255, 128, 40, "f32", 5), (2, 257, 64, 257, "bf16", 30),
    (3, 2000, 128, 300, "bf16", 2000),        # no structure: hardly a token is left out
    (5, 6001, 64, 90, "f32", 12), (2, 400001, 64, 9, "bf16", 3), (1, 1700000, 64, 3, "bf16", 2)])
def test_kmeans_pp_block_edges_and_skipped_tokens(svg2, oracle, H, N, d, C, dtype, comps):
    """Lengths around a chunk of 256 tokens, workgroups with one chunk and with several, one centre and as many as tokens,
    components far enough apart that most tokens are left out of a draw."""
    r = np.random.default_rng(700 + N)
    centres = (4.0 * r.standard_normal((comps, d))).astype(np.float32)
    X = centres[np.sort(r.integers(0, comps, size=(H, N)), axis=1)] + r.standard_normal((H, N, d), dtype=np.float32)
    X = wl.round_to_bf16(X) if dtype == "bf16" else X
    u = r.random((H, C))
    res = svg2.svg2_kmeans_pp_init(to_dev(X, dtype), C, torch.from_numpy(u).cuda())
    torch.cuda.synchronize()
    for i in range(H):
        picked, rows = oracle.kmeans_pp(X[i], C, u[i])
        np.testing.assert_array_equal(to_np(res.picked[i]), picked)
        np.testing.assert_array_equal(to_np(res.centroids[i]), rows)


@pytest.mark.parametrize("dtype,magnitude", [("bf16", 1e-9), ("bf16", 3e-10), ("f32", 1e-15), ("bf16", 1e-20), ("f32", 1e-20),
                                             ("bf16", 1e-21), ("bf16", 2e-21), ("f32", 1e-21), ("bf16", 1e-25)])
def test_kmeans_pp_tokens_whose_squares_underflow(svg2, oracle, dtype, magnitude):
    """The fp32 bound that rules tokens out of a draw works with squares; the draws have to be the oracle's (fp64) also
    where these are denormal or zero in fp32, and around the limit below which every token is measured."""
    r = np.random.default_rng(41)
    centres = 2.0 * r.standard_normal((40, 128))
    X = centres[np.sort(r.integers(0, 40, size=4000))] + 0.3 * r.standard_normal((4000, 128))
    X = (magnitude * X).astype(np.float32)
    X = wl.round_to_bf16(X) if dtype == "bf16" else X
    u = r.random((1, 120))
    res = svg2.svg2_kmeans_pp_init(to_dev(X[None], dtype), 120, torch.from_numpy(u).cuda())
    torch.cuda.synchronize()
    picked, rows = oracle.kmeans_pp(X, 120, u[0])
    np.testing.assert_array_equal(to_np(res.picked[0]), picked)
    np.testing.assert_array_equal(to_np(res.centroids[0]), rows)


def test_kmeans_pp_then_lloyd_lowers_the_objective(svg2):
    # seeding feeds svg2_kmeans: the objective after the first assign step is the k-means++ potential and it
    # does not grow over the iterations (Section 4.1 / 4.3)
    w = wl.WORKLOADS["small"]
    Q, K, V, _, _ = head_inputs(w, [1])
    Kd = to_dev(K, w.dtype)
    u = torch.from_numpy(np.random.default_rng(3).random((1, 50))).cuda()
    init = svg2.svg2_kmeans_pp_init(Kd, 50, u).centroids
    res = svg2.svg2_kmeans(Kd, init, 6, want_objective=True)
    torch.cuda.synchronize()
    obj = to_np(res.objective[0])
    assert np.all(np.diff(obj) <= 1e-4 * obj[0])


def _seeding_case(dtype, H, N, d, C):
    r = np.random.default_rng(9100 + N + d)
    centres = 1.5 * r.standard_normal((H, 9, d)).astype(np.float32)
    X = np.stack([centres[h][np.sort(r.integers(0, 9, size=N))] for h in range(H)]) + r.standard_normal((H, N, d)).astype(np.float32)
    X = wl.round_to_bf16(X) if dtype == "bf16" else X.astype(np.float32)
    u = r.random((H, C))
    return X, u, to_dev(X, dtype), torch.from_numpy(u).cuda()


def _check_draws(oracle, X, u, picked, cent):
    H, C = u.shape
    for h in range(0, H, max(1, H // 3)):
        ref, centres = oracle.kmeans_pp(X[h], C, u[h])
        np.testing.assert_array_equal(to_np(picked[h]), ref)
        np.testing.assert_array_equal(to_np(cent[h]), centres)


@pytest.mark.parametrize("dtype,H,N,d,C", [
    # one workgroup per head, the most it holds and a chunk more; several, and a ragged last one; a launch per draw
    ("bf16", 2, 2048, 64, 40), ("bf16", 2, 2049, 128, 40), ("f32", 3, 5000, 128, 60), ("bf16", 24, 16384, 128, 12),
    ("bf16", 1, 65536, 64, 30), ("bf16", 1, 65537, 64, 5), ("bf16", 140, 2300, 64, 6)])
def test_kmeans_pp_draws_of_one_launch(svg2, oracle, dtype, H, N, d, C):
    """All draws of a head in one launch: the tokens of the oracle's draws."""
    X, u, Xd, ud = _seeding_case(dtype, H, N, d, C)
    res = svg2.svg2_kmeans_pp_init(Xd, C, ud)
    torch.cuda.synchronize()
    _check_draws(oracle, X, u, res.picked, res.centroids)


def _test_library():
    from paper_2505_18875_amd import build
    lib = ctypes.CDLL(build.TEST_LIB)
    lib.svg2_test_kmeans_pp_given_up.restype = ctypes.c_size_t
    return lib


@pytest.mark.parametrize("dtype,H,N,d,C", [
    # several workgroups per head
    ("bf16", 2, 2049, 128, 40), ("f32", 3, 5000, 128, 60), ("bf16", 24, 16384, 128, 12), ("bf16", 1, 65536, 64, 30)])
def test_kmeans_pp_heads_that_are_given_up_are_done_again(svg2, oracle, dtype, H, N, d, C):
    """Without patience a workgroup gives its head up at its first look for the others' sums; a single workgroup
    then does the head again."""
    X, u, Xd, ud = _seeding_case(dtype, H, N, d, C)
    lib = _test_library()
    picked = torch.full((H, C), -1, dtype=torch.int32, device="cuda")
    cent = torch.zeros((H, C, d), dtype=torch.float32, device="cuda")
    ws = torch.zeros(svg2.load_library().svg2_kmeans_pp_init_workspace_size(H, N, C), dtype=torch.uint8, device="cuda")
    vp = ctypes.c_void_p
    rc = lib.svg2_test_kmeans_pp_init(
        vp(Xd.data_ptr()), svg2.SVG2_BF16 if dtype == "bf16" else svg2.SVG2_F32, H, N, d, C, vp(ud.data_ptr()),
        vp(cent.data_ptr()), vp(picked.data_ptr()), vp(ws.data_ptr()), 0, vp(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    at = lib.svg2_test_kmeans_pp_given_up(H, N, d, C)
    assert torch.equal(ws[at:at + 4 * H].view(torch.int32), torch.ones(H, dtype=torch.int32, device="cuda"))
    _check_draws(oracle, X, u, picked, cent)


def test_kmeans_pp_waiting_workgroups_fit_the_streams_compute_units(svg2):
    """The workgroups that wait for one another are at most as many as the CUs that the stream may use.  (The mask has bits in every
    group of 32 and of 8 CUs; nothing is launched on the stream.)"""
    lib, vp = _test_library(), ctypes.c_void_p
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = [(24, 16384), (1, 65536), (10, 30000), (1, 2048), (40, 75600)]
    whole = [lib.svg2_test_kmeans_pp_waiting(H, N, vp(torch.cuda.current_stream().cuda_stream)) for H, N in shapes]
    # chunks of 256 tokens, 2, 4, 6 or 8 of them to a workgroup
    assert cus < 256 or whole == [192, 128, 200, 0, 0]
    for bits, n in ((0xFFFF, cus // 2), (0xFF, cus // 4)):
        mask = (ctypes.c_uint32 * (cus // 32))(*[bits] * (cus // 32))
        st = vp()
        assert lib.hipExtStreamCreateWithCUMask(ctypes.byref(st), len(mask), mask) == 0
        part = [lib.svg2_test_kmeans_pp_waiting(H, N, st) for H, N in shapes]
        assert lib.hipStreamDestroy(st) == 0
        assert all(0 <= p <= n for p in part) and part[1] == min(whole[1], n)


def test_kmeans_pp_in_a_graph(svg2):
    # several workgroups per head; the draws change with u between replays
    X, u, Xd, ud = _seeding_case("bf16", 3, 5000, 128, 20)
    ws = torch.empty(svg2.load_library().svg2_kmeans_pp_init_workspace_size(3, 5000, 20), dtype=torch.uint8, device="cuda")
    svg2.svg2_kmeans_pp_init(Xd, 20, ud, ws=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        res = svg2.svg2_kmeans_pp_init(Xd, 20, ud, ws=ws)
    for i in range(4):
        ud.copy_(torch.from_numpy(np.random.default_rng(i).random((3, 20))))
        g.replay()
        torch.cuda.synchronize()
        eager = svg2.svg2_kmeans_pp_init(Xd, 20, ud)
        torch.cuda.synchronize()
        assert torch.equal(res.picked, eager.picked) and torch.equal(res.centroids, eager.centroids)
