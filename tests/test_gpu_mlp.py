"""GPU parity of the cost model's network kernels against the FP64 oracle:
logits, loss and every gradient tensor within 1e-5 relative (norm), and one
Adam step within 1e-5 relative.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DIMS = (16, 64, 64, 48)


def _params(g, F, H1, H2, K):
    return {"W1": g.standard_normal((H1, F)) * 0.4, "b1": g.standard_normal(H1) * 0.1,
            "W2": g.standard_normal((H2, H1)) * 0.2, "b2": g.standard_normal(H2) * 0.1,
            "W3": g.standard_normal((K, H2)) * 0.2, "b3": g.standard_normal(K) * 0.1}


def _flat(P):
    return np.concatenate([P[k].ravel() for k in ("W1", "b1", "W2", "b2", "W3", "b3")])


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("B", [1, 7, 256, 4096])
def test_loss_grad_vs_oracle(gpu_lib, B):
    om = gpu_lib
    F, H1, H2, K = DIMS
    g = np.random.Generator(np.random.PCG64(B))
    P = _params(g, F, H1, H2, K)
    P32 = {k: v.astype(np.float32) for k, v in P.items()}
    X = g.standard_normal((B, F)).astype(np.float32)
    y = g.integers(0, K, B).astype(np.int32)
    loss_ref, Z_ref, g_ref = oracle.mlp_loss_grad(X.astype(np.float64), y,
                                                  {k: v.astype(np.float64) for k, v in P32.items()})
    params = torch.from_numpy(_flat(P32)).cuda()
    assert params.numel() == om.mlp_param_count(*DIMS)
    Xd = torch.from_numpy(X).cuda()
    yd = torch.from_numpy(y).cuda()
    Z = torch.zeros((B, K), dtype=torch.float32, device="cuda")
    om.mlp_forward(DIMS, params, Xd, Z)
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    grads = torch.zeros_like(params)
    om.mlp_loss_grad(DIMS, params, Xd, yd, loss, grads)
    torch.cuda.synchronize()
    assert _rel(Z.cpu().numpy().astype(np.float64), Z_ref) < 1e-5
    assert abs(loss.item() - loss_ref) <= 1e-5 * abs(loss_ref)
    gh = grads.cpu().numpy().astype(np.float64)
    off = 0
    for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
        sz = g_ref[k].size
        assert _rel(gh[off:off + sz], g_ref[k].ravel()) < 1e-5, k
        off += sz


@pytest.mark.parametrize("dims", [(16, 64, 64, 64), (1, 1, 1, 2), (5, 33, 7, 3), (17, 32, 96, 24),
                                  (16, 96, 96, 64), (16, 97, 66, 130), (16, 128, 128, 64),
                                  (16, 160, 200, 10)])
@pytest.mark.parametrize("B", [1, 5, 512, 513, 1025])
def test_network_shapes_vs_oracle(gpu_lib, dims, B):
    """Networks on both sides of the LDS limit, layer widths off whole 16-byte
    blocks and off whole waves, batches at the edges of the row tiles (4 and 16
    rows) and of the gradient slices (512 rows), parameters off 16-byte alignment."""
    om = gpu_lib
    F, H1, H2, K = dims
    g = np.random.Generator(np.random.PCG64(B))
    P32 = {k: v.astype(np.float32) for k, v in _params(g, F, H1, H2, K).items()}
    X = g.standard_normal((B, F)).astype(np.float32)
    y = g.integers(0, K, B).astype(np.int32)
    loss_ref, Z_ref, g_ref = oracle.mlp_loss_grad(X.astype(np.float64), y,
                                                  {k: v.astype(np.float64) for k, v in P32.items()})
    ref = np.concatenate([g_ref[k].ravel() for k in ("W1", "b1", "W2", "b2", "W3", "b3")])
    flat = torch.from_numpy(_flat(P32))
    for shift in (0, 1):
        params = torch.zeros(flat.numel() + shift, device="cuda")[shift:]
        params.copy_(flat)
        Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
        Z = torch.zeros((B, K), dtype=torch.float32, device="cuda")
        om.mlp_forward(dims, params, Xd, Z)
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        grads = torch.full_like(params, float("nan"))
        om.mlp_loss_grad(dims, params, Xd, yd, loss, grads)
        torch.cuda.synchronize()
        assert _rel(Z.cpu().numpy().astype(np.float64), Z_ref) < 1e-5
        assert abs(loss.item() - loss_ref) <= 1e-5 * abs(loss_ref)
        gh = grads.cpu().numpy().astype(np.float64)
        off = 0
        for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
            sz = g_ref[k].size
            assert _rel(gh[off:off + sz], ref[off:off + sz]) < 1e-5, (k, shift)
            off += sz


def test_adam_vs_oracle(gpu_lib):
    om = gpu_lib
    g = np.random.Generator(np.random.PCG64(3))
    n = 10_000
    w = g.standard_normal(n).astype(np.float32)
    m = (g.standard_normal(n) * 0.01).astype(np.float32)
    v = np.abs(g.standard_normal(n) * 0.001).astype(np.float32)
    gr = g.standard_normal(n).astype(np.float32)
    wd, md, vd, gd = (torch.from_numpy(a.copy()).cuda() for a in (w, m, v, gr))
    om.mlp_adam(wd, md, vd, gd, 7, lr=1e-2)
    torch.cuda.synchronize()
    # the kernel receives fp32 hyperparameters: give the oracle the same values
    f32 = lambda v: float(np.float32(v))
    w2, m2, v2 = oracle.adam(w, m, v, gr, 7, lr=f32(1e-2), beta1=f32(0.9), beta2=f32(0.999),
                             eps=f32(1e-8))
    assert _rel(wd.cpu().numpy(), w2) < 1e-6
    assert _rel(md.cpu().numpy(), m2) < 1e-6
    assert _rel(vd.cpu().numpy(), v2) < 1e-6


def test_adam_counted_equals_adam(gpu_lib):
    """The step number in device memory gives the update of omprt_mlp_adam at that step,
    bit for bit, and advances the counter by one per call."""
    om = gpu_lib
    g = np.random.Generator(np.random.PCG64(3))
    n = 9000
    p = torch.from_numpy(g.standard_normal(n).astype(np.float32)).cuda()
    a = [p.clone(), torch.zeros_like(p), torch.zeros_like(p)]
    b = [p.clone(), torch.zeros_like(p), torch.zeros_like(p)]
    step = torch.zeros(1, dtype=torch.int32, device="cuda")
    for t in range(1, 6):
        grads = torch.from_numpy(g.standard_normal(n).astype(np.float32)).cuda()
        om.mlp_adam(a[0], a[1], a[2], grads, t, lr=1e-2)
        om.mlp_adam_counted(b[0], b[1], b[2], grads, step, lr=1e-2)
        torch.cuda.synchronize()
        for u, w in zip(a, b):
            assert torch.equal(u.view(torch.int32), w.view(torch.int32)), t
        assert int(step.item()) == t


@pytest.mark.parametrize("n", [1, 256, 257, 20_000])
@pytest.mark.parametrize("captured", [False, True])
def test_adam_counted_sizes(gpu_lib, n, captured):
    """One workgroup and several; eager (the step advanced by the last workgroup) and
    captured on a stream without a workspace (by a launch of its own), replayed."""
    om = gpu_lib
    g = np.random.Generator(np.random.PCG64(n))
    p = torch.from_numpy(g.standard_normal(n).astype(np.float32)).cuda()
    grads = torch.from_numpy(g.standard_normal(n).astype(np.float32)).cuda()
    a = [p.clone(), torch.zeros_like(p), torch.zeros_like(p)]
    b = [p.clone(), torch.zeros_like(p), torch.zeros_like(p)]
    step = torch.full((1,), 6, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    graph = None
    if captured:
        om.finalize()   # no stream has a workspace any more
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            om.mlp_adam_counted(b[0], b[1], b[2], grads, step, lr=1e-2)
    for t in (7, 8, 9):
        om.mlp_adam(a[0], a[1], a[2], grads, t, lr=1e-2)
        if captured:
            graph.replay()
        else:
            om.mlp_adam_counted(b[0], b[1], b[2], grads, step, lr=1e-2)
        torch.cuda.synchronize()
        for u, w in zip(a, b):
            assert torch.equal(u.view(torch.int32), w.view(torch.int32)), t
        assert int(step.item()) == t


def test_training_graph_replays_match_eager(gpu_lib):
    """One epoch of training steps captured in a HIP graph and replayed every epoch
    (with the epoch's permutation done eagerly between replays) makes the same
    parameters, bit for bit, as the steps launched one by one and as the plain loop
    that copies every batch from the host and reads every loss back."""
    from paper_2106_03219_amd import train as tr
    om = gpu_lib
    g = np.random.Generator(np.random.PCG64(11))
    X = g.standard_normal((1000, 16)).astype(np.float32)
    y = g.integers(0, tr.DIMS[3], 1000).astype(np.int32)
    out = {}
    for mode in ("sync", "eager", "graph"):
        logs = []
        p = tr.train(om, torch, X, y, epochs=4, batch=96, lr=1e-3, seed=5, mode=mode,
                     log=logs.append)
        out[mode] = (p.cpu().numpy(), logs)
    for mode in ("eager", "graph"):
        assert np.array_equal(out[mode][0].view(np.uint32), out["sync"][0].view(np.uint32)), mode
    assert out["graph"][1][-1].split()[-1] == out["eager"][1][-1].split()[-1]


def test_adam_graph_beside_reductions(gpu_lib):
    """A graph of the counted Adam step alone, replayed on another stream while the stream that it
    was captured on runs reductions: the two share nothing."""
    om = gpu_lib
    n, reps = 9472, 300
    g = np.random.Generator(np.random.PCG64(3))
    state = [torch.from_numpy(g.standard_normal(n).astype(np.float32)).cuda() for _ in range(2)]
    a, b = ([state[0].clone(), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")]
            for _ in range(2))
    grads = state[1]
    step = torch.zeros(1, dtype=torch.int32, device="cuda")
    big = torch.ones(1 << 24, dtype=torch.int32, device="cuda")
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    xs = torch.zeros(reps, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        om.reduce(big, "sum", xs[:1])
    s.synchronize()
    xs.zero_()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        om.mlp_adam_counted(b[0], b[1], b[2], grads, step, lr=1e-2)
    torch.cuda.synchronize()
    for k in range(reps):
        with torch.cuda.stream(s):
            om.reduce(big, "sum", xs[k:k + 1])
        with torch.cuda.stream(t):
            graph.replay()
    for k in range(reps):
        om.mlp_adam(a[0], a[1], a[2], grads, k + 1, lr=1e-2)
    torch.cuda.synchronize()
    assert step.item() == reps
    assert bool((xs == big.numel()).all())
    for p, q in zip(a, b):
        assert torch.equal(p, q)


@pytest.mark.parametrize("dims", [(16, 64, 64, 64), (16, 128, 128, 64), (16, 160, 200, 10)])
def test_larger_batch_covers_smaller_capture(gpu_lib, dims):
    """Batches on both sides of 4096 rows, where the row tiles change: the scratch of a call made
    once with the larger batch is enough for a capture with a smaller one, of a network whose
    tiles of 16 rows fit the LDS, whose tiles of 4 alone do, and of neither."""
    om = gpu_lib
    F, H1, H2, K = dims
    g = np.random.Generator(np.random.PCG64(H1))
    P32 = {k: v.astype(np.float32) for k, v in _params(g, F, H1, H2, K).items()}
    X = g.standard_normal((4097, F)).astype(np.float32)
    y = g.integers(0, K, 4097).astype(np.int32)
    params = torch.from_numpy(_flat(P32)).cuda()
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    loss = torch.zeros(1, device="cuda")
    grads = torch.zeros_like(params)

    def check(B):
        loss_ref, _, g_ref = oracle.mlp_loss_grad(X[:B].astype(np.float64), y[:B],
                                                  {k: v.astype(np.float64) for k, v in P32.items()})
        assert abs(loss.item() - loss_ref) <= 1e-5 * abs(loss_ref)
        gh, off = grads.cpu().numpy().astype(np.float64), 0
        for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
            sz = g_ref[k].size
            assert _rel(gh[off:off + sz], g_ref[k].ravel()) < 1e-5, (k, B)
            off += sz

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        om.mlp_loss_grad(dims, params, Xd, yd, loss, grads)
    s.synchronize()
    check(4097)
    for B in (4096, 300):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            om.mlp_loss_grad(dims, params, Xd[:B], yd[:B], loss, grads)
        for _ in range(2):
            loss.fill_(-1.0)
            grads.fill_(-1.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            check(B)
