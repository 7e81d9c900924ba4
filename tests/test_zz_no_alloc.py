"""adapter_predict_static (no allocation, scratch in a static device array)
against adapter_predict (a context's scratch), through the C ABI: the same
priorities on two calls in a row, the second with a smaller batch, for batch-1
and batched launches; sizes above the static scratch are refused before any
device work."""
import sys

import numpy as np
import pytest

import oracle as o
import workload as w

pytestmark = pytest.mark.gpu


def _log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# bf16 with a batched router (D % 16 == 0), rank 8 and rank 6; the Qwen-shaped adapter (n 128, r 64)
CASES = [w.MoEConfig(name="static_bf16_D256_n12_r8", L=2, D=256, n=12, K=3, I=64, r=8, S=12, windows=(2,),
                     tokens=2, batch=16, seed=9),
         w.MoEConfig(name="static_bf16_D256_n12_r6", L=2, D=256, n=12, K=3, I=64, r=6, S=12, windows=(2,),
                     tokens=2, batch=16, seed=10),
         w.get("c1").with_(L=2, batch=16, S=128, I=16)]


@pytest.mark.parametrize("cfg", CASES, ids=["r8", "r6", "qwen_shape"])
def test_static_scratch_entry_point_matches_adapter_predict(torch_cuda, cfg):
    import torch
    from paper_2607_24787_amd import spp
    from paper_2607_24787_amd.model import OffloadedMoEStack
    st = OffloadedMoEStack(cfg)
    try:
        rng = np.random.default_rng(3)
        A, Bm = st.adapter[0]
        A_ref, B_ref = o.OracleWeights(cfg).adapter(0)
        s_dev = torch.empty(cfg.n, dtype=torch.float32, device=st.device)
        for B in (cfg.batch, 5, 1):       # two calls in a row with a smaller batch after a larger one
            _log(f"[static] {cfg.name} B={B}")
            x = rng.normal(size=(B, cfg.D)).astype(np.float32)
            xd = torch.from_numpy(x).to(st.device)
            s_dev.fill_(float("nan"))
            spp.adapter_predict_static(A.data_ptr(), Bm.data_ptr(), st.dtype_code, cfg.D, cfg.n, cfg.r,
                                       xd.data_ptr(), B, s_dev.data_ptr(), st.stream.cuda_stream)
            torch.cuda.synchronize()
            got = s_dev.cpu().numpy()
            want = spp.adapter_predict(st.ctx, 0, xd.data_ptr(), B, cfg.n)
            assert np.array_equal(got, want), (B, np.max(np.abs(got - want)))
            _, _, s_ora = o.adapter_scores(A_ref, B_ref, x.astype(np.float64))
            np.testing.assert_allclose(got, s_ora, rtol=1e-5, atol=2e-6)
        # refused before any device work: too large for the static scratch, NULL or misaligned pointers
        big = spp.STATIC_SCRATCH_FLOATS // (cfg.n + cfg.r) + 1
        for args in ((A.data_ptr(), xd.data_ptr(), big), (0, xd.data_ptr(), 1), (A.data_ptr() + 8, xd.data_ptr(), 1),
                     (A.data_ptr(), xd.data_ptr() + 4, 1)):
            with pytest.raises(spp.SppError) as e:
                spp.adapter_predict_static(args[0], Bm.data_ptr(), st.dtype_code, cfg.D, cfg.n, cfg.r, args[1],
                                           args[2], s_dev.data_ptr(), st.stream.cuda_stream)
            assert e.value.status == spp.SPP_EINVAL
    finally:
        st.close()


@pytest.mark.parametrize("n,r,D,dtype", [(12, 8, 256, "bf16"), (128, 64, 2048, "bf16"), (72, 5, 256, "bf16"),
                                         (33, 16, 640, "f32")], ids=["one_wave", "two_per_lane", "wide_tail", "f32"])
@pytest.mark.parametrize("B", [1, 3])
def test_static_scratch_replays_of_a_graph(torch_cuda, n, r, D, dtype, B):
    """Replays with new inputs, eager calls of other sizes between them: every one gives the eager result."""
    import torch
    from paper_2607_24787_amd import spp
    dt, code = (torch.bfloat16, spp.DTYPE_BF16) if dtype == "bf16" else (torch.float32, spp.DTYPE_F32)
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.empty((r, D), device="cuda").normal_(0, 0.05, generator=g).to(dt)
    Bm = torch.empty((n, r), device="cuda").normal_(0, 0.5, generator=g).to(dt)
    x, out, eager = (torch.zeros(s, device="cuda") for s in ((B, D), (n,), (n,)))
    x2 = torch.empty((5, D), device="cuda").normal_(generator=g)

    def call(xs, b, dst):
        spp.adapter_predict_static(A.data_ptr(), Bm.data_ptr(), code, D, n, r, xs.data_ptr(), b, dst.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)

    call(x, B, eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, B, out)
        call(x, B, out)
    for t in range(6):
        _log(f"[static graph] n={n} r={r} B={B} replay {t}")
        x.normal_(generator=g)
        out.fill_(float("nan"))
        graph.replay()
        call(x, B, eager)
        if t % 2:
            call(x2, 5 if t == 3 else 1, torch.empty_like(eager))
        torch.cuda.synchronize()
        want = torch.softmax(x.double() @ A.double().T @ Bm.double().T, dim=-1).sum(0)
        assert torch.equal(out, eager), t
        assert torch.allclose(out.double(), want, rtol=1e-5, atol=2e-6), t


def test_static_scratch_after_calls_that_overlapped(torch_cuda):
    """Calls that overlap on one device race for the scratch; a call after them, in order, must give its own result.
    Ordered calls of several ranks in turn, after batches of overlapping ones on two streams."""
    import torch
    from paper_2607_24787_amd import spp
    n, D = 128, 2048
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.empty((64, D), device="cuda").normal_(0, 0.05, generator=g).to(torch.bfloat16)
    Bm = {r: torch.empty((n, r), device="cuda").normal_(0, 0.5, generator=g).to(torch.bfloat16) for r in (64, 24, 8)}
    xs = torch.empty((8, D), device="cuda").normal_(generator=g)
    streams = [torch.cuda.Stream() for _ in range(2)]
    sink = torch.empty((2, n), device="cuda")
    out = torch.empty(n, device="cuda")
    torch.cuda.synchronize()

    def call(r, x, dst, stream):
        spp.adapter_predict_static(A.data_ptr(), Bm[r].data_ptr(), spp.DTYPE_BF16, D, n, r, x.data_ptr(), 1,
                                   dst.data_ptr(), stream.cuda_stream)

    for t in range(12):
        _log(f"[static overlap] round {t}")
        for k in range(20):
            call((64, 24)[(k + t) % 2 if t % 3 else 0], xs[k % 8], sink[k % 2], streams[k % 2])
        torch.cuda.synchronize()
        for r in (64, 24, 8, 64):
            x = xs[(t + r) % 8]
            out.fill_(float("nan"))
            call(r, x, out, torch.cuda.current_stream())
            torch.cuda.synchronize()
            want = torch.softmax(x.double() @ A[:r].double().T @ Bm[r].double().T, dim=-1)
            assert torch.allclose(out.double(), want, rtol=1e-5, atol=2e-6), (t, r)
