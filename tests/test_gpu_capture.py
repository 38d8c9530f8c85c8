"""Calls captured into a graph, which keep to the caller's stream: prompts of states that fold with one workgroup per
unit (256 units) and of states that share rows when they are not captured (8 units), and a backward pass."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("schedule", [0, 1, pytest.param(2, marks=pytest.mark.skip(
    reason="several streams in one graph: the runtime crashed at a replay, cause unknown; the schedule is not taken in a capture"))])
@pytest.mark.parametrize("batch,heads,chunk", [(8, 32, 64), (1, 8, 128)])
def test_captured_prefill(batch, heads, chunk, schedule):
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=batch, n_q_heads=heads, n_kv_heads=heads, chunk_len=chunk,
                  seq=chunk * 19 + 5, budget_fixed=3 * chunk)
    q, k, v = sy.make_qkv(w, DEV)
    params = sy.make_params(w, DEV, plain=False)
    st = pkg.state_for(w, device=DEV, **params)
    st.debug_set(2, schedule)
    assert st.fold_path == 1
    want = st.prefill(q, k, v, params["gate"])
    ref = st.export()
    torch.cuda.synchronize()
    st.reset()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = st.prefill(q, k, v, params["gate"])
    for _ in range(3):   # with eager work of another state in between
        got.zero_()
        pkg.state_for(w, device=DEV, **params).prefill(q, k, v, params["gate"])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        e = st.export()
        for key in ("sK", "sV", "rho", "n", "w", "khat", "vhat", "win_k", "win_v"):
            assert torch.equal(e[key], ref[key]), key


@pytest.mark.parametrize("launches", [0, 2, 3])   # by the library's choice one a chunk; several, on its streams when not captured
def test_captured_backward(launches):
    """The gradients of a captured backward pass, which keeps to the caller's stream, are those of one that does not."""
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import binding as b
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=2, n_q_heads=4, n_kv_heads=2, chunk_len=256, seq=256 * 4 + 77,
                  budget_fixed=300)
    q, k, v = sy.make_qkv(w, DEV)
    params = sy.make_params(w, DEV, plain=False)
    dout = torch.randn(q.shape, generator=torch.Generator(DEV).manual_seed(1), device=DEV).to(q.dtype)
    st = pkg.state_for(w, device=DEV, **params)
    st.debug_set(b.KVM_DEBUG_BACKWARD_LAUNCHES, launches)
    assign, score = st.trace(w.seq // w.chunk_len + 1)
    out, lse = st.prefill(q, k, v, params["gate"], want_lse=True)
    args = (q, k, v, params["gate"], out, lse, dout, assign, score)
    want = st.backward(*args)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = st.backward(*args)
    for _ in range(3):
        for x in got.values():
            x.zero_()
        st.backward(*args)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name in ("dq", "dk", "dv", "dgate"):
            assert torch.equal(got[name], want[name]), name
        for name in ("dgamma", "dbeta", "dtau_state", "dtau_bswa"):   # sums by fp64 atomics: the last fp32 bit
            torch.testing.assert_close(got[name], want[name], rtol=2 ** -22, atol=1e-6)
