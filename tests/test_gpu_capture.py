"""A prompt captured into a graph: folds on the library's streams, joined to the caller's by events, one workgroup per
unit (256 units) and states that share rows when they are not captured (8 units)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("schedule", [1, 2])
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
