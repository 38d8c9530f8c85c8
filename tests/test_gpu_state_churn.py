"""States made and dropped in quick succession share the library's streams: training steps from several threads,
each on a stream of its own, give bit for bit what one thread alone gives."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _step(T, C, seed):
    import paper_2605_09877_amd as kvm
    gen = torch.Generator(device=DEV).manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=gen, device=DEV).bfloat16().requires_grad_(True)
    q, k, v = r(2, T, 4, 128), r(2, T, 4, 128), r(2, T, 4, 128)
    out = kvm.kvm_attention(q, k, v, chunk_len=C, rope_dims=32, budget_fixed=2 * C)
    return (out.detach(),) + torch.autograd.grad(out, (q, k, v), torch.ones_like(out))


def test_the_long_step_shares_rows():
    """What the last case below is there for: its state of 8 units folds on the path whose workgroups wait for each other."""
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=2, n_q_heads=4, n_kv_heads=4, chunk_len=128, seq=128 * 14 + 5, budget_fixed=256)
    assert pkg.state_for(w, device=DEV).fold_path == 1


# a call of one chunk, one with a few folds, one with runs of folds whose workgroups wait for each other
@pytest.mark.parametrize("T,C", [(43, 64), (64 * 5 + 3, 64), (128 * 14 + 5, 128)])
def test_threads_that_make_and_drop_states(T, C):
    want = [_step(T, C, seed) for seed in range(4)]
    torch.cuda.synchronize()
    wrong, right = [], []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for rep in range(8):
                    got = _step(T, C, i)
                    torch.cuda.current_stream().synchronize()
                    same = all(torch.equal(a, b) for a, b in zip(got, want[i]))
                    (right if same else wrong).append((i, rep))
        except Exception as e:   # a thread's exceptions end with it otherwise
            wrong.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    assert len(right) == 4 * 8


@pytest.mark.parametrize("io,d,C,rows", [("f32", 64, 64, 64), ("f32", 128, 128, 360), ("f32", 128, 128, 376),
                                         ("bf16", 64, 256, 256), ("bf16", 64, 96, 130)])
def test_both_schedules_of_small_chunks_agree(io, d, C, rows):
    """Chunk by chunk (below 24 MB of scored rows) and pipelined: the same outputs and the same state."""
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], io=io, batch=2, n_q_heads=4, n_kv_heads=2, head_dim=d, rope_dims=16,
                  seq=7 * C + 13, chunk_len=C, budget_fixed=rows)
    q, k, v = sy.make_qkv(w, DEV)
    params = sy.make_params(w, DEV, plain=False)
    res = []
    for forced in (0, 1, 2):
        st = pkg.state_for(w, device=DEV, **params)
        st.debug_set(2, forced)
        out = st.prefill(q, k, v, params["gate"])
        e = st.export()
        res.append([out] + [e[n] for n in sorted(e) if isinstance(e[n], torch.Tensor)])
    for other in res[1:]:
        assert all(torch.equal(a, b) for a, b in zip(res[0], other))
