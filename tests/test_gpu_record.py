"""The record of the folds (kvm_state_trace) is written and never read: whatever another stream does to the caller's buffers
meanwhile, the folds are the same to the bit; and nothing is written beyond what was asked for."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KEYS = ("sK", "sV", "rho", "w", "n", "khat", "vhat")

CASES = [   # io, head_dim, chunk, batch, heads, schedule (1 chunk by chunk, 2 pipelined), budget by block
    ("f32", 64, 64, 1, 2, 1, (64, 64, 64, 100, 101, 101)), ("bf16", 64, 64, 2, 16, 1, (64, 64, 64, 100, 101, 101)),
    ("bf16", 128, 256, 2, 4, 2, (256, 256, 256, 300, 301, 301)), ("bf16", 128, 256, 1, 3, 1, (256, 256, 260, 600, 601, 601)),
    ("f32", 128, 40, 3, 2, 2, (40, 40, 47, 80, 81, 81)),
]


def setup(io, d, C, batch, heads, schedule, table):
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import binding as b
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["tiny_f32"], io=io, head_dim=d, batch=batch, n_q_heads=heads, n_kv_heads=heads, chunk_len=C, rope_dims=16,
                  seq=C * 24, budget_kind="table", budget_table=table)
    q, k, v = sy.make_qkv(w, DEV)
    params = sy.make_params(w, DEV, plain=False)

    def make():
        st = pkg.state_for(w, device=DEV, **params)
        st.debug_set(b.KVM_DEBUG_FOLD_PATH, 2)
        st.debug_set(b.KVM_DEBUG_PREFILL_SCHEDULE, schedule)
        return st

    return make, lambda st: st.prefill(q, k, v, params["gate"])


@pytest.mark.parametrize("case", CASES)
def test_the_record_is_not_read(case):
    make, run = setup(*case)
    plain = make()
    out = run(plain)
    want = plain.export()
    other = torch.cuda.Stream()
    for _ in range(3):
        st = make()
        assign, score = st.trace(24)
        torch.cuda.synchronize()
        with torch.cuda.stream(other):   # all through the call
            for _ in range(150):
                assign.fill_(-7)
                score.fill_(-7.0)
        got = run(st)
        with torch.cuda.stream(other):
            for _ in range(150):
                assign.fill_(-7)
                score.fill_(-7.0)
        torch.cuda.synchronize()
        assert torch.equal(got, out)
        have = st.export()
        for key in KEYS:
            assert torch.equal(have[key], want[key]), key


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("with_assign,with_score", [(True, True), (True, False), (False, True)])
def test_only_the_folds_asked_for(case, with_assign, with_score):
    """Each record alone is the one of both, its first fold to its last, and what lies behind stays as it is."""
    make, run = setup(*case)
    full = make()
    assign, score = full.trace(24)
    run(full)
    n = full.folds - 2
    st = make()
    a, s = torch.full_like(assign, -9), torch.full_like(score, -9.0)
    from paper_2605_09877_amd import binding as b
    assert st.lib.kvm_state_trace(st.handle, a.data_ptr() if with_assign else None, s.data_ptr() if with_score else None, n) == b.KVM_OK
    run(st)
    torch.cuda.synchronize()
    same = lambda x, y: torch.equal(x.view(torch.int32), y.view(torch.int32))   # (scores that were not computed are NaN)
    assert same(a[:n], assign[:n]) if with_assign else bool((a == -9).all())
    assert same(s[:n], score[:n]) if with_score else bool((s == -9).all())
    assert bool((a[n:] == -9).all()) and bool((s[n:] == -9).all())
