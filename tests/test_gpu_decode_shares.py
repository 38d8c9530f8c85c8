"""Decode steps whose keys are shared among workgroups (few sequences): the step's output against
softmax attention evaluated in fp64 over the readout rows and the window the state holds, at key
counts around a share's size (one round of the kernel's loop: 64 rows of bf16 / 128, 32 of fp32 / 128,
128 of bf16 / 64, 64 of fp32 / 64), with one share, with empty shares, with every head grouping.

Bars: fp32 1e-4 max-abs (the forward's); bf16 2^-8 of the element (the stored value's rounding, one
ulp at worst when the fp32 sum lies at a rounding boundary) plus 1e-4 of fp32 summation."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def reference(st, w, q, k, v, pos):
    """out [B, Hq, d] fp64 of one token at position pos, from the exported state."""
    e = st.export()
    C, L = w.chunk_len, w.chunk_len * w.n_bswa_chunks
    first = max(0, pos // C * C + C - L)
    slots = torch.arange(first, pos, device=DEV) % L
    K = torch.cat([e["khat"].double(), e["win_k"][:, :, slots].double(), k[:, :, None].double()], dim=2)
    V = torch.cat([e["vhat"].double(), e["win_v"][:, :, slots].double(), v[:, :, None].double()], dim=2)
    G = w.n_q_heads // w.n_kv_heads
    qg = q.double().reshape(w.batch, w.n_kv_heads, G, w.head_dim)
    s = torch.matmul(qg, K.transpose(2, 3).contiguous()) / w.head_dim ** 0.5
    return torch.matmul(s.softmax(-1), V).reshape(q.shape)


@pytest.mark.parametrize("io,d", [("bf16", 128), ("f32", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("group", [1, 2, 4])
@pytest.mark.parametrize("rows", [64, 127, 129, 1000, 2200])   # the last: as many shares as there may be, of several rounds
def test_shared_keys_against_softmax_attention(io, d, group, rows):
    run(io, d, 2, 2, group, rows)


@pytest.mark.parametrize("batch,rows", [(1, 1900), (1, 4200), (2, 2200), (3, 2200)])
def test_as_many_shares_as_lanes(batch, rows):
    """fp32, 128 channels: 64 shares for one or two heads, 32 for three."""
    run("f32", 128, batch, 1, 1, rows)


def run(io, d, batch, heads, group, rows):
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["decode"], io=io, batch=batch, n_q_heads=heads * group, n_kv_heads=heads, head_dim=d, rope_dims=16,
                  chunk_len=64, state_rows=rows, budget_fixed=rows)
    st = pkg.state_for(w, max_tokens=rows + 512, device=DEV)
    pre = sy.make_decode_state(w, DEV)
    st.import_(pre)
    gen = torch.Generator(device=DEV).manual_seed(rows + d)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(st.dtype)
    for step in range(3):
        q, k, v = rnd(batch, w.n_q_heads, d), rnd(batch, heads, d), rnd(batch, heads, d)
        want = reference(st, w, q, k, v, st.tokens)
        got = st.decode(q, k, v).double()
        tol = 1e-4 if io == "f32" else 1e-4 + 2.0 ** -8 * want.abs()
        assert bool(((got - want).abs() <= tol).all()), (step, (got - want).abs().max().item())
