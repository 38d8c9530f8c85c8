"""The backward pass on the matrix cores at the edges of its tiles: 32-query and 64-key tiles, 128-key workgroups,
one and several heads per KV head, D formed inside dq and by a pass ahead of the walk (256-token blocks and few
workgroups).  Oracle and bars of test_gpu_backward."""
import pytest
import torch

from test_gpu_backward import run_backward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,rows,T,heads", [
    (64, 65, 64 * 4 + 1, (1, 1)),        # one query in the last tile, one state row beyond a tile
    (64, 127, 64 * 5 + 33, (3, 1)),      # a query beyond a 32-row tile, three heads streamed one after the other
    (128, 129, 128 * 4 + 31, (4, 2)),    # a workgroup with one state row
    (192, 200, 192 * 3 + 95, (2, 2)),    # the block's second workgroup half empty
    (256, 256, 256 * 3 + 1, (2, 1)),     # D ahead
    (256, 300, 256 * 4, (4, 1)),
])
def test_tile_edges(C, rows, T, heads):
    from paper_2605_09877_amd import synth as sy
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=1, n_q_heads=heads[0], n_kv_heads=heads[1], seq=T, chunk_len=C,
                  budget_fixed=rows)
    run_backward_case(w, plain=False)


def test_gradients_do_not_depend_on_the_batch():
    """Alone a sequence has D formed ahead of the walk, among 65 inside dq: the same gradients to the bit."""
    import paper_2605_09877_amd as kvm
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    q, k, v, dout = (torch.randn(65, 256 * 3 + 1, 2, 128, generator=gen, device="cuda:0").bfloat16() for _ in range(4))

    def grads(n):
        leaves = [x[:n].contiguous().requires_grad_(True) for x in (q, k, v)]
        out = kvm.kvm_attention(*leaves, chunk_len=256, rope_dims=32, budget_fixed=256)
        return (out.detach(),) + torch.autograd.grad(out, leaves, dout[:n].contiguous())

    for one, many in zip(grads(1), grads(65)):
        assert torch.equal(one[0], many[0])


@pytest.mark.parametrize("heads,many", [((2, 2), 200), ((2, 1), 200), ((4, 1), 70), ((4, 1), 24)])
@pytest.mark.parametrize("C,rows", [(64, 70), (256, 256)])
def test_gradients_of_one_launch_and_of_several(heads, many, C, rows):
    """A sequence alone, whose chunks are one launch each, and the same one among so many that they are not: the same
    gradients to the bit."""
    import paper_2605_09877_amd as kvm
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    mk = lambda h: torch.randn(many, C * 3 + 33, h, 128, generator=gen, device="cuda:0").bfloat16()
    q, k, v, dout = mk(heads[0]), mk(heads[1]), mk(heads[1]), mk(heads[0])

    def grads(n):
        leaves = [x[:n].contiguous().requires_grad_(True) for x in (q, k, v)]
        out = kvm.kvm_attention(*leaves, chunk_len=C, rope_dims=32, budget_fixed=rows)
        return (out.detach(),) + torch.autograd.grad(out, leaves, dout[:n].contiguous())

    for one, all_ in zip(grads(1), grads(many)):
        assert torch.equal(one[0], all_[0])
