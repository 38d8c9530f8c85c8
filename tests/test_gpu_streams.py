"""Calls on different streams of a program do not wait for each other: not through the launches that share a unit
among workgroups, and not through the library's own streams, which go from state to state."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def kit():
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import synth
    return pkg, synth


def long_sleep(ms):
    """Cycles of torch.cuda._sleep that last about so long."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for n in (1000, 100000):
        a.record()
        torch.cuda._sleep(n)
        b.record()
        torch.cuda.synchronize()
    return int(100000 * ms / a.elapsed_time(b))


def any_attempt_is_independent(attempt):
    """attempt(held, free) enqueues work on both streams, that on `held` behind a sleep; whether `free` got done
    meanwhile.  The streams of both sides share four hardware queues, so an attempt may be held up by chance (about every
    second one, with streams of the library's beside the callers' three of four): one of 40 has to pass."""
    cycles = long_sleep(30.0)
    for n in range(40):
        held, free = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(held):
            torch.cuda._sleep(cycles)
            slept = torch.cuda.Event()
            slept.record()
        attempt(held, free)
        free.synchronize()
        done = not slept.query()
        torch.cuda.synchronize()
        if done:
            print("independent at attempt", n)
            return
    assert False, "work on one stream always waited for the other's"


def workload(**kw):
    pkg, sy = kit()
    w = sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=1, n_q_heads=32, n_kv_heads=32, chunk_len=256, seq=256 * 8,
                  budget_fixed=512, **kw)
    params = sy.make_params(w, DEV, plain=True)

    def make(schedule):
        st = pkg.state_for(w, device=DEV, **params)
        st.debug_set(2, schedule)
        return st

    return make, sy.make_qkv(w, DEV)


def test_shared_folds_of_two_states():
    make, qkv = workload()
    states = [make(1) for _ in range(2)]   # chunk by chunk: no streams but the caller's; 32 units of 256 share a fold
    assert states[0].fold_path == 1
    for st in states:
        st.prefill(*qkv)
    torch.cuda.synchronize()

    def attempt(held, free):
        for st, stream in zip(states, (held, free)):
            with torch.cuda.stream(stream):
                st.reset()
                st.prefill(*qkv)

    any_attempt_is_independent(attempt)


def test_streams_of_a_dropped_state():
    make, qkv = workload(io="f32")
    torch.cuda.synchronize()

    def attempt(held, free):
        for stream in (held, free):
            with torch.cuda.stream(stream):
                make(2).prefill(*qkv)   # the state is dropped at once, its work still waiting

    any_attempt_is_independent(attempt)
