"""A unit's state rows shared among several workgroups of the one-launch folds, against the kernel-per-step
path, at the edges of what the shared launch takes: one 64-row tile per workgroup and four, tiles that
stay in LDS and tiles that stream through it, blocks of 64 to 1024 tokens, more merging tokens per
workgroup than its scratch holds, appends of 1, 16, 17, 64, 65 and all rows, sinks beyond the first
tile, folds in place, a captured step, two threads at once.

Assignments, counts, weights, key and value sums, normalised keys, radii and the value readout are equal to
the bit: the same products added in the same order, the same roots and divisions."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def kit():
    import paper_2605_09877_amd as pkg
    from paper_2605_09877_amd import binding, synth
    return pkg, binding, synth


def make(sy, chunk, units, seq, budget, **kw):
    kind = {"budget_fixed": budget} if isinstance(budget, int) else \
        {"budget_kind": "table", "budget_table": budget} if isinstance(budget, tuple) else {"budget_kind": "sqrt"}
    return sy.shrink(sy.WORKLOADS["prefill_fixed"], batch=1, n_q_heads=units, n_kv_heads=units, chunk_len=chunk, seq=seq,
                     **kind, **kw)


def widest(w):
    """The most workgroups that may share a unit's rows, forced: few units and long blocks are not shared by default."""
    pkg, b, sy = kit()
    tiles = pkg.state_for(w, device=DEV, **sy.make_params(w, DEV, plain=True)).capacity // 64
    units, n = w.batch * w.n_kv_heads, 1
    while 2 * n <= 16 and units * 2 * n <= 256 and tiles >= 2 * n:
        n *= 2
    return {b.KVM_DEBUG_FOLD_SPLIT: n}


def run(w, knobs, decode_tail=0):
    pkg, binding, sy = kit()
    q, k, v = sy.make_qkv(w, DEV)
    p = sy.make_params(w, DEV, plain=False)
    st = pkg.state_for(w, device=DEV, **p)
    for knob, value in knobs.items():
        st.debug_set(knob, value)
    assign, _ = st.trace(w.seq // w.chunk_len + 1)
    n = w.seq - decode_tail
    cut = lambda x, lo, hi: None if x is None else x[:, lo:hi].contiguous()
    st.prefill(cut(q, 0, n), cut(k, 0, n), cut(v, 0, n), cut(p["gate"], 0, n))
    for t in range(n, w.seq):
        one = lambda x: None if x is None else x[:, t].contiguous()
        st.decode(one(q), one(k), one(v), one(p["gate"]))
    torch.cuda.synchronize()
    return st, assign[:st.folds].clone(), st.export()


def same(a, b):
    assert a[0].rows == b[0].rows and a[0].folds == b[0].folds
    assert torch.equal(a[1], b[1]), "assignments"
    for key in ("sK", "sV", "rho", "n", "w", "khat", "vhat"):
        assert torch.equal(a[2][key], b[2][key]), key


STEP = (64, 64, 80, 81, 98, 162, 227, 227, 355, 355)   # appends of 16, 1, 17, 64, 65, 0, 128 rows at 128-token blocks
CASES = {   # chunk, units, tokens, budget, other fields, forced split (0: the widest)
    "one tile each": (64, 2, 64 * 24, 1024, {}, 0),
    "four tiles each": (256, 64, 256 * 8, 1024, {}, 0),
    "sixteen workgroups": (256, 1, 256 * 9, 1024, {}, 16),
    "tiles that stream": (256, 2, 256 * 8, 1024, {}, 2),
    "long block": (1024, 2, 1024 * 4, 1024, {}, 0),
    "scratch too small": (512, 1, 512 * 5 + 5, 512, {}, 2),
    "appends": (128, 3, 128 * 12, tuple(128 + x for x in STEP), {}, 0),
    "appends, long block": (512, 2, 512 * 8, tuple(512 + x for x in STEP), {}, 0),
    "growing": (256, 4, 256 * 24, None, {}, 0),
    "sinks": (256, 2, 256 * 8, 512, {"n_sink": 130}, 0),
}


@pytest.mark.parametrize("case", list(CASES))
def test_shared_rows_agree_with_a_kernel_per_step(case):
    _, b, sy = kit()
    chunk, units, seq, budget, kw, split = CASES[case]
    w = make(sy, chunk, units, seq, budget, **kw)
    knobs = {b.KVM_DEBUG_FOLD_SPLIT: split} if split else widest(w)
    got = run(w, knobs)
    assert got[0].fold_path == 1
    same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}))


# patience 0: the first workgroup of a unit that finds itself alone takes all of it; 0.5 us: some units are taken, some shared
@pytest.mark.parametrize("patience", [1, 51])
@pytest.mark.parametrize("case", ["one tile each", "four tiles each", "long block", "appends", "growing", "sinks"])
def test_units_whose_workgroups_do_not_all_start(case, patience):
    """A unit that one workgroup takes over, because its others have not started in time, folds to the same bits."""
    _, b, sy = kit()
    chunk, units, seq, budget, kw, _ = CASES[case]
    w = make(sy, chunk, units, seq, budget, **kw)
    for tail in (0, chunk + 1):
        got = run(w, {**widest(w), b.KVM_DEBUG_FOLD_PATIENCE: patience}, tail)
        same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}, tail))


@pytest.mark.parametrize("tail", [1, 128 + 3])
def test_folds_in_place(tail):
    _, b, sy = kit()
    w = make(sy, 128, 2, 128 * 9, 512)
    w = sy.shrink(w, seq=w.seq // 128 * 128)
    same(run(w, widest(w), tail), run(w, {b.KVM_DEBUG_FOLD_PATH: 2}, tail))


def test_captured_step():
    """A step that folds, captured: the graph holds no launch that waits for other workgroups."""
    pkg, b, sy = kit()
    w = make(sy, 128, 2, 128 * 8, 512)
    q, k, v = sy.make_qkv(w, DEV)
    p = sy.make_params(w, DEV, plain=True)
    n = w.seq - 1
    res = []
    for captured in (False, True):
        st = pkg.state_for(w, device=DEV, **p)
        for knob, value in widest(w).items():
            st.debug_set(knob, value)
        st.prefill(q[:, :n - 127].contiguous(), k[:, :n - 127].contiguous(), v[:, :n - 127].contiguous())
        one = lambda t: (q[:, t].contiguous(), k[:, t].contiguous(), v[:, t].contiguous())
        for t in range(n - 127, n):
            st.decode(*one(t))
        args = one(n)
        torch.cuda.synchronize()
        if captured:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                y = st.decode(*args)
            g.replay()
        else:
            y = st.decode(*args)
        torch.cuda.synchronize()
        res.append((st, torch.zeros(0), st.export(), y))
    same(*res)
    assert torch.equal(res[0][3], res[1][3])


def test_two_threads():
    """Two states driven from two threads on streams of their own: their launches meet on the chip."""
    pkg, b, sy = kit()
    w = make(sy, 256, 16, 256 * 16, 1024)
    q, k, v = sy.make_qkv(w, DEV)
    want = run(sy.shrink(w), {b.KVM_DEBUG_FOLD_PATH: 2})
    p = sy.make_params(w, DEV, plain=False)
    torch.cuda.synchronize()
    assert pkg.state_for(w, device=DEV, **p).fold_path == 1 and want[0].fold_path == 2
    out = [None, None]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                st = pkg.state_for(w, device=DEV, **p)
                st.prefill(q, k, v, p["gate"])
                torch.cuda.current_stream().synchronize()
            out[i] = (st, want[1], st.export())
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=60)
    for o in out:
        assert o is not None
        same(o, want)


@pytest.mark.parametrize("chunk,units,blocks,path", [(128, 8, 7, 1), (128, 7, 7, 2), (128, 8, 6, 2), (512, 8, 8, 2),
                                                     (64, 64, 5, 1), (64, 64, 4, 2), (64, 63, 5, 2)])
def test_states_that_share_by_default(chunk, units, blocks, path):
    """The edges of the default: 8 units, 256-token blocks, seven blocks, five from 64 units on; results as a kernel per
    step either way."""
    _, b, sy = kit()
    w = make(sy, chunk, units, chunk * blocks, 2 * chunk)
    got = run(w, {})
    assert got[0].fold_path == path
    same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}))


@pytest.mark.parametrize("first", [4, 7])
def test_a_grown_and_an_imported_state_continue_to_the_bit(first):
    """States of 8 units made for fewer blocks than share rows (4) and for as many (7), then grown or carried over into a
    state of full size: outputs and state of the rest of the prompt are those of one that was whole from the start."""
    pkg, b, sy = kit()
    w = make(sy, 128, 8, 128 * 24, None)
    q, k, v = sy.make_qkv(w, DEV)
    p = sy.make_params(w, DEV, plain=False)
    n = 128 * first
    part = lambda x, lo, hi: x[:, lo:hi].contiguous()
    call = lambda st, lo, hi: st.prefill(part(q, lo, hi), part(k, lo, hi), part(v, lo, hi), part(p["gate"], lo, hi))
    whole = pkg.state_for(w, device=DEV, **p)
    want = (call(whole, 0, n), call(whole, n, w.seq))
    grown = pkg.state_for(w, device=DEV, max_tokens=n, **p)
    head = call(grown, 0, n)
    snap = grown.export()
    grown.grow(w.seq)
    loaded = pkg.state_for(w, device=DEV, max_tokens=w.seq + 8192, **p)
    loaded.import_(snap)
    assert torch.equal(head, want[0])
    for st in (grown, loaded):
        assert torch.equal(call(st, n, w.seq), want[1])
        got, ref = st.export(), whole.export()
        for key in ("sK", "sV", "rho", "n", "w", "khat", "vhat"):
            assert torch.equal(got[key], ref[key]), key


@pytest.mark.parametrize("compute_units,path", [(32, 1), (8, 2)])
def test_fewer_compute_units(compute_units, path):
    """A device with fewer compute units than the widest launch has workgroups folds all the same."""
    _, b, sy = kit()
    w = make(sy, 128, 8, 128 * 8, 512)
    got = run(w, {b.KVM_DEBUG_COMPUTE_UNITS: compute_units})
    assert got[0].fold_path == path
    same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}))


def test_exchange_numbers_run_out():
    """A state's shared folds are told apart by 16-bit numbers; the table is cleared before they repeat (after some 65530
    folds: in the 129th of these prompts)."""
    pkg, b, sy = kit()
    w = make(sy, 64, 2, 64 * 512, 128)
    q, k, v = sy.make_qkv(w, DEV)
    p = sy.make_params(w, DEV, plain=False)
    ref = pkg.state_for(w, device=DEV, **p)
    ref.debug_set(b.KVM_DEBUG_FOLD_PATH, 2)
    want = ref.prefill(q, k, v, p["gate"])
    st = pkg.state_for(w, device=DEV, **p)
    st.debug_set(b.KVM_DEBUG_FOLD_SPLIT, 2)
    assert st.fold_path == 1
    for i in range(132):
        st.reset()
        got = st.prefill(q, k, v, p["gate"])
        if i == 0 or i > 124:
            assert torch.equal(got, want), i
    a, e = st.export(), ref.export()
    for key in ("sK", "sV", "rho", "n", "w", "khat", "vhat"):
        assert torch.equal(a[key], e[key]), key


def test_arrangement_changes_between_calls():
    """The workgroups' meeting counts on over launches of different widths, taken-over units among them."""
    pkg, b, sy = kit()
    w = make(sy, 128, 4, 128 * 24, 1024)
    q, k, v = sy.make_qkv(w, DEV)
    p = sy.make_params(w, DEV, plain=False)
    part = lambda x, lo, hi: x[:, lo:hi].contiguous()
    ref = pkg.state_for(w, device=DEV, **p)
    ref.debug_set(b.KVM_DEBUG_FOLD_PATH, 2)
    want = ref.prefill(q, k, v, p["gate"])
    st = pkg.state_for(w, device=DEV, **p)
    out = []
    for i, (split, patience) in enumerate([(2, 0), (16, 0), (4, 1), (8, 51), (1, 0), (16, 1), (2, 0), (4, 0)]):
        st.debug_set(b.KVM_DEBUG_FOLD_SPLIT, split)
        st.debug_set(b.KVM_DEBUG_FOLD_PATIENCE, patience)
        lo, hi = 384 * i, 384 * (i + 1)
        out.append(st.prefill(part(q, lo, hi), part(k, lo, hi), part(v, lo, hi), part(p["gate"], lo, hi)))
    assert torch.equal(torch.cat(out, dim=1), want)
    a, e = st.export(), ref.export()
    for key in ("sK", "sV", "rho", "n", "w", "khat", "vhat"):
        assert torch.equal(a[key], e[key]), key


@pytest.mark.parametrize("chunk,units,heads,blocks,path", [
    (512, 8, 8, 12, 1), (512, 8, 8, 11, 2), (512, 64, 64, 8, 1), (512, 64, 64, 7, 2), (512, 8, 16, 12, 1), (512, 8, 32, 12, 2),
    (1024, 8, 8, 12, 2),
])
def test_long_blocks_on_either_side_of_the_rule(chunk, units, heads, blocks, path):
    """Blocks of more than 256 tokens by the library's own choice, growing state, against a kernel per step."""
    _, b, sy = kit()
    w = make(sy, chunk, units, chunk * blocks, None)
    w = sy.shrink(w, n_q_heads=heads)
    got = run(w, {})
    assert got[0].fold_path == path
    same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}))


@pytest.mark.parametrize("chunk,units,heads,blocks,budget,path", [
    (64, 1, 1, 32, 256, 1), (64, 7, 7, 31, 256, 2), (64, 4, 4, 32, 192, 2), (128, 2, 8, 20, 512, 1), (128, 2, 8, 19, 512, 2), (256, 4, 4, 20, 448, 2),
    (256, 3, 6, 32, None, 1), (64, 5, 5, 32, (64, 64, 65, 130, 190, 254, 300) + (300,) * 25, 1), (512, 4, 4, 32, 512, 2),
])
def test_few_units_on_either_side_of_the_rule(chunk, units, heads, blocks, budget, path):
    """Fewer than 8 units by the library's own choice, with two decoded tokens behind the prompt, against a kernel per step."""
    _, b, sy = kit()
    w = make(sy, chunk, units, chunk * blocks, budget)
    w = sy.shrink(w, n_q_heads=heads)
    got = run(w, {}, 2)
    assert got[0].fold_path == path
    same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}, 2))


@pytest.mark.parametrize("chunk,steps", [(128, (12, 13, 1, 0, 40)), (256, (11, 12, 13)), (512, (32, 33, 1, 100)), (1024, (5, 33, 300))])
def test_selection_forms_agree_with_a_kernel_per_step(chunk, steps):
    """Appends on either side of the lines between the forms of the selection (one by one, bit by bit in registers, from
    LDS), every block holding its first half twice, so that scores are equal and the earliest of them have to be taken."""
    pkg, b, sy = kit()
    rows = [chunk, chunk]
    for n in steps:
        rows.append(rows[-1] + n)
    w = make(sy, chunk, 3, chunk * len(rows), tuple(rows))
    q, k, v = sy.make_qkv(w, DEV)
    for c in range(len(rows)):
        k[:, c * chunk + chunk // 2:(c + 1) * chunk] = k[:, c * chunk:c * chunk + chunk // 2]
    p = sy.make_params(w, DEV, plain=False)
    res = []
    for knobs in (widest(w), {b.KVM_DEBUG_FOLD_PATH: 2}):
        st = pkg.state_for(w, device=DEV, **p)
        for knob, value in knobs.items():
            st.debug_set(knob, value)
        assign, _ = st.trace(len(rows))
        st.prefill(q, k, v, p["gate"])
        torch.cuda.synchronize()
        res.append((st, assign[:st.folds].clone(), st.export()))
    same(*res)


@pytest.mark.parametrize("chunk,heads,tail,blocks,rows", [
    (256, (16, 16), 0, 8, 512), (256, (16, 16), 97, 8, 512),     # room beside every launch; not beside the last, behind which nothing folds
    (256, (48, 16), 1, 11, 300), (256, (48, 16), 1, 13, 300),    # three heads on a KV head: none in short calls
    (128, (48, 16), 1, 8, 300), (256, (128, 16), 5, 13, 512),    # blocks of 128; eight heads, one tile a workgroup: none
])
def test_outputs_do_not_depend_on_the_room_beside_attention(chunk, heads, tail, blocks, rows):
    """Outputs and state of a prompt whose folds are shared beside attention, against a kernel per step, chunk by chunk."""
    pkg, b, sy = kit()
    w = make(sy, chunk, heads[1], chunk * blocks + tail, rows)
    w = sy.shrink(w, n_q_heads=heads[0])
    q, k, v = sy.make_qkv(w, DEV)
    p = sy.make_params(w, DEV, plain=False)
    res = []
    for knobs in ({}, {b.KVM_DEBUG_FOLD_PATH: 2, b.KVM_DEBUG_PREFILL_SCHEDULE: 1}):
        st = pkg.state_for(w, device=DEV, **p)
        for knob, value in knobs.items():
            st.debug_set(knob, value)
        assign, _ = st.trace(blocks + 1)
        out, lse = st.prefill(q, k, v, p["gate"], want_lse=True)
        torch.cuda.synchronize()
        res.append((st, assign[:st.folds].clone(), st.export(), out, lse))
    assert res[0][0].fold_path == 1 and torch.equal(res[0][3], res[1][3]) and torch.equal(res[0][4], res[1][4])
    same(*[r[:3] for r in res])


@pytest.mark.parametrize("chunk,units,budget,path", [
    (256, 1, 256, 2), (256, 2, 256, 1), (256, 3, 320, 2), (256, 4, 320, 1), (128, 1, 256, 2), (128, 1, 257, 1), (128, 2, 256, 1), (64, 1, 256, 1),
    (256, 1, 512, 1), (256, 1, (256, 256, 257, 300), 1),
])
def test_few_units_that_do_not_grow(chunk, units, budget, path):
    """Prompts of 32 blocks on either side of the rule for states of fewer than 512 rows without appends."""
    _, b, sy = kit()
    w = make(sy, chunk, units, chunk * 32, budget)
    got = run(w, {})
    assert got[0].fold_path == path
    same(got, run(w, {b.KVM_DEBUG_FOLD_PATH: 2}))
