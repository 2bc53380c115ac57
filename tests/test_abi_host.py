"""Host-side checks of the C ABI (no GPU, no compute calls): the library loads, exports every
symbol the header declares, plans sizes correctly and rejects bad arguments before any launch."""
import ctypes as C
import os
import re
import threading

import numpy as np
import pytest

from paper_2605_12110_amd import absb, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module", autouse=True)
def _built():
    if not os.path.exists(absb.LIB_PATH):
        from paper_2605_12110_amd.build import build_library
        build_library(force=False)


def _layer(**kw):
    d = dict(num_q_heads=32, num_kv_heads=8, head_dim=128, page_size=64, dtype=absb.F16,
             block_size=[8, 16, 32, 64, 128, 8, 16, 32], kv_strides=(8 * 64 * 128, 64 * 128, 128))
    d.update(kw)
    return absb.Layer(**d)


def _batch(lens=(4096,), budget=(512,), **kw):
    return absb.Batch(seq_lens_host=list(lens), budget_host=None if budget is None else list(budget),
                      pt_stride=kw.pop("pt_stride", (max(lens) + 63) // 64), **kw)


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "absb.h")).read()
    declared = re.findall(r"ABSB_API\s+[\w\s\*]+?\b(absb_\w+)\s*\(", header)
    assert set(declared) == set(absb.EXPORTS)
    lib = absb.load()
    for name in declared:
        assert getattr(lib, name) is not None
    assert absb.strerror(0) == "ok" and "workspace" in absb.strerror(absb.ERR_WORKSPACE)


def test_plan_matches_the_papers_layout_rules():
    # off[s+1] = off[s] + ceil(L/B_h) (Sec. 3.4 kernel 1); K_s = min(N_s, ceil(T/B_h)) (kernel 2)
    lens, T = (4096, 1000, 77), (512, 100, 4000)
    layer = _layer()
    plan = absb.absb_plan(layer, _batch(lens, T))
    n = np.diff(plan.cent_off).reshape(3, 8)
    ks = []
    for b, L in enumerate(lens):
        for h, B in enumerate(layer.block_size):
            assert n[b, h] == -(-L // B)
            ks.append(min(-(-L // B), -(-T[b] // B)))
    assert plan.total_centroids == n.sum() and plan.cent_off[0] == 0
    assert plan.sel_stride == max(ks)
    assert plan.workspace_bytes > 0 and plan.workspace_bytes % 256 == 0
    # the same offsets as the (independent) generator-side arithmetic of the oracle
    from oracle import oracle as O
    wl = synth.tiny_workload(Bt=3, Hq=8, Hkv=8, P=64, seq_lens=lens, block_size=layer.block_size, budget=T)
    assert np.array_equal(O.offsets(wl), plan.cent_off.astype(np.int64))


def test_plan_sizes_the_build_scratch_for_two_vectors_per_block_with_max_min_pooling():
    lens = (131072,)
    one = absb.absb_plan(_layer(), _batch(lens, (64,)))
    two = absb.absb_plan(_layer(block_repr=absb.REPR_MINMAX), _batch(lens, (64,)))
    assert np.array_equal(one.cent_off, two.cent_off) and one.sel_stride == two.sel_stride
    # the build's binary32 rows dominate the workspace here: 512 B per block and vector
    assert two.workspace_bytes - one.workspace_bytes >= one.total_centroids * 512


def test_plan_without_budget_sizes_for_every_block():
    plan = absb.absb_plan(_layer(), _batch((4096,), None))
    assert plan.sel_stride == 4096 // 8


@pytest.mark.parametrize("kw,status", [
    (dict(head_dim=64), absb.ERR_UNSUPPORTED),
    (dict(dtype=7), absb.ERR_UNSUPPORTED),
    (dict(block_repr=2), absb.ERR_UNSUPPORTED),
    (dict(block_repr=-1), absb.ERR_UNSUPPORTED),
    (dict(num_q_heads=30), absb.ERR_BAD_SHAPE),
    (dict(num_q_heads=128), absb.ERR_UNSUPPORTED),            # group of 16
    (dict(num_q_heads=0), absb.ERR_BAD_SHAPE),
    (dict(page_size=48), absb.ERR_BAD_SHAPE),
    (dict(page_size=4), absb.ERR_BAD_SHAPE),
    (dict(block_size=[8, 16, 32, 64, 128, 8, 16, 24]), absb.ERR_BAD_BLOCK_SIZE),
    (dict(block_size=[4] * 8), absb.ERR_BAD_BLOCK_SIZE),
    (dict(block_size=[256] * 8), absb.ERR_BAD_BLOCK_SIZE),
    (dict(kv_strides=(8 * 64 * 128, 64 * 128, 100)), absb.ERR_BAD_SHAPE),
    (dict(kv_strides=(8 * 64 * 128 + 4, 64 * 128, 128)), absb.ERR_BAD_SHAPE),
    (dict(sm_scale=-1.0), absb.ERR_BAD_SHAPE),
    (dict(sm_scale=float("nan")), absb.ERR_BAD_SHAPE),
])
def test_plan_rejects_bad_layers(kw, status):
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_plan(_layer(**kw), _batch())
    assert e.value.status == status


@pytest.mark.parametrize("lens,budget,pts,status", [
    ((0,), (512,), 64, absb.ERR_BAD_SHAPE),
    ((4096,), (0,), 64, absb.ERR_BAD_SHAPE),
    ((4096,), (-5,), 64, absb.ERR_BAD_SHAPE),
    ((4096,), (512,), 63, absb.ERR_BAD_SHAPE),                # page-table pitch too small
])
def test_plan_rejects_bad_batches(lens, budget, pts, status):
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_plan(_layer(), _batch(lens, budget, pt_stride=pts))
    assert e.value.status == status


def test_null_structs_and_pointers_are_reported_not_dereferenced():
    lib = absb.load()
    assert lib.absb_plan(None, None, None, None, None, None) == absb.ERR_NULL
    layer, batch = _layer(), _batch()
    cl, cb = layer.c(), batch.c()
    assert lib.absb_plan(C.byref(cl), None, None, None, None, None) == absb.ERR_NULL
    # every compute entry point validates host-visible arguments before launching anything:
    # with all device pointers NULL they must return ERR_NULL (and never touch a device)
    null = C.c_void_p(None)
    assert lib.absb_build_centroids(C.byref(cl), C.byref(cb), null, null, null, null, null, C.c_size_t(0), null) \
        == absb.ERR_NULL
    assert lib.absb_score(C.byref(cl), C.byref(cb), null, null, null, null, null, null) == absb.ERR_NULL
    assert lib.absb_topk(C.byref(cl), C.byref(cb), null, null, null, C.c_int32(64), null, C.c_size_t(0), null) \
        == absb.ERR_NULL
    assert lib.absb_sparse_decode(C.byref(cl), C.byref(cb), null, null, null, null, null, C.c_int32(64), null,
                                  null, null, C.c_size_t(0), null) == absb.ERR_NULL
    assert lib.absb_decode_fused(C.byref(cl), C.byref(cb), null, null, null, null, null, null, null, null, null,
                                 null, C.c_size_t(0), null) == absb.ERR_NULL
    # a budget is mandatory for selection
    nb = _batch(budget=None).c()
    assert lib.absb_topk(C.byref(cl), C.byref(nb), null, null, null, C.c_int32(64), null, C.c_size_t(0), null) \
        == absb.ERR_NULL


def test_workspace_and_list_width_checks_come_before_any_launch():
    lib = absb.load()
    layer = _layer()
    fake = C.c_void_p(0x1000)             # never dereferenced: the calls below must fail validation first
    batch = _batch()
    batch_c = batch.c()
    for f in ("seq_lens", "page_table", "cent_off", "budget"):
        setattr(batch_c, f, 0x1000)
    cl = layer.c()
    plan = absb.absb_plan(layer, batch)
    # too small / missing / misaligned workspace
    for ws, nbytes in ((C.c_void_p(None), 0), (C.c_void_p(0x100000), 16), (C.c_void_p(0x100010), plan.workspace_bytes)):
        rc = lib.absb_decode_fused(C.byref(cl), C.byref(batch_c), fake, fake, fake, fake, fake, fake, None, None,
                                   None, ws, C.c_size_t(nbytes), None)
        assert rc == absb.ERR_WORKSPACE
        rc = lib.absb_build_centroids(C.byref(cl), C.byref(batch_c), fake, fake, fake, fake, ws, C.c_size_t(nbytes),
                                      None)
        assert rc == absb.ERR_WORKSPACE
    # selection list narrower than the plan's K
    rc = lib.absb_topk(C.byref(cl), C.byref(batch_c), fake, fake, fake, C.c_int32(plan.sel_stride - 1), None,
                       C.c_size_t(0), None)
    assert rc == absb.ERR_BAD_SHAPE
    rc = lib.absb_sparse_decode(C.byref(cl), C.byref(batch_c), fake, fake, fake, fake, fake, C.c_int32(0), fake,
                                None, fake, C.c_size_t(0), None)
    assert rc == absb.ERR_BAD_SHAPE


def test_launch_options_are_per_call_and_validated():
    """absb_launch_opts travels with the batch of a call: invalid values are refused before anything
    is enqueued, valid ones change the plan of that batch only (another batch object keeps the
    library's choices), and the library exports no process-wide knob."""
    layer = absb.Layer(8, 2, 128, 64, absb.F16, [8, 128], (2 * 64 * 128, 64 * 128, 128))

    def batch(**opts):
        return absb.Batch(seq_lens_host=[4096, 100], budget_host=[512, 64], pt_stride=64, opts=absb.LaunchOpts(**opts))
    base = absb.absb_plan(layer, batch()).workspace_bytes
    assert absb.absb_plan(layer, batch(split_tokens=64)).workspace_bytes >= base      # more splits, more partials
    assert absb.absb_plan(layer, batch()).workspace_bytes == base                     # ... for that batch only
    for bad in (dict(split_tokens=100), dict(split_tokens=-64), dict(score_chunk=65), dict(unit_tokens=32),
                dict(counters_zero=2), dict(counters_zero=-1), dict(step_form=4), dict(step_form=-1)):
        with pytest.raises(absb.AbsbError) as e:
            absb.absb_plan(layer, batch(**bad))
        assert e.value.status == absb.ERR_BAD_SHAPE, bad
        with pytest.raises(absb.AbsbError) as e:
            absb.absb_step_form_used(layer, batch(**bad))
        assert e.value.status == absb.ERR_BAD_SHAPE, bad
    for ok in (dict(split_tokens=128), dict(score_chunk=512), dict(unit_tokens=256), dict(counters_zero=1),
               dict(step_form=1), dict(step_form=2), dict(step_form=3)):
        absb.absb_plan(layer, batch(**ok))
    assert not hasattr(absb.load(), "absb_set_tuning")


@pytest.mark.parametrize("make", [list, lambda v: np.array(v, np.int64), lambda v: np.array(v, np.int32)])
def test_reassigning_one_field_takes_in_what_changed_in_place_in_the_others(make):
    """Lists and arrays of another type are converted, tensors held by address: edited in place, they are as the
    caller sees them once any field has been reassigned."""
    import torch
    lens, table = make([64, 100]), torch.zeros((2, 4), dtype=torch.int32)
    batch = absb.Batch(seq_lens_host=lens, budget_host=[8, 8], page_table=table)
    batch.c()
    lens[0] = 256
    table.resize_((2, 64))
    batch.budget_host = [16, 16]
    rec = batch.c()
    assert C.cast(rec.seq_lens_host, C.POINTER(C.c_int32))[0] == 256
    assert C.cast(rec.budget_host, C.POINTER(C.c_int32))[1] == 16
    assert rec.page_table == table.data_ptr() and rec.pt_stride == 64


def test_a_second_thread_gets_the_reassigned_fields_while_the_first_carries_them_over(monkeypatch):
    """A scheduler reassigns a batch's lengths, then two threads call with it: whichever comes second must not be
    handed the record from before the reassignment while the first one is still at work on the new one."""
    batch = _batch((64,), (8,))
    batch.c()
    batch.seq_lens_host = [128]
    real, inside, go, got = absb._i32_host, threading.Event(), threading.Event(), []

    def slow(a):
        inside.set()
        go.wait(10)
        return real(a)
    monkeypatch.setattr(absb, "_i32_host", slow)
    length = lambda: C.cast(batch.c().seq_lens_host, C.POINTER(C.c_int32))[0]  # noqa: E731
    threads = [threading.Thread(target=lambda: got.append(length())) for _ in range(2)]
    threads[0].start()
    assert inside.wait(10)
    monkeypatch.setattr(absb, "_i32_host", real)
    threads[1].start()
    threads[1].join(0.2)                       # (returns at once with a stale record, or waits for the first thread)
    go.set()
    for t in threads:
        t.join(10)
    assert got == [128, 128]


def test_enqueue_form_of_the_fused_step_follows_the_longest_segment():
    """Pipelined one-launch step while no segment has more than 16384 blocks and no list more than 4096
    entries; beyond 16384 blocks the shared selection, while its estimation work-groups are few enough or mostly
    have work; one launch per stage otherwise; the option forces any of them; the workspace always has room
    for the counters of the one-launch forms."""
    def form(L, B, batch_size=2, budget=64, **opts):
        layer = absb.Layer(8, 2, 128, 64, absb.F16, [B, 128], (2 * 64 * 128, 64 * 128, 128))
        batch = absb.Batch(seq_lens_host=[L] + [100] * (batch_size - 1), budget_host=[budget] * batch_size,
                           pt_stride=(L + 63) // 64, opts=absb.LaunchOpts(**opts))
        return absb.absb_step_form_used(layer, batch), absb.absb_plan(layer, batch).workspace_bytes
    P, U, S = absb.STEP_PIPELINED, absb.STEP_UNITS, absb.STEP_PER_STAGE
    assert form(8192 * 8, 8)[0] == P
    assert form(16384 * 8, 8)[0] == P
    assert form(131072, 16)[0] == P
    assert form(16384 * 8 + 1, 8, batch_size=4)[0] == U        # beyond: the selection is shared
    assert form(16384 * 8 + 1, 8, batch_size=8)[0] == S        # ... unless most of a large grid is empty
    assert form(8192 * 8, 8, budget=4096 * 8)[0] == P
    assert form(8192 * 8, 8, budget=4096 * 8 + 1)[0] == S      # lists of more than 4096 blocks
    assert form(4096, 8, step_form=S)[0] == S
    assert form(4096, 8, step_form=U)[0] == U
    assert form(131072, 8, step_form=P)[0] == P
    nseg = 2 * 2
    assert form(4096, 8)[1] >= 6 * nseg * 256 + 256
    with pytest.raises(absb.AbsbError):
        absb.absb_step_form_used(absb.Layer(8, 2, 128, 64, absb.F16, [8, 8], (16384, 8192, 128)),
                                 absb.Batch(seq_lens_host=[64], budget_host=None, pt_stride=1))


def test_product_package_does_not_reach_the_oracle():
    # the product path must not import, link, load or execute anything under oracle/
    pkg = os.path.join(ROOT, "paper_2605_12110_amd")
    bad = re.compile(r"^\s*(from|import)\s+oracle\b|liboracle|absb_oracle|oracle[/.]oracle", re.M)
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                assert not bad.search(open(os.path.join(dirpath, f)).read()), f


def test_selection_rejects_segments_beyond_its_capacity_before_any_launch():
    """A segment of more than 2^17 blocks does not fit the selection kernel's bitmap: the call must
    say so on the host (nothing is launched, so plain host buffers serve as arguments here)."""
    import torch
    L = (8 << 17) + 1                                        # 131073 blocks of 8 tokens
    layer = _layer(num_q_heads=1, num_kv_heads=1, block_size=[8], kv_strides=(64 * 128, 64 * 128, 128))
    fake = torch.zeros(4, dtype=torch.int32)
    batch = absb.Batch(seq_lens_host=[L], budget_host=[64], pt_stride=(L + 63) // 64, cent_off=fake, budget=fake,
                       seq_lens=fake)
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_topk(layer, batch, fake, fake, fake, 8, stream=0)
    assert e.value.status == absb.ERR_UNSUPPORTED
    with pytest.raises(absb.AbsbError) as e:                 # the whole step: refused before its first stage is enqueued
        absb.absb_decode_fused(layer, batch, fake, fake, fake, fake, fake, fake, None, None, None, fake, stream=0)
    assert e.value.status == absb.ERR_UNSUPPORTED
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_step_form_used(layer, batch)
    assert e.value.status == absb.ERR_UNSUPPORTED


def test_block_size_assignment_rule_matches_the_oracle_on_the_host():
    """Eq. (2) is host-only integer work in the library: identical to the oracle on identical recalls."""
    from oracle import oracle as O
    rng = np.random.default_rng(5)
    cand = [8, 16, 32, 64, 128]
    for tau in (0.5, 0.9, 0.98, 1.0):
        rec = rng.uniform(0.0, 1.0, size=(7, 9, 5)).astype(np.float32)
        rec[:, :, 0] = np.maximum(rec[:, :, 0], 0.8)
        got, mean = absb.absb_assign_block_sizes(rec, cand, tau)
        want, wmean = O.assign_block_sizes(rec.astype(np.float64), cand, tau)
        assert np.array_equal(got, want) and np.array_equal(mean, wmean)
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_assign_block_sizes(rec, [8, 16, 32, 64, 96], 0.9)
    assert e.value.status == absb.ERR_BAD_BLOCK_SIZE


def test_block_size_assignment_rule_on_cases_worked_by_hand():
    """Eq. (2) on tables small enough to do in the head (two samples, exact binary fractions).  Head 0
    falls off at 32; head 1 dips at 16 and recovers at 32 (the set is read as written: its maximum wins);
    head 2 never keeps the share, so B_min it is; head 3 keeps it everywhere."""
    cand = [8, 16, 32, 64]
    sample0 = [[1.0, 1.0, 0.5, 0.25], [0.5, 0.25, 0.5, 0.125], [1.0, 0.5, 0.5, 0.5], [0.5, 0.5, 0.5, 0.5]]
    sample1 = [[0.5, 0.5, 0.5, 0.25], [1.0, 0.25, 0.75, 0.125], [1.0, 0.5, 0.25, 0.5], [1.0, 1.0, 1.0, 1.0]]
    rec = np.array([sample0, sample1], np.float32)
    sizes, mean = absb.absb_assign_block_sizes(rec, cand, 0.75)
    assert np.array_equal(mean, [[0.75, 0.75, 0.5, 0.25], [0.75, 0.25, 0.625, 0.125], [1.0, 0.5, 0.375, 0.5],
                                 [0.75, 0.75, 0.75, 0.75]])
    assert sizes.tolist() == [16, 32, 8, 64]
    # tau = 1: only candidates that lose nothing; tau = 0: the largest candidate, always
    assert absb.absb_assign_block_sizes(rec, cand, 1.0)[0].tolist() == [16, 8, 8, 64]
    assert absb.absb_assign_block_sizes(rec, cand, 0.0)[0].tolist() == [64, 64, 64, 64]
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_assign_block_sizes(rec, [8, 32, 16, 64, 128], 0.9)
    assert e.value.status == absb.ERR_BAD_SHAPE


def test_plan_accepts_65535_selection_segments_and_no_more():
    # selection segments index the second grid dimension of the per-stage kernels
    lens, T = [64] * 65535, [8] * 65535
    one = _layer(num_q_heads=3, num_kv_heads=1, block_size=[16])
    assert absb.absb_plan(one, _batch(lens, T)).total_centroids == 4 * 65535
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_plan(one, _batch(lens + [64], T + [8]))
    assert e.value.status == absb.ERR_BAD_SHAPE
    per_q = _layer(num_q_heads=3, num_kv_heads=1, block_size=[16], selection=absb.SELECT_PER_QUERY_HEAD)
    assert absb.absb_plan(per_q, _batch(lens[:21845], T[:21845])).total_centroids == 4 * 21845
    with pytest.raises(absb.AbsbError):
        absb.absb_plan(per_q, _batch(lens[:21846], T[:21846]))


def test_plan_lays_the_store_out_for_the_capacity_lengths_when_given():
    layer = _layer()
    tight = absb.absb_plan(layer, _batch((1000,), (64,)))
    roomy = absb.absb_plan(layer, absb.Batch(seq_lens_host=[1000], budget_host=[64], pt_stride=64, cap_lens_host=[4096]))
    full = absb.absb_plan(layer, _batch((4096,), (64,)))
    assert np.array_equal(roomy.cent_off, full.cent_off) and roomy.total_centroids == full.total_centroids
    assert roomy.sel_stride == tight.sel_stride                       # selection sizes follow the current lengths
    with pytest.raises(absb.AbsbError) as e:                          # a layout shorter than the context
        absb.absb_plan(layer, absb.Batch(seq_lens_host=[1000], budget_host=[64], pt_stride=64, cap_lens_host=[999]))
    assert e.value.status == absb.ERR_BAD_SHAPE


def test_a_workspace_planned_for_the_capacity_serves_every_length_on_the_way():
    """Longer lists get longer splits, and so at times fewer partials: the plan of a layout with room to grow covers
    the lengths before the last ones, too (what the step needs at lengths L is at least the tight plan's)."""
    rng = np.random.default_rng(3)
    for trial in range(60):
        kv, G = int(rng.choice([2, 8])), int(rng.choice([1, 4, 8]))
        layer = _layer(num_q_heads=kv * G, num_kv_heads=kv, block_size=[int(x) for x in rng.choice([8, 16, 32, 64], kv)],
                       selection=int(rng.integers(0, 3)))
        n = int(rng.integers(1, 17))
        cap = rng.integers(40, 20000 if trial % 2 else 1200, n)
        budget = [int(rng.choice([300, 2048, 9310]))] * n
        wide = dict(pt_stride=1 << 16)
        room = absb.absb_plan(layer, _batch(cap.tolist(), budget, cap_lens_host=cap.tolist(), **wide)).workspace_bytes
        for back in (0, 1, 7, 30, *rng.integers(1, 20000, 12)):
            lens = np.maximum(1, cap - back).tolist()
            assert room >= absb.absb_plan(layer, _batch(lens, budget, **wide)).workspace_bytes, (trial, lens)
            grown = absb.absb_plan(layer, _batch(lens, budget, cap_lens_host=cap.tolist(), **wide)).workspace_bytes
            assert grown >= room                   # ... whatever lengths it is asked at


@pytest.mark.parametrize("repr_", [0, 1])
def test_a_workspace_planned_for_a_long_capacity_serves_the_builds_on_the_way(repr_):
    """A longer context can be built by fewer work-groups (more tokens each), which share less: the plan of a layout with
    room to grow covers the shorter ones, too.  Every part of it follows from the capacity then, so that it is the same
    at whatever lengths it is asked; lengths and capacities around all changes of the work-groups' size, alone and mixed."""
    rng = np.random.default_rng(5 + repr_)
    edge = 512 * 512                                     # tokens that 512 work-groups of one run of 512 take
    caps = [edge - 1, edge, edge + 1, 270000, 300000, 2 * edge + 1, 3 * edge + 1, 7 * edge + 1, 8 * edge, 8 * edge + 1, 9 * edge]
    layer = _layer(num_q_heads=8, num_kv_heads=8, block_repr=repr_)
    for cap in caps:
        on_the_way = {1, 1000, cap // 2, cap - 1, cap, *rng.integers(1, cap, 8).tolist()}
        on_the_way |= {k * edge + d for k in range(1, 10) for d in (-30000, -5, 0, 1, 4096) if 0 < k * edge + d <= cap}
        for other in (None, 700, edge):
            caps_b = [cap] if other is None else [cap, other]
            sizes = {absb.absb_plan(layer, _batch([L] + caps_b[1:], [512] * len(caps_b), cap_lens_host=caps_b,
                                                  pt_stride=1 << 16)).workspace_bytes for L in sorted(on_the_way)}
            assert len(sizes) == 1, (cap, other, sorted(sizes))


def test_room_to_grow_does_not_change_the_form_of_the_step():
    """The form follows the lengths, whatever the layout has room for: batches on both sides of what decides between the
    shared selection and a launch per stage (how many of its work-groups there are and how many of them have blocks)."""
    layer = _layer(block_size=[8, 16, 32, 64, 8, 16, 32, 64])
    def used(lens, cap):
        batch = _batch(lens, [2048] * len(lens), cap_lens_host=cap, pt_stride=1 << 14)
        return absb.absb_step_form_used(layer, batch)
    seen = set()
    for lens in ([262144] * 4, [200000, 3000, 3000, 3000], [262144] * 12, [150000] + [2000] * 15, [140000] * 2, [300000, 300000, 10000]):
        want = used(lens, None)
        seen.add(want)
        for grow in (1, 2, 4):
            assert used(lens, [grow * n for n in lens]) == want, (lens, grow)
        assert used(lens, [1 << 20] * len(lens)) == want, lens
    assert seen == {absb.STEP_UNITS, absb.STEP_PER_STAGE}
