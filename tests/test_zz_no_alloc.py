"""absb_decode_fused_static (the step on the library's built-in scratch array, for callers that cannot
allocate) against absb_decode_fused with a caller-owned workspace, through the C ABI: same
selection bit for bit, outputs within the attention tolerance, on two calls in a row of which
the second is the smaller one (its counters sit elsewhere in the array, which still holds the
first call's data).  Collected last: a failure here must not hide the other GPU tests."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_12110_amd import synth

pytestmark = pytest.mark.gpu

TOL = {synth.F16: 2e-3, synth.BF16: 1e-2}


def _both_entry_points(wl, what, opts=None, fits=True):
    import torch
    from paper_2605_12110_amd import absb
    from paper_2605_12110_amd.device import DeviceWorkload
    print(f"[no-alloc {what}] Bt={wl.batch} L={wl.seq_lens.tolist()} B={wl.block_size.tolist()} "
          f"T={wl.budget.tolist()} dtype={wl.dtype}", flush=True)
    dw = DeviceWorkload(wl, opts=opts)
    assert (dw.plan.workspace_bytes <= absb.STATIC_WORKSPACE_BYTES) == fits
    dw.build()
    # the existing entry point, on the caller's workspace
    dw.decode_fused()
    torch.cuda.synchronize()
    want_out = dw.out.float().cpu().numpy().astype(np.float64)
    want_lse = dw.lse.cpu().numpy().astype(np.float64)
    want_idx, want_cnt = dw.sel_idx.cpu().numpy().copy(), dw.sel_cnt.cpu().numpy().copy()
    # the new one: outputs poisoned first, everything it needs allocated before the call
    dw.out.fill_(float("nan")); dw.lse.fill_(float("nan")); dw.sel_idx.fill_(-7); dw.sel_cnt.fill_(-7)
    torch.cuda.synchronize()
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    absb.absb_decode_fused_static(dw.layer, dw.batch, dw.q, dw.codes, dw.qscale, dw.k_cache, dw.v_cache, dw.out,
                                  dw.lse, dw.sel_idx, dw.sel_cnt)
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before      # not through torch either
    torch.cuda.synchronize()
    got_out = dw.out.float().cpu().numpy().astype(np.float64)
    got_lse = dw.lse.cpu().numpy().astype(np.float64)
    assert np.array_equal(dw.sel_cnt.cpu().numpy(), want_cnt)
    assert np.array_equal(dw.sel_idx.cpu().numpy(), want_idx)
    err = np.abs(got_out - want_out).max()
    print(f"    max|out(static) - out(workspace)| = {err:.3e}", flush=True)
    assert np.isfinite(got_out).all() and err <= TOL[wl.dtype]
    assert np.abs(got_lse - want_lse).max() <= 1e-4
    # and the oracle agrees with what both computed
    ref = O.decode_step(wl, O.build_centroids(wl))
    K = dw.sel_stride
    assert np.array_equal(want_idx, ref["sel_idx"][:, :K]) and np.array_equal(want_cnt, ref["sel_cnt"])
    assert np.abs(got_out - ref["out"]).max() <= TOL[wl.dtype]


def test_zz_static_scratch_step_matches_workspace_step_twice_second_call_smaller():
    big = synth.make_workload(1, batch=3, context=6144, budget=768, seed=71)         # 24 segments
    small = synth.make_workload(1, batch=1, context=1100, budget=200, seed=72)       # 8 segments, ragged tail
    _both_entry_points(big, "first call")
    _both_entry_points(small, "second call, smaller")


@pytest.mark.parametrize("form", [0, 2])
def test_zz_static_scratch_gives_up_the_shared_selection_before_the_call(form):
    """512 segments: the step needs 15.3 MiB, with the shared selection's rows 17.4: more than the array has.  The call
    is taken all the same (asked for the form that shares, too), and so is a smaller one after it."""
    near = synth.tiny_workload(seed=73, Hq=128, Hkv=32, P=16, seq_lens=(18,) * 15 + (1200,), block_size=(8, 32, 16, 128) * 8,
                               budget=(16,) * 15 + (832,))
    small = synth.make_workload(1, batch=1, context=1100, budget=200, seed=74)
    _both_entry_points(near, f"near the array's size, form {form}", dict(step_form=form, split_tokens=64), fits=False)
    _both_entry_points(small, "smaller, after it", dict(step_form=form))


def test_zz_static_scratch_refuses_what_it_cannot_hold():
    """Host-side check only: nothing is enqueued for a batch that needs more than the array holds."""
    from paper_2605_12110_amd import absb
    Hkv = 8
    layer = absb.Layer(32, Hkv, 128, 64, absb.F16, [8] * Hkv, (Hkv * 64 * 128, 64 * 128, 128))
    lens = [1 << 20] * 8                                       # 8 x 1 Mi tokens at block size 8: 4 MiB of scores per request
    batch = absb.Batch(seq_lens_host=lens, budget_host=[4096] * 8, pt_stride=(1 << 20) // 64)
    assert absb.absb_plan(layer, batch).workspace_bytes > absb.STATIC_WORKSPACE_BYTES
    with pytest.raises(absb.AbsbError) as e:
        absb.absb_decode_fused_static(layer, batch, 1, 1, 1, 1, 1, 1)
    assert e.value.status == absb.ERR_STATIC_WORKSPACE
