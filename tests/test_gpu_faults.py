"""Error paths of the boundary, forced from the host (PRNU_FAULT): a device failure marks
the context failed, the failing call and every later call return PRNU_E_DEVICE, and
every video in the serving engine ends with PRNU_E_DEVICE.  The injected fault fires
before any of the failing call's GPU work is issued, so the GPU itself never fails."""
import os
import sys

import numpy as np
import pytest

from paper_2207_14507_amd import synth

pytestmark = pytest.mark.gpu

GRID = (5, 0.97, 1.03, 5, -1.0, 1.0)


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2207_14507_amd import prnu
    return prnu


def faulty_context(P, spec):
    os.environ["PRNU_FAULT"] = spec
    try:
        return P.prnu_create(0, flags=P.PRNU_FLAG_NO_AUTOTUNE)
    finally:
        del os.environ["PRNU_FAULT"]


def expect_device_error(P, fn, *args, **kw):
    with pytest.raises(P.PrnuError) as e:
        fn(*args, **kw)
    assert e.value.status == P.PRNU_E_DEVICE, e.value


def test_launch_fault_poisons_the_synchronous_path(P):
    seq = synth.tiny(n_frames=2, config=70)
    opts = P.make_opts(grid=GRID, radius=16)
    ctx = faulty_context(P, "launch:2")
    try:
        fp = P.prnu_open_fingerprint(ctx, seq.K)
        res, _ = P.prnu_search_frames(ctx, fp, seq.frames, opts)   # launch 1: fine
        assert all(r.status == 0 for r in res)
        expect_device_error(P, P.prnu_search_frames, ctx, fp, seq.frames, opts)   # launch 2: injected
        expect_device_error(P, P.prnu_search_frames, ctx, fp, seq.frames, opts)   # failed earlier
        expect_device_error(P, P.prnu_open_fingerprint, ctx, seq.K)
        expect_device_error(P, P.prnu_submit_video, ctx, fp, seq.frames, opts)
    finally:
        P.prnu_destroy(ctx)
    # a fresh context is unaffected
    ctx = P.prnu_create(0, flags=P.PRNU_FLAG_NO_AUTOTUNE)
    try:
        fp = P.prnu_open_fingerprint(ctx, seq.K)
        again, _ = P.prnu_search_frames(ctx, fp, seq.frames, opts)
        assert [r.pce for r in again] == [r.pce for r in res]
    finally:
        P.prnu_destroy(ctx)


def test_launch_fault_ends_every_video_in_the_engine(P):
    seqs = [synth.walk_sequence(71, i, 256, 256, 6, radius=8) for i in range(3)]
    opts = P.make_opts(grid=GRID, radius=16, warm=True, local=(3, 3, 0.005, 0.2), fallback_pce=60.0)
    ctx = faulty_context(P, "launch:3")
    try:
        fps = [P.prnu_open_fingerprint(ctx, s.K) for s in seqs]
        tickets = []
        for fp, s in zip(fps, seqs):
            # a submission may already meet the failed engine: it is refused the same way
            try:
                tickets.append(P.prnu_submit_video(ctx, fp, s.frames, opts))
            except P.PrnuError as e:
                assert e.status == P.PRNU_E_DEVICE
            say("submitted", len(tickets))
        for t, s in zip(tickets, seqs):
            say("polling", t)
            expect_device_error(P, P.prnu_poll, ctx, t, len(s.frames), 30000)
        expect_device_error(P, P.prnu_submit_video, ctx, fps[0], seqs[0].frames, opts)
    finally:
        P.prnu_destroy(ctx)


def test_staging_fault(P):
    seq = synth.tiny(n_frames=1, config=72)
    opts = P.make_opts(grid=GRID, radius=16)
    ctx = faulty_context(P, "stage:1")
    try:
        fp = P.prnu_open_fingerprint(ctx, seq.K)
        expect_device_error(P, P.prnu_search_frames, ctx, fp, seq.frames, opts)
        expect_device_error(P, P.prnu_score_grid, ctx, fp, seq.frames, 0, opts)
    finally:
        P.prnu_destroy(ctx)


@pytest.mark.parametrize("spec", ["grow:1", "grow:2"])
def test_a_refused_larger_workspace_leaves_the_smaller_batches(P, spec):
    """A fallback grid of 361 candidates against batches of 256 asks for one larger
    workspace; where the card has no room for it, the chain runs in the batches it had,
    with the same results, in that call and in later ones.  (The second growth, of another
    shape, on a workspace that already grew once.)"""
    opts = P.make_opts(grid=(19, 0.97, 1.03, 19, -1.0, 1.0), radius=16, warm=True, local=(3, 3, 0.005, 0.2),
                       fallback_pce=1e12)
    seqs = [synth.walk_sequence(73, i, M, N, 3, radius=8) for i, (M, N) in enumerate([(160, 160), (256, 256)])]

    def run(ctx):
        out = []
        for s in seqs + seqs[:1]:
            fp = P.prnu_open_fingerprint(ctx, s.K)
            out += [(r.status, r.cand_index, r.fell_back, r.n_evaluated, r.pce, r.rho, r.dx, r.dy)
                    for r in P.prnu_search_frames(ctx, fp, s.frames, opts)[0]]
            P.prnu_close_fingerprint(ctx, fp)
        return out

    ctx = P.prnu_create(0, flags=P.PRNU_FLAG_NO_AUTOTUNE)
    try:
        want = run(ctx)
    finally:
        P.prnu_destroy(ctx)
    assert all(w[0] == 0 for w in want) and sum(w[2] for w in want) == 6
    ctx = faulty_context(P, spec)
    try:
        assert run(ctx) == want
        assert run(ctx) == want
    finally:
        P.prnu_destroy(ctx)


def test_a_failed_wait_on_closing_poisons_the_context(P):
    """A spectrum whose readers are not known to have finished is not handed on, and the
    device error is not lost."""
    seq = synth.tiny(n_frames=1, config=74)
    ctx = faulty_context(P, "close:2")
    try:
        first, second = P.prnu_open_fingerprint(ctx, seq.K), P.prnu_open_fingerprint(ctx, seq.K)
        P.prnu_close_fingerprint(ctx, first)
        expect_device_error(P, P.prnu_close_fingerprint, ctx, second)
        expect_device_error(P, P.prnu_open_fingerprint, ctx, seq.K)
        with pytest.raises(P.PrnuError) as e:
            P.prnu_close_fingerprint(ctx, second)
        assert e.value.status == P.PRNU_E_HANDLE   # closed all the same
    finally:
        P.prnu_destroy(ctx)


def test_spare_spectra_are_given_back_when_memory_is_short(P):
    """The spectra kept from closed fingerprints, of any context on the device, make room
    for whatever cannot be allocated."""
    import torch
    seq = synth.walk_sequence(75, 0, 160, 160, 2, radius=8)
    wide = synth.fingerprint(synth.rng(75), 1080, 1920)
    small, large = (P.make_opts(grid=(n, 0.97, 1.03, n, -1.0, 1.0), radius=16, warm=True, local=(3, 3, 0.005, 0.2),
                                fallback_pce=1e12) for n in (16, 19))
    other = P.prnu_create(0, flags=P.PRNU_FLAG_NO_AUTOTUNE)
    ctx = faulty_context(P, "grow:1")
    try:
        for c in (other, ctx):   # 8.3 MB each
            P.prnu_close_fingerprint(c, P.prnu_open_fingerprint(c, wide))
        fp = P.prnu_open_fingerprint(ctx, seq.K)
        P.prnu_search_frames(ctx, fp, seq.frames, small)   # batches of 256, as large as the next search's
        before = torch.cuda.mem_get_info()[0]
        res, _ = P.prnu_search_frames(ctx, fp, seq.frames, large)   # asks for one of 361, refused
        assert [r.status for r in res] == [0, 0] and res[1].fell_back == 1
        freed = torch.cuda.mem_get_info()[0] - before
        say("freed", freed)
        assert freed > 12 << 20
        # both contexts go on: spectra are allocated anew
        for c in (other, ctx):
            P.prnu_close_fingerprint(c, P.prnu_open_fingerprint(c, wide))
    finally:
        P.prnu_destroy(ctx)
        P.prnu_destroy(other)
