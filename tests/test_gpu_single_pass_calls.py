"""Calls of one context after one another: the single pass carries a bit per partial sum from one call to the next, so
which tensors a call covers, by which route their pointers come, and whether its workgroups wait must not matter."""
import pytest
import torch

import paper_2507_17511_amd as cf
from helpers import drift_stream, run_parity
from paper_2507_17511_amd.session import CodecSession

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("flags", [0, cf.CF_FLAG_FIXED_GRID, cf.CF_FLAG_TEST_NO_WAIT])
@pytest.mark.parametrize("ef", [cf.CF_EF_RECON, cf.CF_EF_OFF])
def test_calls_over_changing_ranges(ef, flags):
    """Ten channel-scale tensors, groups of one item to six, and one of group scales: calls with that one by the table of pointers,
    the others with their pointers as arguments, up to eight tensors with their descriptors too; one tensor alone, odd and even
    numbers of calls for each tensor; every output bit for bit what the two-kernel path gives in the same sequence."""
    shapes = [(1500, 1096), (700, 520), (1, 8), (257, 256), (256, 264), (129, 72), (1030, 512), (300, 3072), (64, 64), (511, 1032)]
    descs = [cf.desc(n, c, cf.CF_F32 if t % 4 == 1 else cf.CF_BF16, (1, 2, 4)[t % 3], cf.CF_SCALE_CHANNEL) for t, (n, c) in enumerate(shapes)]
    descs.append(cf.desc(70, 256, cf.CF_BF16, 4, cf.CF_SCALE_GROUP))
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=4, seed=910 + t, device=DEV) for t, d in enumerate(descs)]
    one = CodecSession(descs, cf.options(ef=ef, flags=cf.CF_FLAG_SINGLE_PASS | flags), device=DEV)
    two = CodecSession(descs, cf.options(ef=ef, flags=cf.CF_FLAG_TWO_KERNEL), device=DEV)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for event in events:
        event.record()              # before it has a handle
    uploads = 0
    try:
        for sess in (one, two):
            sess.warmup([s[0] for s in streams])
        for k, (first, count) in enumerate([(0, 11), (0, 3), (1, 9), (7, 1), (7, 1), (3, 8), (0, 8), (2, 8), (0, 10), (0, 11), (9, 1), (0, 10), (0, 11), (0, 10)]):
            x = [s[1 + k % 3] for s in streams]
            cf.cf_profile_next_call(one.ctx, [e.cuda_event for e in events], 1)
            for sess in (one, two):
                sess.step_fused(x[first:first + count], first, count)
            cf.cf_check_device(one.ctx, one.stream_handle)
            kernels = [cf.cf_profile_kernel_name(one.ctx, j) for j in range(cf.cf_profile_launch_count(one.ctx))]
            short = ef == cf.CF_EF_RECON and flags != cf.CF_FLAG_FIXED_GRID and count <= 8 and first + count < 11
            name = "k_short_items" if short else "k_single_pass"
            assert name in kernels and (first + count == 11 or kernels == [name])
            uploads += "k_upload_ptrs" in kernels
            say(f"ef={ef} flags={flags} call {k}: tensors {first}..{first + count - 1}, {cf.cf_given_up_items(one.ctx, one.stream_handle)} items given up")
            for t in range(len(descs)):
                for name in ("codes", "scales", "recon", "err"):
                    a, b = getattr(one, name)[t], getattr(two, name)[t]
                    assert torch.equal(a.view(torch.uint8).reshape(-1), b.view(torch.uint8).reshape(-1)), f"call {k}: {name}[{t}]"
        assert uploads == 3         # the last of four calls by the table finds there what the one before left
    finally:
        one.close()
        two.close()


@pytest.mark.parametrize("dtype", [cf.CF_BF16, cf.CF_F32])
@pytest.mark.parametrize("err_dtype", [cf.CF_F32, cf.CF_BF16])
@pytest.mark.parametrize("flags", [0, cf.CF_FLAG_TEST_NO_WAIT])
def test_short_items(dtype, err_dtype, flags):
    """Small calls, whose items are 128 rows of bf16 (64 of fp32) x 64 channels: token counts and widths around one item and
    around the longest group, 64 items, every code width, fused and split; bits against the oracle."""
    rows = 64 if dtype == cf.CF_F32 else 128
    shapes = [(1, 8, 1), (rows - 1, 56, 2), (rows, 64, 4), (rows + 1, 72, 1), (8 * rows + 1, 136, 2), (9 * rows - 1, 120, 4), (64 * rows, 64, 2), (63 * rows + 1, 32, 1)]
    descs = [cf.desc(n, c, dtype, bits, cf.CF_SCALE_CHANNEL) for n, c, bits in shapes]
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=3, seed=980 + t, device=DEV) for t, d in enumerate(descs)]
    xs = [[streams[t][s] for t in range(len(descs))] for s in range(3)]
    say(f"short items dtype={dtype} err_dtype={err_dtype} flags={flags}: {shapes}")
    for mode in ("fused", "split"):
        run_parity(descs, cf.options(err_dtype=err_dtype, flags=flags), xs, mode=mode)


@pytest.mark.parametrize("dtype", [cf.CF_BF16, cf.CF_F32])
@pytest.mark.parametrize("flags", [0, cf.CF_FLAG_TEST_NO_WAIT])
@pytest.mark.parametrize("shapes", [[(64, 1), (1, 2816)],                                               # row blocks of one item, 64-channel stripes: 64 x 1 and 1 x 44
                                    [(1, 1), (9, 320), (0.1, 2048), (64, 64), (3, 136), (12, 200)],     # a chunk of the largest alone, groups of 1 to 64
                                    [(16, 512), (8, 512)], [(16, 512), (7, 512)]])                      # 64 and 72 workgroups that would have no item: both sides of the line
def test_short_items_of_unlike_tensors(shapes, dtype, flags):
    """Calls whose tensors have few row blocks or stripes in common, one workgroup per item, and ones with a workgroup for each of the most; a
    part of the context's tensors too; every code width, bits against the oracle."""
    rows = 64 if dtype == cf.CF_F32 else 128
    descs = [cf.desc(max(1, int(n * rows)), max(8, c // 8 * 8), dtype, (1, 2, 4)[t % 3], cf.CF_SCALE_CHANNEL) for t, (n, c) in enumerate([(2, 64)] + shapes)]
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=4, seed=1020 + t, device=DEV) for t, d in enumerate(descs)]
    xs = [[streams[t][s] for t in range(len(descs))] for s in range(4)]
    say(f"short items of unlike tensors dtype={dtype} flags={flags}: {[(d.n_tokens, d.n_channels) for d in descs]}")
    run_parity(descs[1:], cf.options(flags=flags), [x[1:] for x in xs], mode="fused")
    run_parity(descs[1:], cf.options(flags=flags, err_dtype=cf.CF_BF16), [x[1:] for x in xs], mode="split")
    part, whole = (CodecSession(descs, cf.options(flags=flags), device=DEV) for _ in range(2))
    try:
        for sess in (part, whole):
            sess.warmup(xs[0])
        for x in xs[1:]:
            part.step_fused(x[:1], 0, 1)
            part.step_fused(x[1:], 1, len(descs) - 1)
            whole.step_fused(x)
        torch.cuda.synchronize()
        for t in range(len(descs)):
            for name in ("codes", "scales", "recon", "err"):
                assert torch.equal(getattr(part, name)[t], getattr(whole, name)[t]), f"{name}[{t}]"
    finally:
        part.close()
        whole.close()


UNEVEN_ROWS = [(21, 1153, (328, 264, 1096)),        # 256 channels, 10 items a group: none begins where the one before did
               (30, 4700, (104, 136, 72)),          # 128 channels, 19 items
               (2, 16387, (424, 408))]              # 64 channels, 33 items


def uneven_rows(n, tokens, widths, options, mode, steps):
    descs = [cf.desc(tokens - t % 3, widths[t % len(widths)], cf.CF_BF16, (1, 2, 4)[(t + t // 3) % 3], cf.CF_SCALE_CHANNEL) for t in range(n)]
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=steps, seed=870 + t, device=DEV) for t, d in enumerate(descs)]
    xs = [[streams[t][s] for t in range(n)] for s in range(steps)]
    say(f"uneven rows {n} x [{tokens}, {widths}] {mode} err_dtype={options['err_dtype']} flags={options['flags']}")
    run_parity(descs, cf.options(**options), xs, mode=mode)


@pytest.mark.parametrize("err_dtype", [cf.CF_F32, cf.CF_BF16])
@pytest.mark.parametrize("flags", [0, cf.CF_FLAG_TEST_NO_WAIT])
@pytest.mark.parametrize("n, tokens, widths", UNEVEN_ROWS + [(30, 1024, (1104, 336, 16)),           # channels a multiple of 16, up to four 128-channel items; 8 items
                                                             (2, 12291, (552, 568)),                # 128 channels, 49 items
                                                             (2, 4097, (760, 776)), (2, 4097, (752, 784))])        # short items, 33 a group
def test_rows_of_no_whole_blocks(n, tokens, widths, err_dtype, flags):
    """bf16 rows that are no whole blocks of 64 bytes, whose parts are stored another way in calls that write enough: code widths in turn,
    fused and split; bits against the oracle."""
    for mode in ("fused", "split"):
        uneven_rows(n, tokens, widths, dict(err_dtype=err_dtype, flags=cf.CF_FLAG_SINGLE_PASS | flags), mode, 3)


@pytest.mark.parametrize("n, tokens, widths", UNEVEN_ROWS)
def test_sent_rows_of_no_whole_blocks_with_bf16_errors(n, tokens, widths):
    """The same where a call writes bf16 errors alone: twice the tensors."""
    uneven_rows(2 * n, tokens, widths, dict(err_dtype=cf.CF_BF16, flags=cf.CF_FLAG_SINGLE_PASS), "split", 2)


def test_small_call_replays_from_a_graph():
    """A captured call that carries its pointers: replays, eager calls and a warm-up in turn, against an eager context."""
    descs = [cf.desc(1024, 512, cf.CF_BF16, 2, cf.CF_SCALE_CHANNEL), cf.desc(900, 384, cf.CF_BF16, 1, cf.CF_SCALE_CHANNEL)]
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=8, seed=950 + t, device=DEV) for t, d in enumerate(descs)]
    graphed, eager = (CodecSession(descs, cf.options(flags=cf.CF_FLAG_SINGLE_PASS), device=DEV) for _ in range(2))
    try:
        x = [s[0].clone() for s in streams]
        for sess in (graphed, eager):
            sess.warmup(x)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            graphed.step_fused(x)
        for k in range(1, 8):
            for t in range(len(descs)):
                x[t].copy_(streams[t][k])
            if k == 6:
                for sess in (graphed, eager):
                    sess.warmup([s[0] for s in streams])
            if k in (3, 4):
                graphed.step_fused(x)
            else:
                g.replay()
            eager.step_fused([s[k] for s in streams])
            torch.cuda.synchronize()
            for t in range(len(descs)):
                for name in ("codes", "scales", "recon", "err"):
                    assert torch.equal(getattr(graphed, name)[t], getattr(eager, name)[t]), f"step {k}: {name}[{t}]"
    finally:
        graphed.close()
        eager.close()


@pytest.mark.parametrize("ef", [cf.CF_EF_RECON, cf.CF_EF_NAIVE])
def test_streams_in_turn(ef):
    """Calls of one context on two streams in turn, each after the other has been waited for: short items (default feedback mode, up
    to eight tensors) and tall ones, and warm-ups of some tensors in between, which set the bits of their partial sums anew then and
    must leave their neighbours' as they are; against two kernels."""
    shapes = [(700, 520), (1, 8), (1030, 512), (64, 72), (2600, 264), (129, 72), (511, 1032), (257, 256), (300, 64)]
    descs = [cf.desc(n, c, cf.CF_F32 if t % 4 == 1 else cf.CF_BF16, (1, 2, 4)[t % 3], cf.CF_SCALE_CHANNEL) for t, (n, c) in enumerate(shapes)]
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=4, seed=870 + t, device=DEV) for t, d in enumerate(descs)]
    one = CodecSession(descs, cf.options(ef=ef, flags=cf.CF_FLAG_SINGLE_PASS), device=DEV)
    two = CodecSession(descs, cf.options(ef=ef, flags=cf.CF_FLAG_TWO_KERNEL), device=DEV)
    other = torch.cuda.Stream(device=DEV)
    try:
        for sess in (one, two):
            sess.warmup([s[0] for s in streams])
        calls = [(0, 9, 0), (0, 3, 0), (3, 1, 1), (0, 9, 1), (2, 1, 0), (1, 8, 1), (4, 1, 1), (0, 9, 0), (8, 1, 1), (0, 9, 0), (0, 8, 0)]
        warm = {3: (2, 3), 4: (4, 1), 6: (0, 9), 7: (0, 1), 9: (5, 4)}         # before these calls
        for k, (first, count, where) in enumerate(calls):
            x = [s[1 + k % 3] for s in streams]
            if k in warm:
                two.warmup(x[warm[k][0]:sum(warm[k])], *warm[k])
            two.step_fused(x[first:first + count], first, count)
            torch.cuda.synchronize()
            with torch.cuda.stream(other if where else torch.cuda.current_stream()):
                if k in warm:
                    one.warmup(x[warm[k][0]:sum(warm[k])], *warm[k])
                one.step_fused(x[first:first + count], first, count)
                cf.cf_check_device(one.ctx, one.stream_handle)
                assert cf.cf_given_up_items(one.ctx, one.stream_handle) == 0
            say(f"ef={ef} call {k}: tensors {first}..{first + count - 1} on stream {where}")
            for t in range(len(descs)):
                for name in ("codes", "scales", "recon", "err"):
                    a, b = getattr(one, name)[t], getattr(two, name)[t]
                    assert torch.equal(a.view(torch.uint8).reshape(-1), b.view(torch.uint8).reshape(-1)), f"call {k}: {name}[{t}]"
    finally:
        one.close()
        two.close()


@pytest.mark.parametrize("ef, err_dtype, shapes", [
    (cf.CF_EF_RECON, cf.CF_F32, [(8192, 64), (4096, 512), (1000, 136)]),       # short items, 64 a group
    (cf.CF_EF_RECON, cf.CF_BF16, [(8192, 64), (4096, 512), (1000, 136)]),
    (cf.CF_EF_RECON, cf.CF_F32, [(4097, 760), (4097, 776)]),                   # short items, rows of no whole blocks of 64 bytes
    (cf.CF_EF_RECON, cf.CF_F32, [(9000, 136), (4096, 512)]),                   # too many for them: 128-channel stripes
    (cf.CF_EF_RECON, cf.CF_F32, [(9000, 520), (9000, 536)]),                   # the same, rows of no whole blocks
    (cf.CF_EF_RECON, cf.CF_F32, [(12500, 224), (20000, 96)]),                  # 64-channel stripes
    (cf.CF_EF_RECON, cf.CF_BF16, [(12500, 224), (20000, 96)]),
    (cf.CF_EF_RECON, cf.CF_F32, [(16400, 424), (20000, 136)]),                 # rows of no whole blocks
    (cf.CF_EF_RECON, cf.CF_F32, [(2000, 1056)] * 9),                           # more than eight tensors: 256-channel stripes
    (cf.CF_EF_RECON, cf.CF_F32, [(2000, 1032)] * 9),                           # rows of no whole blocks
    (cf.CF_EF_OFF, cf.CF_F32, [(4096, 512), (1000, 136)]),
    (cf.CF_EF_NAIVE, cf.CF_BF16, [(4096, 512), (1000, 136)]),
])
def test_missing_partial_sums_are_computed(ef, err_dtype, shapes):
    """CF_FLAG_TEST_NO_WAIT in every geometry of items: some are given up, their workgroups store other items' partial sums while those
    start, publish and write over their operands, and the bits are those of an ordinary run, in which nobody gives up."""
    descs = [cf.desc(n, c, cf.CF_BF16, (2, 1, 4)[t % 3], cf.CF_SCALE_CHANNEL) for t, (n, c) in enumerate(shapes)]
    streams = [drift_stream((d.n_tokens, d.n_channels), d.dtype, steps=4, seed=830 + t, device=DEV) for t, d in enumerate(descs)]
    options = dict(ef=ef, err_dtype=err_dtype)
    hasty = CodecSession(descs, cf.options(flags=cf.CF_FLAG_SINGLE_PASS | cf.CF_FLAG_TEST_NO_WAIT, **options), device=DEV)
    quiet = CodecSession(descs, cf.options(flags=cf.CF_FLAG_SINGLE_PASS, **options), device=DEV)
    try:
        gave_up = 0
        for k in range(4):
            for sess in (hasty, quiet):
                (sess.step_fused if k else sess.warmup)([s[k] for s in streams])
                cf.cf_check_device(sess.ctx, sess.stream_handle)
            if k == 0:
                continue
            gave_up += cf.cf_given_up_items(hasty.ctx, hasty.stream_handle)
            assert cf.cf_given_up_items(quiet.ctx, quiet.stream_handle) == 0
            for t in range(len(descs)):
                for name in ("codes", "scales", "recon", "err"):
                    assert torch.equal(getattr(hasty, name)[t], getattr(quiet, name)[t]), f"call {k}: {name}[{t}]"
        say(f"ef={ef} {shapes}: {gave_up} items given up in three calls")
        assert gave_up > 0, "nobody helped"
    finally:
        hasty.close()
        quiet.close()
