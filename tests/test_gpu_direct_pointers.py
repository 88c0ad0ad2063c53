"""Calls over at most eight tensors (single passes over channel scales alone: sixty-four) carry their device pointers in the
kernel's arguments, larger ones in a table in the workspace: both have to give the same bits, whatever was called before and
wherever in the context the call starts."""
import pytest
import torch

import paper_2507_17511_amd as cf

pytestmark = pytest.mark.gpu

KINDS = {"channel": (cf.CF_SCALE_CHANNEL, 128, 2), "group": (cf.CF_SCALE_GROUP, 128, 4), "sparse": (cf.CF_SPARSE_NM, 8, 2),
         "lowrank": (cf.CF_LOWRANK, 32, 1), "sparse16": (cf.CF_SPARSE_NM, 16, 2), "rank1": (cf.CF_SCALE_RANK1, 128, 2)}
DTYPES = {"mixed": lambda k: cf.CF_BF16 if k % 3 else cf.CF_F32, "bf16": lambda k: cf.CF_BF16, "f32": lambda k: cf.CF_F32}


class _Side:
    """One context of ten tensors with their buffers, all made from the same seed.  Among channel scales the last one is a group
    scale, with which a call reads the table."""

    def __init__(self, kind, dtypes="mixed", **options):
        scale, group, bits = KINDS[kind]
        self.descs = [cf.desc(40 + 7 * k, 384, DTYPES[dtypes](k), bits, scale, group) for k in range(10)]
        if kind == "channel":
            self.descs[9] = cf.desc(103, 384, DTYPES[dtypes](9), 4, cf.CF_SCALE_GROUP)
        opts = cf.options(**options)
        nbytes = cf.cf_workspace_bytes(self.descs, opts)
        self.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        self.stream = torch.cuda.current_stream().cuda_stream
        self.ctx = cf.cf_init(self.descs, opts, self.ws, nbytes, self.stream)
        g = torch.Generator(device="cuda")
        g.manual_seed(7)
        sizes = [cf.cf_sizes(d, opts) for d in self.descs]
        blank = lambda col: [torch.zeros(max(16, s[col]), dtype=torch.uint8, device="cuda") for s in sizes]
        self.codes, self.scales, self.recon, self.err = blank(0), blank(1), blank(2), blank(3)
        if kind == "lowrank":
            for t in self.scales:
                t.view(torch.float32).normal_(generator=g)
        self.xs = []
        for _ in range(2):
            self.xs.append([torch.randn(d.n_tokens, d.n_channels, generator=g, device="cuda").to(
                torch.bfloat16 if d.dtype == cf.CF_BF16 else torch.float32) for d in self.descs])

    def calls(self, pieces):
        """Warm-up, a step, a send and a receive, each in calls over the given pieces of the context."""
        at = lambda bufs, p: cf.ptr_array(bufs[p[0]:p[0] + p[1]])
        for p in pieces:
            cf.cf_warmup(self.ctx, *p, at(self.xs[0], p), at(self.recon, p), at(self.err, p), self.stream)
        for p in pieces:
            cf.cf_step_fused(self.ctx, *p, at(self.xs[1], p), at(self.recon, p), at(self.err, p), at(self.codes, p), at(self.scales, p), self.stream)
        for p in pieces:
            cf.cf_compress(self.ctx, *p, at(self.xs[0], p), at(self.recon, p), at(self.err, p), at(self.codes, p), at(self.scales, p), self.stream)
        for p in pieces:
            cf.cf_decompress(self.ctx, *p, at(self.codes, p), at(self.scales, p), at(self.recon, p), self.stream)
        torch.cuda.synchronize()

    def outputs(self):
        return self.codes + self.scales + self.recon + self.err


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("pieces", [[(0, 1), (1, 8), (9, 1)], [(0, 9), (9, 1)], [(2, 8), (0, 2)]])
def test_pointers_in_arguments_and_in_the_table_give_the_same_bits(kind, pieces):
    whole, cut = _Side(kind), _Side(kind)
    for _ in range(2):
        whole.calls([(0, 10)])
        cut.calls(pieces)
        for a, b in zip(whole.outputs(), cut.outputs()):
            assert torch.equal(a, b)
    cut.calls([(0, 10)])        # the table again, after calls that left it alone
    whole.calls([(0, 10)])
    for a, b in zip(whole.outputs(), cut.outputs()):
        assert torch.equal(a, b)
    for side in (whole, cut):
        cf.cf_destroy(side.ctx)


# (kind, storage types, options): the kernels have an instance for each feedback mode, error type, mix of storage types and wire
FORMS = [(kind, dtypes, dict(ef=ef, err_dtype=err))
         for kind in ("group", "sparse", "sparse16", "rank1", "channel")
         for ef, err, dtypes in ((cf.CF_EF_RECON, cf.CF_BF16, "bf16"), (cf.CF_EF_LITERAL, cf.CF_F32, "mixed"), (cf.CF_EF_LITERAL, cf.CF_BF16, "f32"),
                                 (cf.CF_EF_OFF, cf.CF_F32, "bf16"), (cf.CF_EF_OFF, cf.CF_BF16, "mixed"), (cf.CF_EF_NAIVE, cf.CF_F32, "f32"),
                                 (cf.CF_EF_NAIVE, cf.CF_BF16, "bf16"))]
FORMS += [(kind, dtypes, dict()) for kind in ("group", "sparse", "sparse16", "rank1", "lowrank") for dtypes in ("bf16", "f32")]
FORMS += [("sparse16", "mixed", dict()), ("rank1", "mixed", dict())]
FORMS += [("lowrank", dtypes, dict(err_dtype=err, flags=cf.CF_FLAG_LOWRANK_INT4)) for dtypes, err in (("mixed", cf.CF_F32), ("bf16", cf.CF_BF16), ("f32", cf.CF_F32))]


@pytest.mark.parametrize("kind, dtypes, options", FORMS)
def test_every_form_of_the_kernels_by_both_routes(kind, dtypes, options):
    """Ten tensors a call read the table, calls of eight and fewer bring their pointers: two warm-ups, steps, sends and receives."""
    whole, cut = _Side(kind, dtypes, **options), _Side(kind, dtypes, **options)
    try:
        for _ in range(2):
            whole.calls([(0, 10)])
            cut.calls([(0, 8), (8, 2)])
            for a, b in zip(whole.outputs(), cut.outputs()):
                assert torch.equal(a, b)
    finally:
        for side in (whole, cut):
            cf.cf_destroy(side.ctx)


@pytest.mark.parametrize("kind", ["group", "sparse", "sparse16"])
def test_direct_calls_on_another_stream_and_from_a_graph(kind):
    """Calls that bring their pointers, between calls by the table on the context's own stream: on a second stream, and captured with
    other inputs and replayed, against the same calls one after the other on one stream."""
    side, plain = _Side(kind), _Side(kind)
    other = torch.cuda.Stream()
    own = side.stream
    try:
        for s in (side, plain):
            s.calls([(0, 10)])
        plain.calls([(0, 8), (8, 2)])
        side.stream = other.cuda_stream             # calls() ends with a synchronisation
        side.calls([(0, 8), (8, 2)])
        side.stream = own
        for a, b in zip(side.outputs(), plain.outputs()):
            assert torch.equal(a, b)
        at = lambda bufs, first, count: cf.ptr_array(bufs[first:first + count])
        fed = [x.clone() for x in side.xs[0]]

        def step(s, xs, stream):
            cf.cf_step_fused(s.ctx, 2, 8, at(xs, 2, 8), at(s.recon, 2, 8), at(s.err, 2, 8), at(s.codes, 2, 8), at(s.scales, 2, 8), stream)

        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            step(side, fed, torch.cuda.current_stream().cuda_stream)
        for k in range(4):
            side.calls([(0, 10)])                   # the table's pointers, and a synchronisation
            plain.calls([(0, 10)])
            for x, y in zip(fed, side.xs[k % 2]):
                x.copy_(y).mul_(1.0 + k)
            g.replay()
            step(plain, [y * (1.0 + k) for y in plain.xs[k % 2]], plain.stream)
            torch.cuda.synchronize()
            for a, b in zip(side.outputs(), plain.outputs()):
                assert torch.equal(a, b), f"replay {k}"
    finally:
        for s in (side, plain):
            cf.cf_destroy(s.ctx)
