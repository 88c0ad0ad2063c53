"""Calls over at most eight tensors carry their device pointers in the kernel's arguments, larger ones in a table in the
workspace: both have to give the same bits, whatever was called before and wherever in the context the call starts."""
import pytest
import torch

import paper_2507_17511_amd as cf

pytestmark = pytest.mark.gpu

KINDS = {"channel": (cf.CF_SCALE_CHANNEL, 128, 2), "group": (cf.CF_SCALE_GROUP, 128, 4), "sparse": (cf.CF_SPARSE_NM, 8, 2),
         "lowrank": (cf.CF_LOWRANK, 32, 1)}


class _Side:
    """One context of ten tensors with their buffers, all made from the same seed."""

    def __init__(self, kind):
        scale, group, bits = KINDS[kind]
        self.descs = [cf.desc(40 + 7 * k, 384, cf.CF_BF16 if k % 3 else cf.CF_F32, bits, scale, group) for k in range(10)]
        opts = cf.options()
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
