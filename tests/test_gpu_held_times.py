"""GPU: times of the route that holds rows on chip, against the launches that it stands for and in the
forms that a working program does not normally reach.  The bounds leave a factor to the noise of a shared
machine; what they catch is a fallback or a choice of size that costs several times the plain way."""
import pytest
import torch

import paper_1905_05957_amd as P

pytestmark = pytest.mark.gpu

NOFB_SID = P.FLAG_NO_ERROR_FEEDBACK | P.FLAG_SERVER_IDENTITY


def best_us(call, calls=10, runs=5):
    """GPU time of one call of a captured run of calls, the best of `runs`."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        for _ in range(calls):
            call()
    best = float("inf")
    for _ in range(runs):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


class Sign:
    """Buffers and calls of one 1-bit context with one scale per vector."""

    def __init__(self, dev, n, d, dtype="f32", **kw):
        gen = torch.Generator(device=dev)
        gen.manual_seed(d)
        self.ctx = P.Context("sign", n, d, grad_dtype=dtype, scale_mode="whole", **kw)
        self.g = torch.randn((n, d), device=dev, generator=gen).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        self.delta = torch.zeros((n, d), device=dev)
        self.delta_s, self.x = torch.zeros(d, device=dev), torch.zeros(d, device=dev)
        self.msg, self.out = self.ctx.alloc_payload(n, dev), self.ctx.alloc_server_payload(dev)
        self.ctx.worker_compress(0, self.g, self.delta, self.msg)

    def worker(self):
        self.ctx.worker_compress(0, self.g, self.delta, self.msg)

    def two_looks(self):
        P.ds_worker_compress_sign_noalloc(self.g, self.delta, self.msg.sign_words, self.msg.scales)

    def server(self):
        self.ctx.server_aggregate_compress_update(0, self.msg, self.delta_s, self.out, self.x, None, 0.05)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_worker_call_that_gives_up_costs_what_two_looks_cost(gpu_device, dtype):
    s = Sign(gpu_device, 8, 11_173_962, dtype, topk_spin_limit=-1)
    gave_up, plain = best_us(s.worker), best_us(s.two_looks)
    s.ctx.close()
    assert gave_up < 2.0 * plain, (gave_up, plain)


def test_a_server_call_that_gives_up_costs_what_separate_launches_cost(gpu_device):
    s = Sign(gpu_device, 8, 11_173_962, topk_spin_limit=-1)
    apart = Sign(gpu_device, 8, 11_173_962, flags=P.FLAG_DEFERRED_ERROR)
    gave_up, plain = best_us(s.server), best_us(apart.server)
    s.ctx.close()
    apart.ctx.close()
    assert gave_up < 2.5 * plain, (gave_up, plain)     # `plain` looks once at the error


# Short rows and rows of few workers, where a launch costs as much as the work: the sizes that are taken may
# not cost more than the launches that they stand for.
@pytest.mark.parametrize("n", [1, 8, 16])
@pytest.mark.parametrize("d,dtype", [(4 * 2048, "bf16"), (8 * 2048 - 2, "f32"), (12 * 2048, "bf16"), (14 * 2048 - 3, "f32"), (20 * 2048 + 1, "f32"),
                                     (24 * 2048, "f32"), (24 * 2048 - 1, "bf16"), (30 * 2048, "f32"), (300_001, "f32"), (1_000_003, "f32")])
def test_a_short_row_costs_no_more_than_two_looks(gpu_device, n, d, dtype):
    s = Sign(gpu_device, n, d, dtype)
    held, plain = best_us(s.worker, 30), best_us(s.two_looks, 30)
    s.ctx.close()
    assert held < 1.25 * plain, (held, plain)


@pytest.mark.parametrize("n,d", [(1, 4 * 2048), (8, 4 * 2048), (16, 4 * 2048), (64, 2 * 2048), (1, 8 * 2048), (8, 12 * 2048), (16, 16 * 2048),
                                 (4, 24 * 2048), (16, 24 * 2048), (4, 1_000_003), (200, 2_500_001), (64, 11_173_962)])
def test_a_server_call_costs_no_more_than_separate_launches(gpu_device, n, d):
    us = []
    for flags in (0, P.FLAG_DEFERRED_ERROR):
        ctx = P.Context("sign", n, d, scale_mode="whole", flags=flags)
        msg, out = ctx.alloc_payload(n, gpu_device), ctx.alloc_server_payload(gpu_device)
        delta_s, x = torch.zeros(d, device=gpu_device), torch.zeros(d, device=gpu_device)

        def call():     # the deferred form and its second look: the launches of the plain form, apart
            ctx.server_aggregate_compress_update(0, msg, delta_s, out, x, None, 0.05)
            ctx.materialize_error(None, delta_s)

        us.append(best_us(call, 30))
        ctx.close()
    assert us[0] < 1.15 * us[1], us


def test_a_ternary_call_that_gives_up(gpu_device):
    n, d = 8, 11_173_962
    g = torch.randn((n, d), device=gpu_device)
    us = []
    for patience in (0, -1):
        ctx = P.Context("ternary", n, d, flags=NOFB_SID, topk_spin_limit=patience)
        msg = ctx.alloc_payload(n, gpu_device)
        us.append(best_us(lambda: ctx.worker_compress(0, g, None, msg)))
        ctx.close()
    assert us[1] < 2.5 * us[0], us                      # the gradients are read once more and encoded apart


# The first shape has a fraction of the second one's work, or the same work on narrower gradients.
@pytest.mark.parametrize("less,more,factor", [((1, 1_000_003, "f32"), (8, 1_000_003, "f32"), 1.0), ((1, 5_000_003, "bf16"), (4, 5_000_003, "bf16"), 0.8),
                                              ((8, 24 * 2048, "f32"), (8, 100_001, "f32"), 1.3), ((4, 14 * 2048, "bf16"), (4, 100_001, "bf16"), 1.3),
                                              ((16, 11_173_962, "bf16"), (16, 11_173_962, "f32"), 1.25), ((3, 9_000_001, "f32"), (4, 9_000_001, "f32"), 0.9),
                                              ((5, 6_000_000, "bf16"), (6, 6_000_000, "bf16"), 0.9), ((8, 24_000_000, "bf16"), (8, 24_000_000, "f32"), 1.2)])
def test_ternary_times_follow_the_work(gpu_device, less, more, factor):
    us = []
    for n, d, dtype in (less, more):
        g = torch.randn((n, d), device=gpu_device).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
        ctx = P.Context("ternary", n, d, grad_dtype=dtype, flags=NOFB_SID)
        msg = ctx.alloc_payload(n, gpu_device)
        us.append(best_us(lambda: ctx.worker_compress(0, g, None, msg), 20))
        ctx.close()
    assert us[0] < factor * us[1], us


@pytest.mark.parametrize("d", [5000, 2_500_001])
def test_a_ternary_server_of_one_worker_costs_what_the_decoder_costs(gpu_device, d):
    """Both read one message and write it out."""
    ctx = P.Context("ternary", 1, d, flags=NOFB_SID)
    msg, out, dense = ctx.alloc_payload(1, gpu_device), ctx.alloc_server_payload(gpu_device), torch.empty(d, device=gpu_device)
    ctx.worker_compress(0, torch.randn((1, d), device=gpu_device), None, msg)
    server = best_us(lambda: ctx.server_aggregate_compress(0, msg, None, out), 50)
    decoder = best_us(lambda: ctx.decompress(msg, 0, dense), 50)
    ctx.close()
    assert server < 1.12 * decoder, (server, decoder)
