"""GPU parity: clipping of low bits (Section 3.2 "Clipping") against the CPU oracle.  The
message bytes must be bit-exact; the error v - Q[v] is exact in fp32, so errors agree too."""
import pytest
import torch

import ds_workloads as W
import paper_1905_05957_amd as P
from parity_util import Pair

pytestmark = pytest.mark.gpu


def _wl(d, bits, n=3, **kw):
    base = dict(name=f"clip{bits}_d{d}", comp="clip", n=n, d=d, clip_bits=bits, dist="normal", sigma=1e-2, gamma=0.05)
    base.update(kw)
    return W.Workload(**base)


def _run(wl, device, steps=2):
    pair = Pair(wl, device)
    try:
        for t in range(steps):
            pair.compared_step(t, wl.gradients(t % 2, device))
    finally:
        pair.close()


@pytest.mark.parametrize("bits", [1, 8, 16, 20, 24, 31])
@pytest.mark.parametrize("d", [1, 7, 2048, 2049, 5 * 2048 + 37, 100_003])
def test_clip_shapes_and_widths(gpu_device, d, bits):
    _run(_wl(d, bits), gpu_device)


def test_clip_bf16_gradients_and_momentum(gpu_device):
    _run(_wl(50_000, 16, n=4, grad_dtype="bf16", beta=0.9), gpu_device, steps=3)


def test_clip_many_workers_and_extreme_values(gpu_device):
    wl = _wl(30_001, 16, n=19)
    pair = Pair(wl, gpu_device)
    try:
        g = wl.gradients(0, gpu_device)
        g[:, :8] = torch.tensor([0.0, -0.0, 1e-40, -3e-42, 3.0e38, -1.17549435e-38, 1.0, -1.0], device=gpu_device)
        pair.compared_step(0, g)
        pair.compared_step(1, g)
    finally:
        pair.close()


@pytest.mark.parametrize("n", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("bits,beta", [(8, None), (16, 0.9), (24, None)])
def test_clip_batches_of_workers_and_the_update_in_one_call(gpu_device, n, bits, beta):
    """Partial and full batches of eight messages of every width, rows that end inside a group of four, and the model
    updated in the server's pass: bit for bit what the two calls give, which are compared with the oracle here."""
    wl = W.Workload(f"clip{bits}", "clip", n=n, d=2 * 2048 + 1027, clip_bits=bits, dist="normal", sigma=1e-3, gamma=0.05, beta=beta)
    two, one = Pair(wl, gpu_device), Pair(wl, gpu_device)
    try:
        for t in range(2):
            g = wl.gradients(t, gpu_device)
            two.compared_step(t, g)
            one.ctx.worker_compress(t, g, one.delta, one.pw)
            one.ctx.server_aggregate_compress_update(t, one.pw, one.delta_s, one.ps, one.x, one.m, wl.gamma, beta or 0.0)
            assert torch.equal(one.x, two.x) and torch.equal(one.delta_s, two.delta_s) and torch.equal(one.ps.levels, two.ps.levels)
            assert one.m is None or torch.equal(one.m, two.m)
    finally:
        two.close()
        one.close()


@pytest.mark.parametrize("n,d,update", [(12, 8_400_003, None), (24, 4_200_003, 1), (24, 4_200_001, 2)])
def test_clip_servers_that_take_messages_one_by_one(gpu_device, n, d, update):
    """Many long messages of four bytes an element are taken one by one, short ones in batches; every element stands for
    itself, so stretches of the long rows are what a short context gives for them.  update: none, without and with momentum."""
    def server(ctx, msg, e, out, x, m):
        if update is None:
            ctx.server_aggregate_compress(0, msg, e, out)
        else:
            ctx.server_aggregate_compress_update(0, msg, e, out, x, m if update == 2 else None, 0.05, 0.9)

    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(1)
    long = P.Context("clip", n, d, levels=8)
    try:
        msg, out = long.alloc_payload(n, gpu_device), long.alloc_server_payload(gpu_device)
        msg.levels.view(torch.int32).copy_(torch.randn((n, d), device=gpu_device, generator=gen).view(torch.int32) & ~255)
        err, x, m = (torch.randn(d, device=gpu_device, generator=gen) for _ in range(3))
        before = [t.clone() for t in (err, x, m)]
        server(long, msg, err, out, x, m)
        for first, last in ((0, 5003), (4_000_000, 4_003_000), (d - 2051, d)):
            short = P.Context("clip", n, last - first, levels=8)
            part, got = short.alloc_payload(n, gpu_device), short.alloc_server_payload(gpu_device)
            part.levels.copy_(msg.levels[:, 4 * first: 4 * last])
            e, xs, ms = (t[first:last].clone() for t in before)
            server(short, part, e, got, xs, ms)
            torch.cuda.synchronize()
            short.close()
            assert torch.equal(got.levels, out.levels[:, 4 * first: 4 * last])
            assert torch.equal(e, err[first:last]) and torch.equal(xs, x[first:last]) and torch.equal(ms, m[first:last])
    finally:
        long.close()
