"""The order of the batched server's batches on the device, by their events: a batch issued behind
one that fills the GPU starts when that one has ended, and requests fewer than overlap_backlog wait
for the batch in flight.  Images are those of the requests alone, and the batches in flight
together stay within the budget."""
import pytest

import workloads as wl
from tests.test_gpu_parity import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bank():
    from paper_2510_05814_amd.serve import ModelBank
    return ModelBank([wl.random_model(3000, 3, 1, 500, 500, 40 + i) for i in range(2)], 3, 1)


@pytest.mark.parametrize("how,budget_mb", [("behind", 4096), ("behind", 500), ("backlog", 4096)])
def test_batches_follow_each_other(bank, how, budget_mb):
    import torch

    import paper_2510_05814_amd as smoe
    from paper_2510_05814_amd.serve import RenderRequest, Server
    say("serving order", how, budget_mb)
    reqs = [RenderRequest(model=i % 2, scale=4, width=2000 - 7 * i, height=1990 + i, origin_x=i,
                          origin_y=2 * i) for i in range(8)]
    more = dict(fill_blocks=1, max_batch=2) if how == "behind" else dict(
        fill_blocks=1 << 30, overlap_backlog=9, max_batch=1)
    srv = Server(bank, budget_bytes=budget_mb << 20, streams=2, **more)
    for _ in range(2):     # (the first run also grows the streams' workspaces)
        res, summ = srv.serve(reqs, realtime=False, keep_outputs=True)
    assert summ["peak_bytes"] <= summ["budget_bytes"]
    assert summ["batches"] == (4 if how == "behind" else 8)
    batches = {}
    for r in res:
        batches.setdefault(r.batch, []).append(r)
    order = [batches[k] for k in sorted(batches)]
    for a, b in zip(order, order[1:]):
        assert b[0].started >= a[0].done - 2e-6, (b[0].batch, b[0].started, a[0].done)
    for r in res:
        q = r.request
        grid = smoe.make_grid(q.width, q.height, q.scale, q.origin_x, q.origin_y)
        img, _, _, _ = smoe.render(bank.rows(q.model), 3, 1, grid)
        assert torch.equal(r.image, img)
