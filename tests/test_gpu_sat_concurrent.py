"""hb_sat2d's one-launch tables on two streams at once, each call with a workspace of its own: the two grids share the compute units, so
neither need be resident as a whole, and workgroups clear the words, stop waiting and finish for others as it comes.  0/1 images: exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limit", [0, 2, -1])                 # the default, a few polls, "stop waiting at once"
@pytest.mark.parametrize("shapes", [((4096, 4096), (4096, 4096)), ((2817, 2815), (1024, 1024)), ((300, 257), (4096, 4000))])
def test_two_streams(shapes, limit):
    import torch
    from paper_2512_02371_amd import hb
    gen = torch.Generator(device="cuda").manual_seed(1)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    calls = []
    for s, (H, W) in zip(streams, shapes):
        x = (torch.rand(H, W, generator=gen, device="cuda") < 0.4).half()
        ws = torch.full((hb.hb_sat2d_workspace_size(H, W),), 0xff, dtype=torch.uint8, device="cuda")
        calls.append((s, x, [torch.full((H, W), 7.0, device="cuda") for _ in range(4)], ws))
    torch.cuda.synchronize()
    print(f"hb_sat2d on two streams {shapes} limit {limit}", flush=True)
    prev = hb.hb_sat2d_set_wait_limit(limit)
    try:
        for i in range(4):
            for s, x, outs, ws in calls:
                with torch.cuda.stream(s):
                    hb.hb_sat2d(x, outs[i], ws)
        torch.cuda.synchronize()
    finally:
        hb.hb_sat2d_set_wait_limit(prev)
    for _, x, outs, _ in calls:
        want = x.cpu().double().cumsum(0).cumsum(1)
        for out in outs:
            assert torch.equal(out.cpu().double(), want)
