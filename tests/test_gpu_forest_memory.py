"""Device memory kept from destroyed forests goes back to the device on request,
so that any other allocator of the process can have it, and the next forest
takes it back in time."""
import pytest

from tests.gpu_util import banner, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def test_trim_gives_everything_back(dev):
    import torch
    import paper_1801_08361_amd as rl
    p = rl.params_default(n_trees=16, depth=13, reservoir_size=1024, max_modes=10)
    rl.Forest(p).close()   # what the runtime itself keeps is there before the first reading
    rl.trim()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    banner("two forests of 2.8 GB, created and destroyed")
    fs = [rl.Forest(p) for _ in range(2)]
    assert torch.cuda.mem_get_info()[0] < free0 - (4 << 30)
    for f in fs:
        f.close()
    rl.trim()
    # 64 MB is the runtime's own granularity; a reservoir table has 2 GB
    assert torch.cuda.mem_get_info()[0] >= free0 - (64 << 20)
    rl.trim()
    f = rl.Forest(p)
    assert f.memory() > 2 << 30
    f.close()
    rl.trim()
    assert torch.cuda.mem_get_info()[0] >= free0 - (64 << 20)
