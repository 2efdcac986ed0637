"""JobLauncher over job lists around the number of records that travel in the
launch's arguments, with and without a volume in one list, in the default and
in a given shape; bitwise each stack's own deskew."""
import pytest
import torch

import paper_2211_00645_amd as dsk
from paper_2211_00645_amd.batch import JobLauncher, plan_job

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_jobs", [1, 2, 9, 32, 33])
@pytest.mark.parametrize("tune", [None, dict(block=128, per_thread=8, unroll=1)])
def test_job_lists(n_jobs, tune):
    g = torch.Generator().manual_seed(n_jobs)
    launcher = JobLauncher(max_jobs=40)
    for mixed in (False, True):
        jobs, keep = [], []
        for i in range(n_jobs):
            shape = (1 + 7 * i % 23, 1 + 5 * i % 19, 1 + 37 * i % 301)
            st = torch.randint(0, 65536, shape, generator=g, dtype=torch.int32).to(torch.uint16).to(DEV)
            job, out = plan_job(st, 35.0, 0.4, 0.115, vol=not (mixed and i % 2))
            jobs.append(job)
            keep.append((st, out))
        for _ in range(2):
            launcher.launch(jobs, tune=tune)
        torch.cuda.synchronize()
        for st, out in keep:
            ref = dsk.deskew(st, 35.0, 0.4, 0.115)
            for k in ("vol", "psum", "pmax"):
                if k in out:
                    assert torch.equal(out[k], ref[k]), (tuple(st.shape), k)


def test_large_and_small_stacks_together():
    """Stacks that go out in launches of their own beside ones that share one."""
    launcher = JobLauncher(max_jobs=4)
    jobs, keep = [], []
    for shape in ((9, 20, 61), (64, 512, 2048), (30, 31, 200)):
        st = torch.randint(0, 65536, shape, dtype=torch.int32, device=DEV).to(torch.uint16)
        job, out = plan_job(st, 35.0, 0.4, 0.115)
        jobs.append(job)
        keep.append((st, out))
    assert keep[1][1]["vol"].numel() * 4 > 280e6
    launcher.launch(jobs)
    torch.cuda.synchronize()
    for st, out in keep:
        ref = dsk.deskew(st, 35.0, 0.4, 0.115)
        for k in ("vol", "psum", "pmax"):
            assert torch.equal(out[k], ref[k]), (tuple(st.shape), k)
