"""The autotuner on clouds whose walks are cut into parts shorter than most of
its splits: those splits give the same tasks and share one timing."""
import itertools

import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,c", [(2000, 2.0), (20000, 8.0)])
def test_equal_tasks_are_timed_once(n, c):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2405_16634_amd as w
    w.load_library()
    print(f"[case] autotune splits {n} c={c}", flush=True)
    ctx = w.Context(0)
    x, _ = ctx.normalize(torch.from_numpy(synth.fibonacci_sphere(n, 1).points).to("cuda:0"))
    ctx.build(x, c)
    tasks = {}
    for split in (0, 64, 128, 256, 512, 1024):
        ctx.set_split(split)
        tasks[split] = ctx.stats()["n_tasks"]
    assert tasks[256] == tasks[1024] != tasks[0]
    ms = ctx.autotune(0.002)
    assert len(ms) == w.AUTOTUNE_CONFIGS and all(t > 0 for t in ms.values())
    for pf, (a, b) in itertools.product((0, 1), itertools.combinations(sorted(tasks), 2)):
        if tasks[a] == tasks[b]:
            assert ms[1, pf, a] == ms[1, pf, b], (pf, a, b, ms)
    # the tasks kept are those of the split reported
    assert ctx.tile() != 1 or ctx.stats()["n_tasks"] == tasks[ctx.split()]
    ctx.close()
