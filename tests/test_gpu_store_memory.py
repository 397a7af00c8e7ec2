"""A store on a device whose memory is nearly full: the bit planes are left out
rather than taken from what the batches need, and the kernels that do without
them give the same results."""
import numpy as np
import pytest

import oracle
from helpers import mutate_codes, rand_codes, workload_from
from test_gpu_parity import assert_same

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

import paper_2001_10049_amd as xd  # noqa: E402


def batch(store, w):
    pairs, seeds, x = xd.workload_tensors(w, "cuda")
    out = xd.align_batch(store, pairs, seeds, x=x, k=w.k, persistent=True)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


def test_planes_leave_room():
    rng = np.random.default_rng(2)
    reads, tasks = [], []
    for q in range(60):
        a = rand_codes(rng, 700)
        reads += [a, mutate_codes(rng, a, 0.1)]
        tasks.append((2 * q, 2 * q + 1, 300, min(300, len(reads[-1]) - 17), (7, 25, 50)[q % 3]))
    filler = np.resize(rand_codes(rng, 1 << 20), 1 << 22)
    w = workload_from(reads + [filler] * 128, tasks)  # 537 M bases: 134 MB packed
    ref = oracle.align_workload(w)
    at = np.arange(12_400) % len(tasks)  # as many as the lane tiers take
    want = {k: ref[k][at] for k in ("status", "score", "beg", "end", "cells")}
    many = w.subset(at)
    print("with planes", flush=True)
    store = xd.ReadStore.from_workload(w)
    with_planes = store.info()["device_bytes"]
    assert_same(batch(store, many), want, label="with planes")
    store.close()
    xd.release_memory()
    torch.cuda.empty_cache()
    print("filling the memory", flush=True)
    held = []
    try:
        while (free := torch.cuda.mem_get_info()[0]) > (3 << 30) // 4 + (64 << 20):
            held.append(torch.empty(min(free - ((3 << 30) // 4), 32 << 30), dtype=torch.uint8,
                                    device="cuda"))
        print("without", flush=True)
        store = xd.ReadStore.from_workload(w)
        assert store.info()["device_bytes"] < 0.6 * with_planes
        assert_same(batch(store, many), want, label="without planes")
        store.close()
    finally:
        held.clear()
        torch.cuda.empty_cache()
