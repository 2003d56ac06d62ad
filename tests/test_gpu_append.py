"""GPU append against the oracle, bit for bit, where the lookup and the launch shape change: one token
per workgroup up to 2,048 tokens and eight beyond, loaded early up to 2,560 waves (20,480 tokens of one wave each) and
in turn beyond, and waves of more than 64 requests (bisection, then one candidate per lane) with idle requests
between active ones."""
import numpy as np
import pytest

import oracle
import paper_2609_35263_amd as wp
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16, 1, 64, 64), (16, 16, 128, 128), (16, 1, 576, 512)])
@pytest.mark.parametrize("requests,total", [(1, 1), (64, 65), (65, 100), (200, 2048), (200, 2049), (3, 2055),
                                            (200, 20480), (200, 20485)])
def test_append_matches_oracle(shape, requests, total):
    import torch
    Hq, Hkv, dk, dv = shape
    rng = np.random.default_rng(requests * 4099 + total)
    chunk = rng.multinomial(total, rng.dirichlet(np.full(requests, 0.3)))     # many requests get no token
    spec = wl.custom_wave(Hq, Hkv, dk, dv, 16, rng.integers(0, 70, requests), chunk, kv_shared=dk == 576,
                          seed=total)
    print(f"[append] {shape} R={requests} T={total} idle={int((chunk == 0).sum())}", flush=True)
    t = wl.make_tensors(spec, seed=7)
    bits = {k: wl.to_bits(v) for k, v in t.items()}
    k_ref, v_ref = oracle.append_kv(bits["k_pool"], bits["v_pool"], bits["k_new"], bits["v_new"], spec.prefix_lens,
                                    spec.chunk_lens, spec.block_table, spec.page_size)
    d = {k: None if v is None else v.cuda() for k, v in t.items()}
    p = wp.plan_for(spec)
    ws = wp.new_workspace(p)
    wp.plan_upload(p, ws)
    wp.append_kv(p, d["k_new"], d["v_new"], d["k_pool"], d["v_pool"], ws)
    torch.cuda.synchronize()
    assert np.array_equal(wl.to_bits(d["k_pool"]), k_ref)
    assert v_ref is None or np.array_equal(wl.to_bits(d["v_pool"]), v_ref)
