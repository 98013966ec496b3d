"""The pinned staging ring under several threads: compressions on streams of their own, with tables and read-backs of
every size the ring treats differently, give what the same call gives alone."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,T", [(3, 300),       # a few KB each
                                     (160, 40)])     # 0.4 MB each: the ring of 2 MB wraps under the four threads
@pytest.mark.parametrize("mixed", [False, True])
def test_threads_share_the_staging_ring(batch, T, mixed):
    from paper_2605_08317_amd import binding as b
    hq, hkv, S_w = 8, 8, 32
    rng = np.random.default_rng(5)
    K, V = (torch.from_numpy(rng.standard_normal((batch * hkv * T, 128)).astype(np.float32)).to(torch.bfloat16).cuda()
            for _ in range(2))
    Q = torch.from_numpy(rng.standard_normal((batch, hq, S_w, 128)).astype(np.float32)).to(torch.bfloat16).cuda()
    q = torch.from_numpy(rng.standard_normal((batch, hq, 128)).astype(np.float32)).to(torch.bfloat16).cuda()
    kw = {"k_mode": b.RDKV_K_CHANNELWISE, "kv_split_rk": 0.5} if mixed else {}
    cfgs = [b.Config([T] * batch, hq, hkv, budget_bits=[x] * batch, s_obs=S_w, **kw) for x in (0.5, 1.0, 2.0, 4.0)]

    def run(cfg):
        cache = b.rdkv_compress(cfg, K, V, Q)
        out = b.rdkv_decode_attn(cache, q)[0].clone()
        torch.cuda.current_stream().synchronize()
        cache.free()
        return out

    print(f"[case] staging ring, 4 threads, {batch} sequences, mixed {mixed}", flush=True)
    alone = [run(cfg) for cfg in cfgs]
    torch.cuda.synchronize()
    bad = []

    def worker(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(8):
                    if not torch.equal(run(cfgs[k]), alone[k]):
                        bad.append(k)
        except Exception as e:                                  # noqa: BLE001  (shown by the assertion below)
            bad.append(repr(e))

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
