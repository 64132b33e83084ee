"""GPU parity of every extend tile (256, 128 and 64 query rows per workgroup)
with what it can meet: bf16 and 8-bit stores, one launch and split key ranges,
1 to 8 query heads per KV head, windows, sinks and slots masked by a deferred
eviction.  Each case states the tile and whether the key range is split, and
the plan is asked first, so that a case that the planner sends elsewhere fails
instead of testing another kernel.  Sampled rows (the first and last of the
chunk, of the first, second and last query block) of the first and last KV
head against the float64 oracle, over the seeded inputs."""

import math

import numpy as np
import pytest

from oracle import extend as oex
from oracle import fp8 as of8
from paper_2602_22603_amd import workload as wl

pytestmark = pytest.mark.gpu
TOL = 5e-4
SCALES = (0.011, 0.0095)


@pytest.fixture(scope="module")
def sq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the plans below are those of 256 compute units")
    from paper_2602_22603_amd import sq as sqmod
    sqmod.lib()
    return sqmod


@pytest.fixture(autouse=True)
def _free_memory():
    yield
    import gc
    import torch
    gc.collect()
    if torch.cuda.is_available():
        torch.cuda.empty_cache()


def _check(sq, rows, split, hq, hkv, d, kv8, prefix, n, window=0, sinks=False, masks=False):
    import torch
    L, g = prefix + n, hq // hkv
    s = sq.Store(1, hq, hkv, d, L // 16 + 2, 1, L // 16 + 2, device="cuda", kv_scales=[SCALES] if kv8 else None)
    a = s.seq_create()
    k, v = (wl.device_normal_bf16((1, L, hkv, d), 1000 * prefix + 2 * n + i, "cuda") for i in (0, 1))
    keep = np.ones(L, dtype=np.uint8)
    s.append(a, k[:, :prefix].contiguous(), v[:, :prefix].contiguous())
    if masks:
        spans = [(x, x + 37) for x in range(11, prefix - 60, prefix // 9)] + [(prefix - 16, prefix)]
        for c, (x, y) in enumerate(spans):
            s.span_mark(a, c, x, y)
            keep[x:y] = 0
        s.evict(a, list(range(len(spans))), deferred=True)
    s.append(a, k[:, prefix:].contiguous(), v[:, prefix:].contiguous())
    plan = s.extend_plan_info(a, n, window=window)
    assert (plan["rows"], plan["n_split"] > 1) == (rows, split), plan
    q = wl.device_normal_bf16((n, hq, d), 7 * n, "cuda")
    sk = torch.randn(hq, generator=torch.Generator().manual_seed(n)) if sinks else None
    out = s.extend(0, a, q, window=window, sinks=None if sk is None else sk.to("cuda"))
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    s.close()
    assert np.all(np.isfinite(got))
    qf = wl.torch_bf16_to_f64(q)
    tq = rows // g
    last_block = (n - 1) // tq * tq
    js = sorted({j for j in (0, tq - 1, tq, 2 * tq - 1, last_block, n // 2, n - 1) if 0 <= j < n})
    err = 0.0
    for kv in sorted({0, hkv - 1}):
        kf, vf = (wl.torch_bf16_to_f64(x[0, :, kv:kv + 1]) for x in (k, v))
        if kv8:
            kf, vf = of8.roundtrip(kf, SCALES[0]), of8.roundtrip(vf, SCALES[1])
        hs = slice(kv * g, kv * g + g)
        for j in js:
            end = prefix + j + 1
            ref = oex.extend_attention(qf[j:j + 1, hs], kf[:end], vf[:end], 1 / math.sqrt(d), g,
                                       mask=keep[:end], window=window,
                                       sinks=None if sk is None else sk[hs].double().numpy())
            err = max(err, float(np.max(np.abs(got[j, hs] - ref[0]))))
    print(f"extend {plan} hq={hq} hkv={hkv} d={d} kv8={kv8} prefix={prefix} n={n}: {err:.2e}")
    assert err <= TOL


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("prefix,short", [(16000, 0), (20000, 1), (30000, 0)])
@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_extend_64_row_tile(sq, g, prefix, short, kv8):
    """Chunks that fill a 64-row tile exactly, or all but its last token, over
    4, 5 and 8 key blocks per split (the tile alternates two block buffers)."""
    _check(sq, 64, True, 8 * g, 8, 128, kv8, prefix, 64 // g - short)


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("split,hq,hkv,d,prefix,n", [
    (False, 32, 8, 128, 100, 3000), (False, 64, 8, 128, 700, 1200), (True, 32, 8, 128, 3000, 512),
    (True, 16, 8, 128, 3000, 512), (True, 8, 8, 128, 100, 2400), (True, 64, 8, 128, 3000, 512),
    (False, 32, 8, 64, 100, 3000), (False, 64, 8, 64, 700, 1200), (True, 32, 8, 64, 3000, 512),
    (True, 16, 8, 64, 3000, 512), (True, 8, 8, 64, 100, 2400), (True, 64, 8, 64, 3000, 512),
    (True, 8, 1, 128, 300, 1999)])
def test_extend_256_row_tile(sq, split, hq, hkv, d, prefix, n, kv8):
    _check(sq, 256, split, hq, hkv, d, kv8, prefix, n)


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("split,hq,hkv,d,prefix,n,kw", [
    (False, 64, 8, 64, 300, 1999, dict(window=128)), (False, 64, 8, 128, 300, 1999, dict(window=128)),
    (False, 64, 8, 128, 300, 1999, dict(window=700, sinks=True)),
    (False, 64, 8, 64, 300, 1999, dict(sinks=True)), (False, 32, 8, 128, 100, 3000, dict(sinks=True)),
    (True, 16, 8, 128, 2000, 900, dict(sinks=True)), (True, 32, 8, 64, 3000, 512, dict(sinks=True)),
    (True, 32, 8, 128, 3000, 512, dict(masks=True)), (False, 64, 8, 64, 2000, 900, dict(masks=True)),
    (False, 64, 8, 128, 2000, 900, dict(masks=True, sinks=True)), (True, 16, 8, 64, 3000, 512, dict(masks=True))])
def test_extend_256_row_tile_options(sq, split, hq, hkv, d, prefix, n, kw, kv8):
    _check(sq, 256, split, hq, hkv, d, kv8, prefix, n, **kw)


@pytest.mark.parametrize("kv8", [False, True])
@pytest.mark.parametrize("split,hq,hkv,d,prefix,n,kw", [
    (True, 8, 1, 128, 227, 4140, {}), (True, 4, 2, 64, 40, 5484, {}), (True, 16, 8, 128, 364, 882, dict(sinks=True)),
    (True, 32, 8, 128, 60547, 77, {}), (True, 8, 8, 128, 8000, 64, dict(masks=True)),
    (False, 16, 2, 128, 93, 2805, {}), (False, 32, 8, 64, 100, 300, dict(window=50, sinks=True))])
def test_extend_128_row_tile(sq, split, hq, hkv, d, prefix, n, kw, kv8):
    """Three and five splits of long chunks over short prefixes, the splits of a
    short chunk late in a task, and one launch."""
    _check(sq, 128, split, hq, hkv, d, kv8, prefix, n, **kw)
