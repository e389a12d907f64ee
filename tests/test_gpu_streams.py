"""The library enqueues on the caller's stream: a side stream, and a captured HIP graph that is
replayed several times with eager work in between (every replay must equal the eager result)."""
import numpy as np
import pytest
import torch

from workloads.scenarios import Runner, make_config

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from paper_2505_04021_amd import PrismKV
    return PrismKV()


def setup(gpu):
    cfg = make_config(2, "small")
    r = Runner(gpu, cfg).setup()
    mids = r.active_models()
    qs = [torch.from_numpy(r.queries(0, mi).view(np.int16)).cuda() for mi in mids]
    ctxs = [torch.from_numpy(r.ctx[mi]).cuda() for mi in mids]
    outs = [torch.zeros((cfg.models[mi].batch, cfg.models[mi].q_heads, cfg.models[mi].head_dim), dtype=torch.float32, device="cuda")
            for mi in mids]
    return r, [r.models[mi] for mi in mids], qs, ctxs, outs


def test_side_stream(gpu):
    r, models, qs, ctxs, outs = setup(gpu)
    assert gpu.decode_attention_multi_dev(models, qs, ctxs, outs) == 0
    torch.cuda.synchronize()
    want = [o.clone() for o in outs]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        gpu.use_current_stream()
        for o in outs:
            o.zero_()
        assert gpu.decode_attention_multi_dev(models, qs, ctxs, outs) == 0
    side.synchronize()
    gpu.use_current_stream()
    for a, b in zip(outs, want):
        assert torch.equal(a, b)
    assert gpu.device_errors() == 0
    r.teardown()


def test_graph_replays_equal_eager(gpu):
    """The very first attention call on freshly registered models is the captured one: the library
    sized its workspaces at registration, so the capture meets no allocation and no wait."""
    r, models, qs, ctxs, outs = setup(gpu)
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        gpu.use_current_stream()
        graph.capture_begin()
        rc = gpu.decode_attention_multi_dev(models, qs, ctxs, outs)
        graph.capture_end()
    gpu.use_current_stream()
    assert rc == 0
    want = [torch.empty_like(o) for o in outs]
    assert gpu.decode_attention_multi_dev(models, qs, ctxs, want) == 0        # the eager result
    torch.cuda.synchronize()
    for rep in range(4):
        for o in outs:
            o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(outs, want):
            assert torch.equal(a, b), rep
        # eager work of the library between the replays, on new queries, then back
        q2 = [torch.roll(q, 1, dims=0) for q in qs]
        o2 = [torch.empty_like(o) for o in outs]
        assert gpu.decode_attention_multi_dev(models, q2, ctxs, o2) == 0
        torch.cuda.synchronize()
    assert gpu.device_errors() == 0
    r.teardown()


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
def test_neighbouring_tokens_written_on_two_streams(gpu, dtype, d):
    """Two streams write alternating runs of ten tokens of one sequence, so that most runs end inside a group of four tokens
    (one 16-byte unit of V) whose other tokens the other stream is writing: every token arrives, whichever call is first."""
    hkv, n, run = 4, 2000, 10
    pool = gpu.pool_create(16 << 20, 16, 2 << 20)
    m = gpu.model_register(pool, hkv, hkv, d, dtype, 1, 128)
    assert pool >= 0 and m >= 0 and gpu.balloon_resize(m, 8) == 8 and gpu.seq_reserve(m, 0, n) >= 0
    rng = np.random.RandomState(3)
    et, tt = (np.int16, torch.int16) if dtype == 0 else (np.uint8, torch.uint8)
    scale = torch.ones((n // 16 + 1, hkv), device="cuda")
    ends = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    sides = [torch.cuda.Stream(), torch.cuda.Stream()]
    for trial in range(4):
        want = [rng.randint(0, 120, (n, hkv, d)).astype(et) for _ in range(2)]
        k, v = (torch.from_numpy(x).to(device="cuda", dtype=tt) for x in want)
        torch.cuda.synchronize()
        for i, a in enumerate(range(0, n, run)):
            with torch.cuda.stream(sides[i & 1]):
                gpu.use_current_stream()
                if dtype == 0 and trial & 1 and i & 1:
                    rc = gpu.kv_append_chunk_dev(m, k[a:a + run], v[a:a + run], [run], ends[a + run:a + run + 1])
                else:
                    rc = gpu.lib.kv_write(m, 0, a, run, gpu._p(k[a:a + run]), gpu._p(v[a:a + run]),
                                          *((gpu._p(scale[a // 16:]),) * 2 if dtype else (None, None)))
                assert rc == run
        torch.cuda.synchronize()
        gpu.use_current_stream()
        rc, *got = gpu.kv_read(m, 0, 0, n)
        assert rc == n and gpu.device_errors() == 0
        for x, y in zip(want, got):
            assert np.array_equal(x, y.view(et))
    gpu.seq_release(m, 0)
    assert gpu.balloon_resize(m, 0) == 0 and gpu.model_unregister(m) == 0 and gpu.pool_destroy(pool) == 0
