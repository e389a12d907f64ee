"""Small decode launches (a work-group per row and kv head, or per part of one): rows at the edges of pages, pairs
and parts against the oracle, and a captured launch whose rows have outgrown the parts it was laid out with."""
import numpy as np
import pytest
import torch

from parity import TOL, row_rel_err
from test_gpu_prefill import BF16, E4M3, Twin, gpu  # noqa: F401  (fixture)
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g,hkv,d,dtype", [(1, 3, 128, BF16), (3, 2, 64, BF16), (4, 2, 128, E4M3), (5, 1, 64, E4M3), (8, 1, 128, BF16),
                                           (16, 1, 128, E4M3), (16, 2, 64, BF16)])
def test_small_launch_edges(gpu, oracle, g, hkv, d, dtype):  # noqa: F811
    ctx = [0, 1, 16, 17, 31, 33, 127, 129, 511, 512, 513, 528, 529, 1024, 1025, 2100]
    t = Twin(gpu, oracle, g * hkv, hkv, d, dtype, ctx, max_blocks=140)
    for n in (len(ctx), 5, 1):                       # all rows; short rows only; one empty row
        q = gen.queries((53, d, g, n), n, g * hkv, d)
        rc_o, out_o = oracle.decode_attention(t.models[1], q, np.array(ctx[:n], dtype=np.int32))
        for _ in range(2):                           # the arrival counters are ready again
            rc_g, out_g = gpu.decode_attention(t.models[0], q, np.array(ctx[:n], dtype=np.int32))
            assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
            assert row_rel_err(out_g, out_o) <= TOL[dtype]
    t.close()


def test_rows_outgrow_a_captured_launch(gpu, oracle):  # noqa: F811
    hq, hkv, d = 8, 2, 128
    last = [2300, 900, 40, 1500]
    t = Twin(gpu, oracle, hq, hkv, d, BF16, last, max_blocks=160, poison=False)
    m = t.models[0]
    gpu.seq_release_batch(m, np.arange(4, dtype=np.int32))
    assert gpu.seq_reserve_batch(m, [0, 1, 2, 3], [40] * 4) == 12
    q = gen.queries((59,), 4, hq, d)
    qd = torch.from_numpy(q.view(np.int16)).cuda()
    ctx = torch.tensor([40] * 4, dtype=torch.int32, device="cuda")
    out = torch.zeros((4, hq, d), dtype=torch.float32, device="cuda")
    kv = [gen.seq_kv((13, s), c, hkv, d, BF16, 16) for s, c in enumerate(last)]
    for s in range(4):
        assert gpu.kv_write(m, s, 0, kv[s]["k"][:40], kv[s]["v"][:40]) == 40
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        gpu.use_current_stream()
        graph.capture_begin()
        assert gpu.decode_attention_dev(m, qd, ctx, out) == 0
        graph.capture_end()
    torch.cuda.synchronize()
    gpu.use_current_stream()
    for step in ([40] * 4, [600, 560, 40, 513], last, [1100, 900, 7, 1025], last):
        assert gpu.seq_reserve_batch(m, [0, 1, 2, 3], step) >= 0
        for s in range(4):
            assert gpu.kv_write(m, s, 0, kv[s]["k"][:step[s]], kv[s]["v"][:step[s]]) == step[s]
        ctx.copy_(torch.tensor(step, dtype=torch.int32))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        rc_o, out_o = oracle.decode_attention(t.models[1], q, np.array(step, dtype=np.int32))
        assert rc_o == 0 and gpu.device_errors() == 0 and row_rel_err(out.cpu().numpy(), out_o) <= TOL[BF16]
    t.close()


@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 1, 64, BF16), (4, 1, 128, E4M3), (4, 1, 128, BF16), (2, 1, 64, E4M3)])
def test_long_walks_of_one_part(gpu, oracle, hq, hkv, d, dtype):  # noqa: F811
    """A launch captured with rows in one part: later rows are walked by four waves, and a wave looks up 33 page pairs first and
    then 32 at a time, so up to and past 33 and 65 pairs, a whole or half a pair or a token more or less."""
    pages = [263, 264, 265, 272, 273, 513, 520, 522]
    last = [16 * n - (s % 3) for s, n in enumerate(pages)]
    n = len(last)
    t = Twin(gpu, oracle, hq, hkv, d, dtype, last, max_blocks=540, poison=False)
    m = t.models[0]
    q = gen.queries((71, d), n, hq, d)
    qd = torch.from_numpy(q.view(np.int16)).cuda()
    ctx = torch.tensor(last, dtype=torch.int32, device="cuda")
    out = torch.zeros((n, hq, d), dtype=torch.float32, device="cuda")
    c = np.array(last, dtype=np.int32)
    rc_o, out_o = oracle.decode_attention(t.models[1], q, c)
    gpu.seq_release_batch(m, np.arange(n, dtype=np.int32))
    assert gpu.seq_reserve_batch(m, list(range(n)), [40] * n) == 3 * n
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        gpu.use_current_stream()
        graph.capture_begin()
        assert gpu.decode_attention_dev(m, qd, ctx, out) == 0
        graph.capture_end()
    torch.cuda.synchronize()
    gpu.use_current_stream()
    assert gpu.last_kernel_form() == 2 and gpu.last_launch_items() == n * hkv
    assert gpu.seq_reserve_batch(m, list(range(n)), last) >= 0
    for s in range(n):
        kv = gen.seq_kv((13, s), last[s], hkv, d, dtype, 16)
        assert gpu.kv_write(m, s, 0, kv["k"], kv["v"], kv.get("k_scale"), kv.get("v_scale")) == last[s]
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert rc_o == 0 and gpu.device_errors() == 0 and row_rel_err(out.cpu().numpy(), out_o) <= TOL[dtype]
    t.close()


@pytest.mark.parametrize("ctx", [[300], [64, 200, 128], [2100, 90]])
def test_tokens_of_logit_minus_infinity(gpu, oracle, ctx):  # noqa: F811
    """Keys of -inf in pages 2 to 5, 10, 11 and 64 to 95: those tokens weigh nothing, also where they are all that one wave of
    a work-group, or one part of a row, gets to see."""
    hq, hkv, d = 8, 2, 64
    t = Twin(gpu, oracle, hq, hkv, d, BF16, ctx, max_blocks=140)
    try:
        for s, c in enumerate(ctx):
            kv = gen.seq_kv((13, s), c, hkv, d, BF16, 16)
            page = np.arange(c) // 16
            kv["k"][((page >= 2) & (page < 6)) | (page == 10) | (page == 11) | ((page >= 64) & (page < 96)), :, 0] = 0xFF80
            for be, m in zip(t.be, t.models):
                assert be.kv_write(m, s, 0, kv["k"], kv["v"]) == c
        q = gen.queries((61,), len(ctx), hq, d)
        q[:, :, 0] = 0x3F80                              # a positive factor of the infinite element
        rc_o, out_o = oracle.decode_attention(t.models[1], q, np.array(ctx, dtype=np.int32))
        rc_g, out_g = gpu.decode_attention(t.models[0], q, np.array(ctx, dtype=np.int32))
        assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
        assert row_rel_err(out_g, out_o) <= TOL[BF16]
    finally:
        t.close()


@pytest.mark.parametrize("ctx,small", [([100] * 60 + [2000], True), ([256] * 30 + [4096], True), ([128] * 63 + [8192], False),
                                       ([8192] + [128] * 63, False), ([64] * 64 + [9600], False), ([16] * 300, True), ([16] * 500, False)])
def test_rows_of_unlike_length(gpu, oracle, ctx, small):  # noqa: F811
    """A few long rows among many short ones, and very many rows: whether such a launch is cut into parts of rows or goes to
    the forms that deal pages out evenly, no row waits for one work-group to walk a long context, and all rows are right."""
    hq, hkv, d = 8, 8, 64
    t = Twin(gpu, oracle, hq, hkv, d, BF16, ctx, max_blocks=640)
    try:
        q = gen.queries((67, len(ctx)), len(ctx), hq, d)
        c = np.array(ctx, dtype=np.int32)
        rc_o, out_o = oracle.decode_attention(t.models[1], q, c)
        for _ in range(2):
            rc_g, out_g = gpu.decode_attention(t.models[0], q, c)
            assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
            assert (gpu.last_kernel_form() == 2) == small
            assert row_rel_err(out_g, out_o) <= TOL[BF16]
    finally:
        t.close()


@pytest.mark.parametrize("hq,hkv,d,dtype,ctx", [(32, 8, 128, BF16, [50] * 60 + [2000]), (32, 8, 128, BF16, [50] * 30 + [4000]),
                                                (8, 2, 128, BF16, [16] * 100 + [6000]), (8, 1, 128, BF16, [39] * 120 + [11055]),
                                                (20, 4, 128, E4M3, [34] * 112 + [7904])])
def test_one_long_row_keeps_the_small_kernel(gpu, oracle, hq, hkv, d, dtype, ctx):  # noqa: F811
    """One long row among some 30 to 120 short ones: the ordinary forms, which join the pieces of a row one after the other, take
    1.2 to 1.8 times as long."""
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=700)
    try:
        q = gen.queries((73, len(ctx)), len(ctx), hq, d)
        c = np.array(ctx, dtype=np.int32)
        rc_o, out_o = oracle.decode_attention(t.models[1], q, c)
        rc_g, out_g = gpu.decode_attention(t.models[0], q, c)
        assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
        assert gpu.last_kernel_form() == 2
        assert row_rel_err(out_g, out_o) <= TOL[dtype]
    finally:
        t.close()


@pytest.mark.parametrize("hq,hkv,d,dtype,ctx,items", [(64, 8, 128, BF16, [1784] * 7, 224), (2, 1, 128, BF16, [6984] * 15, 210), (32, 8, 128, BF16, [1024] * 4 + [512] * 8, 192),
                                                      (32, 8, 128, BF16, [2048] * 4, 192), (16, 4, 128, BF16, [767] * 2, 16),
                                                      (16, 2, 128, BF16, [3689] + [23] * 15, 256)])
def test_parts_keep_a_cu_to_one_work_group(gpu, oracle, hq, hkv, d, dtype, ctx, items):  # noqa: F811
    """Parts of 24 pages where that makes no more than 256 work-groups, and longer ones where it would take some more: two
    work-groups on a CU take longer than the shorter parts save (a sixth of the first two launches)."""
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=512, pool_bytes=128 << 20)
    try:
        q = gen.queries((79, len(ctx)), len(ctx), hq, d)
        c = np.array(ctx, dtype=np.int32)
        rc_o, out_o = oracle.decode_attention(t.models[1], q, c)
        rc_g, out_g = gpu.decode_attention(t.models[0], q, c)
        assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
        assert gpu.last_kernel_form() == 2 and gpu.last_launch_items() == items
        assert row_rel_err(out_g, out_o) <= TOL[dtype]
    finally:
        t.close()
