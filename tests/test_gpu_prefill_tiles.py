"""Prefill at the edges of its tiles: query counts around a wave's tile and a work-group's group (32 // g and
4 * (32 // g) tokens), contexts around page pairs, the rings of pairs in flight and the 64 pairs (2048 tokens) whose
addresses are worked out at a time, against the oracle.  Bars as for all prefill tests (bf16 2e-3, e4m3 2e-2)."""
import numpy as np
import pytest

from parity import TOL, row_rel_err
from test_gpu_prefill import BF16, E4M3, Twin, gpu  # noqa: F401  (fixture)
from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g,hkv,d,dtype", [(1, 2, 128, BF16), (3, 1, 64, BF16), (4, 2, 128, E4M3), (5, 1, 128, BF16), (7, 2, 64, E4M3),
                                           (8, 1, 128, BF16), (16, 1, 64, BF16), (16, 1, 128, E4M3)])
@pytest.mark.parametrize("long", [False, True])
def test_prefill_tile_edges(gpu, oracle, g, hkv, d, dtype, long):  # noqa: F811
    tile = 32 // g
    if long:        # few queries in front of long contexts: parts of the context, more than one window of addresses
        cases = [(2048, 1), (2049, tile), (2081, tile + 1), (2300, 3)]
    else:
        cases = [(1, 1), (16, min(16, tile)), (31, min(31, tile + 1)), (33, 2), (64, min(64, 4 * tile)), (4 * tile + 65, 4 * tile + 1),
                 (97, 5), (129, 97), (161, 160), (200, 0), (5, 5)]
    ctx, qlen = [c for c, _ in cases], [q for _, q in cases]
    t = Twin(gpu, oracle, g * hkv, hkv, d, dtype, ctx, max_blocks=160)
    q = gen.queries((31, d, g), sum(qlen), g * hkv, d)
    rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
    rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
    assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
    assert row_rel_err(out_g, out_o) <= TOL[dtype]
    t.close()


@pytest.mark.parametrize("n,dtype", [(127, BF16), (128, E4M3), (131, BF16), (260, E4M3), (447, BF16), (448, E4M3), (900, BF16)])
def test_chunk_of_many_sequences(gpu, oracle, n, dtype):  # noqa: F811
    """Around 127 and 447 sequences, what the two plans of a launch hold: a chunk of 0 to 3 tokens for each is appended,
    then attends."""
    hq, hkv, d = 4, 1, 64
    ctx = [3 + (5 * s) % 37 for s in range(n)]
    qlen = [(s * 7 + 3) % 4 for s in range(n)]
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=8)
    g = gen.generator(37, n)
    k, v = (gen.randn_bf16((sum(qlen), hkv, d), g) for _ in range(2))
    for be, m in zip(t.be, t.models):
        assert be.kv_append_chunk(m, k, v, qlen, ctx) == sum(qlen)
    q = gen.queries((41, n), sum(qlen), hq, d)
    rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
    rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
    assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
    assert row_rel_err(out_g, out_o) <= TOL[dtype]
    t.close()


@pytest.mark.parametrize("dtype", [BF16, E4M3])
@pytest.mark.parametrize("score", [-1e6, -1e20, -1e29, -1e33, -2e37, 1e6, 1e20, 2e37])
def test_prefill_of_extreme_scores(gpu, oracle, dtype, score):  # noqa: F811
    """Every visible score far from zero, every fifth one (the first token among them) equal to the row's maximum and the
    others far below that: a row is the mean of the V it gives weight to, as for any other level of the scores.  Fresh
    prompts, and few queries in front of a context that is cut into parts."""
    hq, hkv, d = 8, 2, 64
    cases = [(70, 70), (33, 2), (1, 1), (1500, 3), (2100, 1)]
    ctx, qlen = [c for c, _ in cases], [n for _, n in cases]
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=160)
    try:
        size = np.float32(np.sqrt(abs(score) * 8))      # q and k of this size: |q k| / sqrt(64) = |score|
        for s, c in enumerate(ctx):
            kv = gen.seq_kv((13, s), c, hkv, d, dtype, 16)
            level = np.where(np.arange(c) % 5 == 0, -1.0, -2.0) if score < 0 else np.where(np.arange(c) % 5 == 0, 2.0, 1.0)
            if dtype == BF16:
                k = np.zeros((c, hkv, d), dtype=np.float32)
                k[:, :, 0] = level[:, None] * size
                kv["k"] = (k.view(np.uint32) >> 16).astype(np.uint16)
            else:
                kv["k"] = np.zeros((c, hkv, d), dtype=np.uint8)
                kv["k"][:, :, 0] = np.where(abs(level) == 1.0, 0x38, 0x40)[:, None] + (0x80 if score < 0 else 0)
                kv["k_scale"] = np.full_like(kv["k_scale"], size)
            for be, m in zip(t.be, t.models):
                assert be.kv_write(m, s, 0, kv["k"], kv["v"], kv["k_scale"], kv["v_scale"]) == c
        q = np.zeros((sum(qlen), hq, d), dtype=np.float32)
        q[:, :, 0] = size
        q = (q.view(np.uint32) >> 16).astype(np.uint16)
        rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
        rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
        assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
        assert row_rel_err(out_g, out_o) <= TOL[dtype]
        # the last query of every chunk is a decode step
        last = np.cumsum(qlen) - 1
        rc_g, out_g = gpu.decode_attention(t.models[0], q[last], t.ctx)
        assert rc_g == 0 and row_rel_err(out_g, out_o[last]) <= TOL[dtype]
    finally:
        t.close()


@pytest.mark.parametrize("dtype", [BF16, E4M3])
@pytest.mark.parametrize("step", [2.5, 2.75, 2.8125, 5.5, 5.75, 90.0])
def test_scores_that_climb_a_stair(gpu, oracle, dtype, step):  # noqa: F811
    """Every page pair's logits lie `step` above the one before, around the sum (256 for a lane's sixteen tokens: 2^4 each)
    and the level (2^8) at which the reference point of a column's exponentials moves; a fall back to zero after five pairs."""
    hq, hkv, d = 4, 2, 128
    cases = [(700, 9), (33, 33), (2100, 2)]
    ctx, qlen = [c for c, _ in cases], [n for _, n in cases]
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=160)
    try:
        for s, c in enumerate(ctx):
            kv = gen.seq_kv((17, s), c, hkv, d, dtype, 16)
            level = (np.arange(c) // 32 % 6 * step).astype(np.float32)
            if dtype == BF16:
                k = np.zeros((c, hkv, d), dtype=np.float32)
                k[:, :, 0] = level[:, None]
                kv["k"] = (k.view(np.uint32) >> 16).astype(np.uint16)
            else:
                kv["k"] = np.zeros((c, hkv, d), dtype=np.uint8)
                kv["k"][:, :, 0] = 0x38
                kv["k_scale"] = np.maximum(np.repeat(level[::16, None], hkv, axis=1), 1e-3).astype(np.float32)
            for be, m in zip(t.be, t.models):
                assert be.kv_write(m, s, 0, kv["k"], kv["v"], kv["k_scale"], kv["v_scale"]) == c
        q = np.zeros((sum(qlen), hq, d), dtype=np.float32)
        q[:, :, 0] = np.float32(np.sqrt(d))
        q = (q.view(np.uint32) >> 16).astype(np.uint16)
        rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
        rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
        assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
        assert row_rel_err(out_g, out_o) <= TOL[dtype]
    finally:
        t.close()


@pytest.mark.parametrize("n,dtype", [(130, BF16), (460, BF16), (460, E4M3)])
def test_cuts_among_many_sequences(gpu, oracle, n, dtype):  # noqa: F811
    """A few sequences with contexts long enough to be cut, in every launch of the call, among many short ones."""
    hq, hkv, d = 2, 1, 64
    ctx = [2500 if s % 150 == 149 else (1800 if s == 3 else 1 + (7 * s) % 30) for s in range(n)]
    qlen = [1 + s % 2 if c > 100 else (s % 3 if c > 2 else 1) for s, c in enumerate(ctx)]
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=160)
    try:
        q = gen.queries((43, n), sum(qlen), hq, d)
        rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
        for _ in range(2):
            rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
            assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
            assert gpu.last_prefill_parts() > 1
            assert row_rel_err(out_g, out_o) <= TOL[dtype]
    finally:
        t.close()


@pytest.mark.parametrize("ctx,parts,d,dtype", [([3200], (9, 15), 128, BF16), ([4700], (9, 32), 64, E4M3), ([9000, 2300], (17, 32), 64, BF16),
                                               ([16640], (33, 64), 64, BF16), ([16640, 9000, 40], (33, 64), 64, E4M3), ([33000], (64, 64), 64, BF16)])
def test_contexts_in_many_parts(gpu, oracle, ctx, parts, d, dtype):  # noqa: F811
    """One to three queries in front of contexts cut into up to 64 parts: joined eight at a time, by 32 lanes that hold the
    maximum and the denominator of two parts each."""
    hq, hkv = 4, 1
    t = Twin(gpu, oracle, hq, hkv, d, dtype, ctx, max_blocks=2100)
    try:
        for qlen in ([1] * len(ctx), [3] * len(ctx)):
            q = gen.queries((71, sum(ctx)), sum(qlen), hq, d)
            rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
            rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
            assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
            assert parts[0] <= gpu.last_prefill_parts() <= parts[1]
            assert row_rel_err(out_g, out_o) <= TOL[dtype]
    finally:
        t.close()


@pytest.mark.parametrize("g,hkv,longest", [(4, 8, 256), (4, 8, 257), (7, 8, 120), (16, 5, 255)])
def test_short_walks_of_many_work_groups(gpu, oracle, g, hkv, longest):  # noqa: F811
    """e4m3, more than 512 work-groups whose walks are of at most eight pairs, or just of more: such a launch, in which waves meet
    more often, gives the same bits as launches of half of the sequences, in which they do not, and those of the oracle."""
    n = 520 // hkv + 4
    ctx = [max(1, longest - (37 * s) % longest) for s in range(n)]
    qlen = [min(c, 1 + (3 * s) % 8) for s, c in enumerate(ctx)]
    t = Twin(gpu, oracle, g * hkv, hkv, 128, E4M3, ctx, max_blocks=17, pool_bytes=128 << 20)
    try:
        q = gen.queries((83, g, longest), sum(qlen), g * hkv, 128)
        rc_o, out_o = oracle.prefill_attention(t.models[1], q, qlen, ctx)
        rc_g, out_g = gpu.prefill_attention(t.models[0], q, qlen, ctx)
        assert rc_o == 0 and rc_g == 0 and gpu.device_errors() == 0
        assert row_rel_err(out_g, out_o) <= TOL[E4M3]
        at = sum(qlen[:n // 2])
        for part, rows in ((qlen[:n // 2] + [0] * (n - n // 2), slice(0, at)), ([0] * (n // 2) + qlen[n // 2:], slice(at, None))):
            rc_g, out_h = gpu.prefill_attention(t.models[0], q[rows], part, ctx)
            assert rc_g == 0 and np.array_equal(out_h, out_g[rows])
    finally:
        t.close()
