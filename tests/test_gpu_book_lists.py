"""Reserve and release lists at the edges of what the kernels hold at a time: lists that travel in the kernel's arguments
and longer ones (64 / 192 entries), more than 8192 blocks in one call, frames of many slots, sequences listed twice.
State and return values against the oracle, word for word."""
import numpy as np
import pytest

from workloads import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    from paper_2505_04021_amd import PrismKV
    return PrismKV()


@pytest.mark.parametrize("hkv,d,dtype,frames", [(1, 64, 1, 24), (2, 128, 0, 160)])       # 963 and 128 slots per frame
def test_lists(gpu, oracle, hkv, d, dtype, frames):
    both = []
    for be in (gpu, oracle):
        pool = be.pool_create((frames + 3) * (2 << 20), 16, 2 << 20)
        assert be.pool_seed_free_order(pool, gen.free_order(frames + 3, gen.generator(61))) == 0
        m = be.model_register(pool, 4 * hkv, hkv, d, dtype, 400, 12000)
        assert be.balloon_resize(m, frames) == frames
        both.append((be, pool, m))
    rng = np.random.RandomState(5)

    def step(name, *args):
        rc = [getattr(be, name)(m, *args) for be, _, m in both]
        assert rc[0] == rc[1], (name, rc)
        assert np.array_equal(*(be.pool_export_state(pool) for be, pool, _ in both)), name
        return rc[0]

    for n in (1, 2, 63, 64, 65, 200, 341, 700):
        seqs = rng.randint(0, 400, n).astype(np.int32)               # sequences repeat
        step("seq_reserve_batch", seqs, rng.randint(0, 60, n).astype(np.int32) * 16)
    for n in (1, 191, 192, 193, 390):
        step("seq_release_batch", rng.randint(0, 400, n).astype(np.int32))
        step("seq_reserve_batch", rng.permutation(400)[:120].astype(np.int32), rng.randint(1, 500, 120).astype(np.int32))
    assert step("seq_reserve_batch", [399], [9000 * 16]) > 8192      # one row, more than a window of ranks
    step("seq_release_batch", [399, 3, 399])
    assert step("seq_reserve_batch", list(range(300, 400)), [100 * 16] * 100) > 8192
    step("seq_release_batch", list(range(400)))
    for be, pool, m in both:
        assert be.balloon_resize(m, 0) == 0 and be.model_unregister(m) == 0 and be.pool_destroy(pool) == 0
