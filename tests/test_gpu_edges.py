"""GPU edge cases through the C ABI: exhaustive fp8 codes, error paths that
must leave the pool unchanged, selection ties, determinism, fork vs copy,
plan splitting, empty calls."""
import math

import numpy as np
import pytest
import torch

from _parity import assert_attn_close
from oracle.attention import decode_attention
from oracle.formats import bf16_to_f64, e4m3fn_to_f64
from oracle.probe import rank
from paper_2608_08020_amd import gambit
from paper_2608_08020_amd.gambit import GambitError, Pool
from workload.generate import to_bf16_bits

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _bf16(x: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).to(DEV)


def test_all_fp8_codes_decode_exactly():
    codes = np.array([c for c in range(256) if c not in (0x7F, 0xFF)], np.uint8)
    T, Hkv, Hq = len(codes), 1, 1
    p = Pool(num_blocks=T + 8, num_q_heads=Hq, num_kv_heads=Hkv, max_traces=T,
             max_blocks_per_trace=2, kv_dtype="fp8_e4m3")
    ids = np.arange(T)
    p.kv_alloc(ids, np.ones(T))
    zeros = torch.zeros((1, Hkv, 128), dtype=torch.uint8, device=DEV)
    for t, c in enumerate(codes):
        v = torch.full((1, Hkv, 128), int(c), dtype=torch.uint8, device=DEV)
        p.kv_write(t, 0, zeros, v, np.array([[1.0, 1.0]], np.float32))
    q = torch.zeros((T, Hq, 128), dtype=torch.bfloat16, device=DEV)
    knew = torch.zeros((T, Hkv, 128), dtype=torch.uint8, device=DEV)
    out = p.decode_attn(ids, q, knew, knew, out_dtype=torch.float32)
    # both tokens score 0: o = (decode(code) + 0) / 2 exactly
    want = e4m3fn_to_f64(codes) / 2
    got = out[:, 0, :].cpu().numpy().astype(np.float64)
    assert (got == want[:, None]).all()
    p.pool_check()


def test_second_token_equals_mean_and_first_decode():
    """Two-token context with equal keys gives the mean of the two values."""
    p = Pool(num_blocks=8, num_q_heads=8, num_kv_heads=2, max_traces=2, max_blocks_per_trace=4)
    rng = np.random.default_rng(0)
    k0 = _bf16(np.ones((1, 2, 128)))
    v0 = _bf16(rng.standard_normal((1, 2, 128)))
    p.kv_alloc([0], [1])
    p.kv_write(0, 0, k0, v0)
    q = _bf16(rng.standard_normal((1, 8, 128)))
    v1 = _bf16(rng.standard_normal((1, 2, 128)))
    out = p.decode_attn([0], q, k0, v1, out_dtype=torch.float32).cpu().numpy()[0]
    want = (v0.float().cpu().numpy()[0] + v1.float().cpu().numpy()[0]) / 2
    for h in range(8):
        assert np.abs(out[h] - want[h // 4]).max() <= 1e-6


def test_errors_leave_pool_unchanged():
    p = Pool(num_blocks=6, num_q_heads=4, num_kv_heads=1, max_traces=4, max_blocks_per_trace=8)
    x = torch.zeros((40, 1, 128), dtype=torch.bfloat16, device=DEV)
    p.kv_alloc([0], [40])                                    # 3 blocks
    p.kv_write(0, 0, x, x)
    cases = [
        ("OUT_OF_BLOCKS", lambda: p.kv_alloc([1], [64])),
        ("INVALID", lambda: p.kv_alloc([0, 0], [1, 1])),
        ("INVALID", lambda: p.kv_alloc([9], [1])),
        ("INVALID", lambda: p.kv_alloc([1], [200])),         # exceeds max_blocks_per_trace
        ("INVALID", lambda: p.kv_write(0, 30, x[:20], x[:20])),
        ("INVALID", lambda: p.kv_fork([1], [2])),            # empty parent
        ("INVALID", lambda: p.kv_free([3])),                 # already empty
        ("INVALID", lambda: p.decode_attn([1], torch.zeros((1, 4, 128), dtype=torch.bfloat16, device=DEV),
                                          x[:1], x[:1])),    # empty trace
    ]
    for code, fn in cases:
        with pytest.raises(GambitError) as e:
            fn()
        assert e.value.code == code, (code, str(e.value))
        p.pool_check()
    p.kv_fork([0], [1])                                      # takes 1 block (tail of 8)
    with pytest.raises(GambitError) as e:
        p.kv_write(0, 0, x[:1], x[:1])
    assert e.value.code == "SHARED_WRITE"
    with pytest.raises(GambitError) as e:
        p.kv_fork([0], [1])
    assert e.value.code == "INVALID"
    p.kv_alloc([2], [32])                                    # the last 2 blocks
    with pytest.raises(GambitError) as e:
        p.kv_fork([0], [3])
    assert e.value.code == "OUT_OF_BLOCKS"
    with pytest.raises(GambitError) as e:
        p.score_prune_branch([0, 1, 2], torch.zeros((3, 64), dtype=torch.bfloat16, device=DEV),
                             torch.zeros(64, device=DEV), 0.0, 2, 2)   # 1 pruned over 2 parents
    assert e.value.code == "INVALID"
    p.pool_check()
    assert p.free_blocks() == 0


def test_rank_topk_ties_bit_exact():
    rng = np.random.default_rng(1)
    # sizes on both sides of the run-merge sort's limits (runs of 128, at most
    # 1024 keys; the bitonic network beyond), crafted ties
    for n, keep in [(7, 3), (512, 128), (1000, 999), (4096, 17), (33, 33), (1, 1), (64, 10), (128, 64),
                    (129, 1), (256, 256), (1024, 1024), (1025, 500), (2048, 2000)]:
        ids = rng.permutation(n * 3)[:n].astype(np.int32)
        scores = rng.choice(np.array([0.1, 0.5, 0.5000001, 0.9, -2.0], np.float32), size=n)
        got = gambit.rank_topk(torch.from_numpy(ids).to(DEV), torch.from_numpy(scores).to(DEV), keep)
        want = rank(ids, scores.astype(np.float64))[:keep]
        assert got.cpu().numpy().tolist() == want


def test_deterministic_bitwise():
    from paper_2608_08020_amd.runner import PopulationRun
    from workload import Workload, tiny

    outs = []
    for _ in range(2):
        wl = Workload(tiny())
        run = PopulationRun(wl)
        run.setup()
        run.load_steps(range(wl.total_steps))
        run.load_rounds(range(len(wl.rounds_after())))
        res = []
        for s, r in run.schedule():
            res.append(run.decode(s, out_dtype=torch.float32).cpu().numpy())
            if r is not None:
                res.append(np.concatenate([x.cpu().numpy().ravel().view(np.uint32) for x in run.round(r)[1:]]))
        res.append(run.pool.block_table.cpu().numpy())
        outs.append(res)
    for a, b in zip(*outs):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))


def test_fork_and_copy_agree():
    rng = np.random.default_rng(2)
    p = Pool(num_blocks=64, num_q_heads=8, num_kv_heads=2, max_traces=3, max_blocks_per_trace=16)
    k = _bf16(rng.standard_normal((71, 2, 128)))
    v = _bf16(rng.standard_normal((71, 2, 128)))
    p.kv_alloc([0], [71])
    p.kv_write(0, 0, k, v)
    p.kv_fork([0], [1])
    p.kv_alloc([2], [71])
    p.kv_write(2, 0, k.clone(), v.clone())
    q = _bf16(np.repeat(rng.standard_normal((1, 8, 128)), 3, axis=0))
    kn = _bf16(np.repeat(rng.standard_normal((1, 2, 128)), 3, axis=0))
    vn = _bf16(np.repeat(rng.standard_normal((1, 2, 128)), 3, axis=0))
    out = p.decode_attn([0, 1, 2], q, kn, vn, out_dtype=torch.float32).cpu().numpy()
    K = np.concatenate([bf16_to_f64(k.cpu().view(torch.int16).numpy().view(np.uint16)),
                        bf16_to_f64(kn[:1].cpu().view(torch.int16).numpy().view(np.uint16))])
    V = np.concatenate([bf16_to_f64(v.cpu().view(torch.int16).numpy().view(np.uint16)),
                        bf16_to_f64(vn[:1].cpu().view(torch.int16).numpy().view(np.uint16))])
    ref = decode_attention(bf16_to_f64(q[0].cpu().view(torch.int16).numpy().view(np.uint16)), K, V,
                           1 / math.sqrt(128))
    for t in range(3):
        assert_attn_close(out[t], ref, f"fork/copy trace {t}")
    tab = p.block_table.cpu().numpy()
    assert (tab[1, :4] == tab[0, :4]).all() and tab[1, 4] != tab[0, 4]
    p.pool_check()


def test_split_limit_grows_chunks_or_reports():
    rng = np.random.default_rng(3)
    p = Pool(num_blocks=600, num_q_heads=4, num_kv_heads=1, max_traces=2, max_blocks_per_trace=300,
             max_splits=1)
    L = 4000
    k = _bf16(rng.standard_normal((L, 1, 128)))
    v = _bf16(rng.standard_normal((L, 1, 128)))
    p.kv_alloc([0], [L])
    p.kv_write(0, 0, k, v)
    q = _bf16(rng.standard_normal((1, 4, 128)))
    kn = _bf16(rng.standard_normal((1, 1, 128)))
    out = p.decode_attn([0], q, kn, kn, out_dtype=torch.float32).cpu().numpy()[0]
    assert p.plan_stats([0]).max_splits_used == 1
    K = np.concatenate([k.float().cpu().numpy(), kn.float().cpu().numpy()]).astype(np.float64)
    V = np.concatenate([v.float().cpu().numpy(), kn.float().cpu().numpy()]).astype(np.float64)
    ref = decode_attention(q[0].float().cpu().numpy().astype(np.float64), K, V, 1 / math.sqrt(128))
    assert_attn_close(out, ref, "one partial per trace")
    # after a fork every trace has a shared run and a private run: two partials
    p.kv_fork([0], [1])
    with pytest.raises(GambitError) as e:
        p.decode_attn([0, 1], q.repeat(2, 1, 1), kn.repeat(2, 1, 1), kn.repeat(2, 1, 1))
    assert e.value.code == "UNSUPPORTED"
    p.pool_check()


def test_empty_calls_are_no_ops():
    p = Pool(num_blocks=4, num_q_heads=4, num_kv_heads=1, max_traces=2, max_blocks_per_trace=2)
    z = torch.zeros((0, 4, 128), dtype=torch.bfloat16, device=DEV)
    p.kv_alloc([], [])
    p.kv_free([])
    p.kv_fork([], [])
    p.decode_attn([], z, z[:, :1], z[:, :1])
    p.pool_check()
    assert p.free_blocks() == 4


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_many_blocks_opened_in_one_step(kv_dtype):
    """A decode step whose appends open more blocks than its launch carries
    (the allocator kernel runs first) and steps that open fewer (the attention
    launch claims them), with the trace list out of id order and freed blocks
    interleaved with used ones: tables, refcounts, lengths, scales and
    attention as the pool model gives them."""
    from oracle.pool import PoolModel

    fp8 = kv_dtype == "fp8_e4m3"
    T, Hq, Hkv = 300, 4, 1
    rng = np.random.default_rng(11)
    p = Pool(num_blocks=1200, num_q_heads=Hq, num_kv_heads=Hkv, max_traces=T, max_blocks_per_trace=4,
             kv_dtype=kv_dtype)
    om = PoolModel(num_blocks=1200, n_kv_heads=Hkv, head_dim=128, kv_dtype=kv_dtype, max_traces=T,
                   max_blocks_per_trace=4)

    def codes(n):
        if fp8:
            c = rng.integers(0, 256, size=(n, Hkv, 128)).astype(np.uint8)
            c[(c & 0x7F) == 0x7F] = 0x38  # no NaN codes
            return c
        return to_bf16_bits(rng.standard_normal((n, Hkv, 128)).astype(np.float32))

    def bf16_dev(c):
        return torch.from_numpy(c.view(np.int16)).view(torch.bfloat16).to(DEV)

    def dev(c):
        return torch.from_numpy(c).to(DEV) if fp8 else bf16_dev(c)

    def fill(t, L):
        p.kv_alloc([t], [L])
        om.alloc([t], [L])
        k, v = codes(L), codes(L)
        sc = np.full(((L + 15) // 16, 2), 0.5 + t / T, np.float32) if fp8 else None
        p.kv_write(t, 0, dev(k), dev(v), sc)
        om.write(t, 0, k, v, sc)

    for t in range(T):
        fill(t, 16 if t < 270 else 7)

    def step(ids):
        n = len(ids)
        q = to_bf16_bits(rng.standard_normal((n, Hq, 128)).astype(np.float32))
        kn, vn = codes(n), codes(n)
        out = p.decode_attn(ids, bf16_dev(q), dev(kn), dev(vn), out_dtype=torch.float32).cpu().numpy()
        om.append(ids, kn, vn)
        for i in list(range(0, n, 37)) + [n - 1]:
            K, V = om.materialise(int(ids[i]))
            ref = decode_attention(bf16_to_f64(q[i]), K, V, 1 / math.sqrt(128))
            assert_attn_close(out[i], ref, f"trace {ids[i]} (list position {i})")
        assert p.seq_len.cpu().numpy().tolist() == om.seq_len
        assert np.array_equal(p.block_table.cpu().numpy(), om.table_array())
        assert p.refcount.cpu().numpy().tolist() == om.refcount
        if fp8:
            sc = p.kv_scale.cpu().numpy()
            for t in ids:
                assert [tuple(sc[b]) for b in om.table[t]] == om.bscale[t], t
        p.pool_check()

    step(rng.permutation(T))        # 270 blocks opened: more than one launch carries
    step(rng.permutation(T))        # none opened
    for t in range(0, 200, 2):      # frees 100 traces' blocks between used ones
        p.kv_free([t])
        om.free_traces([t])
    for t in range(0, 200, 2):
        fill(t, 32)
    step(rng.permutation(T))        # 100 opened, claimed by the attention launch
    step(rng.permutation(T)[:150])  # a partial list


@pytest.mark.parametrize("opening", [256, 257])
def test_launch_argument_capacity_boundary(opening):
    """Exactly as many new blocks as one launch carries (256: claimed by the
    attention launch) and one more (257: the allocator kernel runs first)."""
    from oracle.pool import PoolModel

    T, Hq, Hkv = 300, 4, 1
    rng = np.random.default_rng(12 + opening)
    p = Pool(num_blocks=800, num_q_heads=Hq, num_kv_heads=Hkv, max_traces=T, max_blocks_per_trace=3)
    om = PoolModel(num_blocks=800, n_kv_heads=Hkv, head_dim=128, kv_dtype="bf16", max_traces=T,
                   max_blocks_per_trace=3)
    for t in range(T):
        L = 16 if t < opening else 9
        kv = to_bf16_bits(rng.standard_normal((L, Hkv, 128)).astype(np.float32))
        dev = torch.from_numpy(kv.view(np.int16)).view(torch.bfloat16).to(DEV)
        p.kv_alloc([t], [L])
        p.kv_write(t, 0, dev, dev)
        om.alloc([t], [L])
        om.write(t, 0, kv, kv)
    ids = rng.permutation(T)
    q = to_bf16_bits(rng.standard_normal((T, Hq, 128)).astype(np.float32))
    kn = to_bf16_bits(rng.standard_normal((T, Hkv, 128)).astype(np.float32))
    bf = lambda a: torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).to(DEV)  # noqa: E731
    out = p.decode_attn(ids, bf(q), bf(kn), bf(kn), out_dtype=torch.float32).cpu().numpy()
    om.append(ids, kn, kn)
    assert np.array_equal(p.block_table.cpu().numpy(), om.table_array())
    assert p.seq_len.cpu().numpy().tolist() == om.seq_len
    for i in (0, 99, T - 1):
        K, V = om.materialise(int(ids[i]))
        ref = decode_attention(bf16_to_f64(q[i]), K, V, 1 / math.sqrt(128))
        assert_attn_close(out[i], ref, f"trace {ids[i]} (list position {i})")
    p.pool_check()


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("hkv,layers", [(1, 1), (2, 3), (8, 2)])
def test_write_places_every_element_and_nothing_else(kv_dtype, hkv, layers):
    """Runs that start and end inside blocks, K and V at any element address:
    every element at its place in the tiles, every other byte as it was."""
    fp8 = kv_dtype == "fp8_e4m3"
    nb, es = 12, 1 if fp8 else 2
    p = Pool(num_blocks=nb, num_q_heads=4 * hkv, num_kv_heads=hkv, max_traces=2, max_blocks_per_trace=8,
             kv_dtype=kv_dtype, num_layers=layers)
    p.kv_alloc([1], [7])      # the run's blocks are not the pool's first
    p.kv_alloc([0], [128])
    for c in (p.k_cache, p.v_cache):
        c.view(torch.uint8).fill_(0xA5)
    blocks = p.block_table.cpu().numpy()[0]
    want = np.full((2, layers, nb, hkv, 16 * 128 * es), 0xA5, np.uint8)
    # tile offsets of element d of token row r: K [d / C][row with bits 2 and 3 swapped][d % C], V [d][r]
    C = 16 // es
    r, d = np.meshgrid(np.arange(16), np.arange(128), indexing="ij")
    phys = (r & 3) | ((r >> 1) & 4) | ((r << 1) & 8)
    place = [(d // C * 16 + phys) * C + d % C, d * 16 + r]
    rng = np.random.default_rng(hkv)
    for pos0, n, off in [(0, 1, 0), (0, 16, 1), (5, 7, 3), (13, 20, 0), (31, 1, 1), (32, 1, 0), (40, 56, 5), (97, 31, 0)]:
        raw = rng.integers(0, 256, (2, off + layers * n * hkv * 128, es), np.uint8)
        dev = torch.from_numpy(raw).to(DEV).view(torch.uint8 if fp8 else torch.bfloat16).view(2, -1)
        k, v = (x[off:].view(layers, n, hkv, 128) for x in dev)
        m = -(-(pos0 + n) // 16) - -(-pos0 // 16)
        p.kv_write(0, pos0, k, v, np.ones((layers, m, 2), np.float32) if fp8 and m else None)
        src = raw[:, off:].reshape(2, layers, n, hkv, 128, es)
        for w in (0, 1):
            tiles = want[w].reshape(layers, nb, hkv, 2048, es)
            for i in range(n):
                tiles[:, blocks[(pos0 + i) // 16]][:, :, place[w][(pos0 + i) % 16]] = src[w, :, i]
    got = [c.view(torch.uint8).cpu().numpy().reshape(want[0].shape) for c in (p.k_cache, p.v_cache)]
    for w in (0, 1):
        assert np.array_equal(got[w], want[w]), "KV"[w]
    p.pool_check()


@pytest.mark.parametrize("traces,blocks", [(3, 70), (40, 5000), (1024, 140000), (1500, 140000)])
def test_allocation_is_lowest_free_first(traces, blocks):
    """Long, short and empty requests over a fragmented free set: one and several
    requests per thread of the allocator, one and several passes over the bitmap."""
    rng = np.random.default_rng(traces)
    p = Pool(num_blocks=blocks, num_q_heads=4, num_kv_heads=1, max_traces=traces, max_blocks_per_trace=blocks // 2 + 64)
    free = np.ones(blocks, bool)
    rows, lens = [[] for _ in range(traces)], np.zeros(traces, np.int64)

    def alloc(ids, ntok):
        p.kv_alloc(ids, ntok)
        order = iter(np.flatnonzero(free))
        for t, n in zip(ids, ntok):
            got = [int(next(order)) for _ in range(-(-(lens[t] + n) // 16) - -(-lens[t] // 16))]
            rows[t] += got
            lens[t] += n
            free[got] = False

    def check():
        tab = p.block_table.cpu().numpy()
        for t in range(traces):
            assert tab[t, :len(rows[t])].tolist() == rows[t] and (tab[t, len(rows[t]):] == -1).all(), t
        assert (p.seq_len.cpu().numpy() == lens).all()
        assert ((p.refcount.cpu().numpy() > 0) == ~free).all()
        p.pool_check()

    ids = np.arange(traces)
    n = rng.integers(0, 3 * 16, traces) * (rng.random(traces) < 0.8)
    n[traces // 2] = 16 * (blocks // 3) + 5  # one long request among short ones
    alloc(ids, n)
    check()
    gone = [t for t in ids if lens[t] and (t % 2 or t == traces // 2)]
    p.kv_free(gone)
    for t in gone:
        free[rows[t]] = True
        rows[t], lens[t] = [], 0
    check()
    alloc(rng.permutation(traces), rng.integers(0, 5 * 16, traces))
    alloc([traces - 1], [16 * (blocks // 4) + 1])
    check()
