"""Attention work units at every GQA group: how a wave finds its rows (member
positions in the unit, scalar or per-lane reads of the member list), blocks
of a run's end that opened after the plan was made (in this launch, or in an
earlier step of the same plan), one- and two-tile units that wait for their
own append.  36 steps with no round between them cross two block openings of
every trace; every output against the oracle at the parity bar."""
import math

import numpy as np
import pytest
import torch

from _parity import assert_attn_close, replay
from oracle.attention import decode_attention
from oracle.formats import e4m3fn_to_f64
from paper_2608_08020_amd.gambit import GambitError, Pool
from workload import Workload, tiny

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("g", [1, 2, 4, 8, 16])
def test_groups_and_growing_runs(g, kv_dtype):
    cfg = tiny(kv_dtype=kv_dtype, n_q_heads=2 * g, gens=(2, 6, 24), prompt_len=37, seg_hi=90, steps=36, interval=40,
               keep=12, n_parents=12)
    replay(Workload(cfg), check_pool_every_step=True, quantise_on_append=kv_dtype != "bf16")


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
def test_unit_lengths_at_the_edges_of_the_tile_loops(kv_dtype):
    """One unit per run (max_splits leaves no other cut): private contexts of
    1 to 9 tiles and around the 64-block id windows, whole and partial last
    tiles, and runs that four traces share (two row blocks of one fp8 wave),
    over steps that open blocks after the plan was made."""
    fp8 = kv_dtype != "bf16"
    Hq, Hkv, steps = 8, 1, 3
    private = [1, 15, 16, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 159, 160, 161, 191, 192, 193, 223, 224, 255,
               257, 1023, 1024, 1025, 1056, 1087, 1089, 2048, 2081]
    shared = [1, 2, 3, 4, 5, 7, 8, 9, 10, 11, 13, 63, 64, 65, 67, 129]  # whole blocks, then 1, 15, 17 or 40 tokens each
    T = len(private) + 4 * len(shared)
    p = Pool(num_blocks=1700, num_q_heads=Hq, num_kv_heads=Hkv, max_traces=T, max_blocks_per_trace=140, kv_dtype=kv_dtype,
             max_splits=2)
    rng = np.random.default_rng(7 + fp8)
    K, V = [None] * T, [None] * T

    def fill(t, pos0, n):
        if fp8:
            codes = rng.integers(0, 127, (2, n, Hkv, 128)) | (rng.integers(0, 2, (2, n, Hkv, 128)) << 7)
            started = [b for b in range(pos0, pos0 + n) if b % 16 == 0]
            sc = (2.0 ** rng.integers(-9, -7, (len(started), 2))).astype(np.float32)
            own = sc[np.arange(n) // 16]  # every write starts a block
            scales[t] = np.concatenate([scales[t], sc])
            p.kv_write(t, pos0, *[torch.from_numpy(c.astype(np.uint8)).to("cuda") for c in codes], sc if len(sc) else None)
            kv = [e4m3fn_to_f64(codes[w].astype(np.uint8)) * own[:, None, None, w].astype(np.float64) for w in (0, 1)]
        else:
            x = [torch.from_numpy(rng.standard_normal((n, Hkv, 128)).astype(np.float32)).to(torch.bfloat16) for _ in (0, 1)]
            p.kv_write(t, pos0, x[0].cuda(), x[1].cuda())
            kv = [a.double().numpy() for a in x]
        for C, a in ((K, kv[0]), (V, kv[1])):
            C[t] = a if C[t] is None else np.concatenate([C[t], a])

    scales = [np.ones((1, 2), np.float32) for _ in range(T)]
    p.kv_alloc(range(len(private)), private)
    for t, n in enumerate(private):
        fill(t, 0, n)
    for i, nb in enumerate(shared):
        t0 = len(private) + 4 * i
        p.kv_alloc([t0], [16 * nb])
        fill(t0, 0, 16 * nb)
        p.kv_fork([t0] * 3, [t0 + 1, t0 + 2, t0 + 3])
        for j, n in enumerate((1, 15, 17, 40)):
            if j:
                K[t0 + j], V[t0 + j], scales[t0 + j] = K[t0].copy(), V[t0].copy(), scales[t0].copy()
        for j, n in enumerate((1, 15, 17, 40)):
            p.kv_alloc([t0 + j], [n])
            fill(t0 + j, 16 * nb, n)
    ids = np.random.default_rng(1).permutation(T)
    for step in range(steps):
        q = torch.from_numpy(rng.standard_normal((T, Hq, 128)).astype(np.float32)).to(torch.bfloat16)
        x = [torch.from_numpy(rng.standard_normal((T, Hkv, 128)).astype(np.float32)).to(torch.bfloat16) for _ in (0, 1)]
        if fp8:  # codes in the append scale's units, or the landing block's
            codes = [rng.integers(0, 120, (T, Hkv, 128)).astype(np.uint8) for _ in (0, 1)]
            new = [torch.from_numpy(c).cuda() for c in codes]
        else:
            new = [a.cuda() for a in x]
        out = p.decode_attn(ids, q.cuda(), *new, out_dtype=torch.float32).cpu().numpy()
        for i, t in enumerate(ids):
            if fp8:
                if len(K[t]) % 16 == 0:
                    scales[t] = np.concatenate([scales[t], np.full((1, 2), 2.0 ** -6, np.float32)])
                kv = [e4m3fn_to_f64(codes[w][i:i + 1]) * float(scales[t][-1, w]) for w in (0, 1)]
            else:
                kv = [a[i:i + 1].double().numpy() for a in x]
            K[t], V[t] = np.concatenate([K[t], kv[0]]), np.concatenate([V[t], kv[1]])
            ref = decode_attention(q[i].double().numpy(), K[t], V[t], 1 / math.sqrt(128))
            assert_attn_close(out[i], ref, f"step {step}, trace {t} of {len(K[t])} tokens")
    p.pool_check()


def test_merge_of_one_to_many_partials():
    """Rows of 1 to 36 partials (a small launch cuts a context every 16 blocks)."""
    n = [256 * k + 1 + 37 * k % 200 for k in range(36)] + [5]
    T, Hq = len(n), 2
    p = Pool(num_blocks=sum(-(-x // 16) for x in n) + T, num_q_heads=Hq, num_kv_heads=1, max_traces=T, max_blocks_per_trace=640)
    rng = np.random.default_rng(3)
    p.kv_alloc(range(T), n)
    bf = lambda *shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(torch.bfloat16)  # noqa: E731
    kv = [(bf(x, 1, 128), bf(x, 1, 128)) for x in n]
    for t, (k, v) in enumerate(kv):
        p.kv_write(t, 0, k.cuda(), v.cuda())
    q, kn, vn = bf(T, Hq, 128), bf(T, 1, 128), bf(T, 1, 128)
    out = p.decode_attn(range(T), q.cuda(), kn.cuda(), vn.cuda(), out_dtype=torch.float32).cpu().numpy()
    assert p.plan_stats(range(T)).max_splits_used == 36
    for t, (k, v) in enumerate(kv):
        K, V = (torch.cat([a, b[t:t + 1]]).double().numpy() for a, b in ((k, kn), (v, vn)))
        assert_attn_close(out[t], decode_attention(q[t].double().numpy(), K, V, 1 / math.sqrt(128)), f"{len(K)} tokens")
    p.pool_check()


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3"])
@pytest.mark.parametrize("shared", [False, True])  # narrow units, or cooperative items
@pytest.mark.parametrize("entry", [0, 3])
@pytest.mark.parametrize("bad", ["outside", "none", "another"])
def test_a_table_entry_that_is_not_the_plans_is_reported(kv_dtype, shared, entry, bad):
    """The first blocks of a unit come with the unit; a device table that says
    otherwise still sets the error word, as it does for every later block."""
    T, Hq = (12, 16) if shared else (2, 4)
    p = Pool(num_blocks=64, num_q_heads=Hq, num_kv_heads=1, max_traces=T, max_blocks_per_trace=16, kv_dtype=kv_dtype)
    for c in (p.k_cache, p.v_cache):
        c.view(torch.uint8).zero_()
    p.kv_alloc([0], [112])
    if shared:
        p.kv_fork([0] * (T - 1), list(range(1, T)))
    ids = list(range(T)) if shared else [0]
    q = torch.zeros((len(ids), Hq, 128), dtype=torch.bfloat16, device="cuda")
    x = torch.zeros((len(ids), 1, 128), dtype=torch.bfloat16 if kv_dtype == "bf16" else torch.uint8, device="cuda")
    p.decode_attn(ids, q, x, x)
    p.pool_check()
    good = p.block_table[0, entry].clone()
    p.block_table[0, entry] = {"outside": 64 + 5, "none": -1, "another": int(good) + 9}[bad]
    p.decode_attn(ids, q, x, x)
    p.block_table[0, entry] = good
    with pytest.raises(GambitError) as e:
        p.pool_check()
    assert e.value.code == "DEVICE" and "error word" in str(e.value)
