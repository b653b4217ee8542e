"""GPU parity of chunked_prefill_attention (through the C ABI) against the fp64 oracle.

Same bar as decode: max abs error 1.5e-2 with bf16 KV, 3e-2 with fp8 e4m3 KV
(bf16 output; the fp32 output to the same bar).  Small cases are compared
row by row in full; the benchmark workloads at full size on every row of their
first chunk and on sampled rows of the others, which the oracle computes one
by one.  Causality, untouched rows and determinism are
checked bit for bit.
"""
import sys

import numpy as np
import pytest
import torch

import workloads
from oracle import prefill

pytestmark = pytest.mark.gpu

TOL = {"bf16": 1.5e-2, "fp8_e4m3": 3e-2}


def note(msg):
    print(f"[gpu-test] {msg}", flush=True)
    sys.stdout.flush()


def oracle_rows(w, rows=None):
    return prefill.chunked_prefill_attention(w.q_bits, w.k_store, w.v_store, w.block_tables, w.context_lens,
                                             w.meta["q_start"], w.scale, kv_format=w.kv_format, k_scale=w.k_scale,
                                             v_scale=w.v_scale, rows=rows)


def gpu_rows(lib, w, dev=None, out_fp32=False, query_tile=0, out=None):
    d = dev if dev is not None else workloads.to_device(w)
    total_q = int(w.meta["q_start"][-1])
    shape = lib.prefill_shape(w.batch, w.n_q_heads, w.n_kv_heads, w.max_blocks_per_seq,
                              max(w.max_context_len, 0), w.num_blocks, total_q,
                              kv_fp8=w.kv_format == "fp8_e4m3", out_fp32=out_fp32, query_tile=query_tile)
    if out is None:
        out = torch.full((total_q, w.n_q_heads, 128), float("nan"), device="cuda",
                         dtype=torch.float32 if out_fp32 else torch.bfloat16)
    lib.chunked_prefill_attention(d["q"], d["k"][0], d["v"][0], d["block_tables"], d["context_lens"], d["q_start"],
                                  w.scale, out, shape, d["k_scale"], d["v_scale"])
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


SMALL = [
    # (chunks [(n, T)], Hq, Hkv, kv)
    ([(100, 300), (64, 64), (33, 1000), (17, 17)], 8, 2, "bf16"),
    ([(1, 40), (1, 129), (1, 1), (1, 500)], 16, 2, "bf16"),          # one-token chunks: decode
    ([(130, 130), (77, 205), (5, 37)], 4, 4, "bf16"),                # G = 1
    ([(96, 300), (31, 31), (200, 700)], 32, 2, "fp8_e4m3"),          # G = 16
    ([(64, 96), (40, 40)], 12, 2, "bf16"),                           # G = 6: columns that cross tokens
]


@pytest.mark.parametrize("case", range(len(SMALL)))
@pytest.mark.parametrize("query_tile", [0, 32])
def test_small_parity(gpu_lib, case, query_tile):
    chunks, hq, hkv, kv = SMALL[case]
    note(f"prefill small case {case} tile {query_tile}: {chunks} {hq}/{hkv} {kv}")
    w = workloads.make_prefill(chunks, hq, hkv, c_max=1024, kv_format=kv, seed=10 + case)
    ref = oracle_rows(w)
    dev = workloads.to_device(w)
    got = gpu_rows(gpu_lib, w, dev, query_tile=query_tile)
    err = float(np.abs(got - ref).max())
    note(f"  max abs err {err:.3e}")
    assert np.isfinite(got).all() and err <= TOL[kv]
    got32 = gpu_rows(gpu_lib, w, dev, out_fp32=True, query_tile=query_tile)
    assert float(np.abs(got32 - ref).max()) <= TOL[kv]


@pytest.mark.parametrize("name", sorted(workloads.PREFILL_CONFIGS))
def test_benchmark_workload(gpu_lib, name):
    """The benchmark workloads at full size: every row of the first chunk (2,048
    query tokens at context 2,048), and sampled rows of the deeper chunks, which
    the oracle computes one by one exactly as in full."""
    note(f"prefill {name}: building")
    w = workloads.make_prefill_config(name)
    qs = w.meta["q_start"]
    rng = np.random.default_rng(99)
    rows = set(range(int(qs[0]), int(qs[1])))
    for s in range(1, w.batch):
        r0, r1 = int(qs[s]), int(qs[s + 1])
        rows.update({r0, r0 + 1, r0 + 63, r0 + 64, r1 - 1})
        rows.update(int(x) for x in rng.integers(r0, r1, 6))
    rows = sorted(rows)
    dev = workloads.to_device(w)
    got = gpu_rows(gpu_lib, w, dev)
    del dev
    torch.cuda.empty_cache()
    note(f"prefill {name}: oracle on {len(rows)} rows")
    ref = oracle_rows(w, rows)
    err = float(np.abs(got[rows] - ref[rows]).max())
    note(f"prefill {name}: max abs err {err:.3e}")
    assert np.isfinite(got).all() and err <= TOL[w.kv_format]


def test_rows_of_other_sequences_and_empty_chunks_untouched(gpu_lib):
    w = workloads.make_prefill([(40, 90), (0, 50), (25, 25)], 8, 2, c_max=256, seed=21)
    dev = workloads.to_device(w)
    total_q = int(w.meta["q_start"][-1])
    out = torch.full((total_q + 8, 8, 128), 7.0, device="cuda", dtype=torch.bfloat16)   # 8 rows past the end
    got = gpu_rows(gpu_lib, w, dev, out=out)
    assert (got[total_q:] == 7.0).all()
    ref = oracle_rows(w)
    assert float(np.abs(got[:total_q] - ref).max()) <= TOL["bf16"]


def test_future_tokens_never_reach_earlier_rows(gpu_lib):
    w = workloads.make_prefill([(150, 400)], 8, 2, c_max=512, seed=22)
    dev = workloads.to_device(w)
    base = gpu_rows(gpu_lib, w, dev)
    T = int(w.context_lens[0])
    blk, slot = int(w.block_tables[0][(T - 1) // 16]), (T - 1) % 16
    dev["k"][0, blk, :, slot, :] = 0
    dev["v"][0, blk, :, :, slot] = int(np.uint16(0x447A).view(np.int16))   # 1000.0 in bf16
    got = gpu_rows(gpu_lib, w, dev)
    np.testing.assert_array_equal(got[:149], base[:149])
    assert np.abs(got[149] - base[149]).max() > 1.0


def test_random_chunks_every_row(gpu_lib):
    """Forty seeded random prefill shapes (cache format, GQA group 1-16 including
    groups whose items end inside a token's heads, 1-4 KV heads, 1-5 chunks of
    1-1,500 context tokens each, fresh prompts and chunks over a cached
    prefix, both query tiles, bf16 and fp32 output), every row against the
    oracle; a second call must equal the first bit for bit."""
    rng = np.random.default_rng(2605)
    for case in range(40):
        kv = ["bf16", "fp8_e4m3"][int(rng.integers(0, 2))]
        G = int(rng.choice([1, 2, 4, 6, 8, 12, 16]))
        Hkv = int(rng.choice([1, 2, 4]))
        chunks = []
        for _ in range(int(rng.integers(1, 6))):
            T = int(rng.integers(1, 1500))
            chunks.append((int(rng.integers(1, T + 1)) if rng.random() < 0.7 else T, T))
        qt = int(rng.choice([0, 32]))
        seed = int(rng.integers(0, 1 << 30))
        note(f"case {case}: kv={kv} G={G} Hkv={Hkv} chunks={chunks} tile={qt} seed={seed}")
        w = workloads.make_prefill(chunks, G * Hkv, Hkv, c_max=1536, kv_format=kv, seed=seed)
        dev = workloads.to_device(w)
        got = gpu_rows(gpu_lib, w, dev, query_tile=qt, out_fp32=bool(case % 2))
        assert np.array_equal(gpu_rows(gpu_lib, w, dev, query_tile=qt, out_fp32=bool(case % 2)), got)
        err = float(np.abs(got - oracle_rows(w)).max())
        assert np.isfinite(got).all() and err <= TOL[kv], f"case {case}: max abs err {err:.3e}"


def test_deterministic(gpu_lib):
    w = workloads.make_prefill_config("chunked_prefill_llama70b")
    dev = workloads.to_device(w)
    a = gpu_rows(gpu_lib, w, dev)
    b = gpu_rows(gpu_lib, w, dev)
    np.testing.assert_array_equal(a, b)


def test_longest_context(gpu_lib):
    """A chunk at the end of a 65,536-token context (the longest the kernel stages
    block ids for), with a ragged last query tile; sampled rows against the oracle."""
    note("prefill at context 65536")
    w = workloads.make_prefill([(77, 65536), (40, 1000)], 16, 2, c_max=65536, seed=23)
    qs = w.meta["q_start"]
    rows = sorted({0, 1, 31, 32, 63, 64, 76, int(qs[1]), int(qs[2]) - 1})
    got = gpu_rows(gpu_lib, w)
    ref = oracle_rows(w, rows)
    err = float(np.abs(got[rows] - ref[rows]).max())
    note(f"  max abs err {err:.3e}")
    assert np.isfinite(got).all() and err <= TOL["bf16"]


def plan(chunks, hq, hkv, c_max, cus):
    """The library's variant (waves, column blocks of a wave, waves that share a
    column's context) for a call, its items, its workgroups and its rounds, by
    the same arithmetic: a change of the rule shows in the tests that name what
    they reach."""
    def up(a, b):
        return -(-a // b)
    G, total, batch = hq // hkv, sum(n for n, _ in chunks), len(chunks)
    per_seq = up(total * G, batch)

    def full(c):
        return up(total * G, c) * hkv

    def items(c):
        return up(per_seq, c) * batch * hkv
    if full(256) >= cus:
        v, most = (8, 2, 1), cus
    elif full(128) > cus:
        v, most = (4, 2, 1), 2 * cus
    elif c_max > 2048 and full(64) <= cus and (per_seq <= 64 or items(64) <= cus):
        v, most = (8, 1, 2), cus
    elif c_max > 2048 and (per_seq <= 64 or items(128) <= cus):
        v, most = (8, 2, 2), cus
    elif c_max <= 2048 and (per_seq <= 64 or items(64) <= 2 * cus):
        v, most = (4, 1, 1), 2 * cus
    else:
        v, most = (4, 2, 1), 2 * cus
    cols = 16 * v[0] * v[1] // v[2]
    count = sum(up(n * G, cols) for n, _ in chunks) * hkv
    grid = min((up(total * G, cols) + batch) * hkv, most)
    return v, count, grid, up(count, grid)


ROUNDS = [
    # (chunks, Hq, Hkv, C_max, variant, items, rounds): one round of every item, then partial second
    # (backward) and third (forward) rounds, on every variant
    ([(2048, 2048), (2200, 4096)], 8, 2, 4096, (4, 2, 1), 266, 1),
    ([(3000, 3000), (1500, 2000)], 8, 4, 4096, (4, 2, 1), 284, 1),
    ([(1400, 1400), (1500, 2000)], 32, 4, 4096, (8, 2, 1), 364, 2),
    ([(2048, 2048), (2200, 4096)], 32, 4, 4096, (8, 2, 1), 532, 3),
    ([(10, 20 + s) for s in range(200)], 32, 4, 512, (4, 2, 1), 800, 2),
    ([(1 + s % 2 * 132, 133 + s) for s in range(60)], 15, 15, 512, (4, 2, 1), 1350, 3),
    ([(1 + s % 8, 20 + s) for s in range(200)], 32, 4, 512, (4, 1, 1), 800, 2),
    ([(1 + s % 8, 20 + s) for s in range(60)], 20, 20, 512, (4, 1, 1), 1200, 3),
    ([(1 + s % 8, 20 + s) for s in range(100)], 32, 4, 4096, (8, 1, 2), 400, 2),
    ([(1 + s % 8, 20 + s) for s in range(60)], 20, 10, 4096, (8, 1, 2), 600, 3),
    ([(1, 20 + s) for s in range(12)] + [(31, 400 + s) for s in range(12)], 64, 8, 4096, (8, 2, 2), 288, 2),
    # more rounds than are looked up at once, up to 64 sequences and more
    ([(1, 1 + s % 40) for s in range(64)], 261, 261, 4096, (8, 2, 1), 16704, 66),
    ([(1, 1 + s % 16) for s in range(2000)], 17, 17, 512, (4, 2, 1), 34000, 67),
]


@pytest.mark.parametrize("case", range(len(ROUNDS)))
def test_item_rounds_with_a_partial_last_round(gpu_lib, case):
    """More items than workgroups, not a multiple of them: every row is written
    (the output starts as NaN) and sampled rows match the oracle."""
    chunks, hq, hkv, c_max, variant, items, rounds = ROUNDS[case]
    note(f"prefill rounds case {case}: {len(chunks)} chunks {hq}/{hkv} C_max {c_max}")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus == 256:
        v, count, grid, r = plan(chunks, hq, hkv, c_max, cus)
        assert (v, count, r) == (variant, items, rounds) and (rounds == 1 or count % grid != 0)
    w = workloads.make_prefill(chunks, hq, hkv, c_max=c_max, seed=29)
    qs = w.meta["q_start"]
    total_q = int(qs[-1])
    rows = sorted(set(range(0, total_q, max(97, total_q // 20))) | {total_q - 1, int(qs[1]) - 1, int(qs[1])})
    got = gpu_rows(gpu_lib, w)
    ref = oracle_rows(w, rows)
    err = float(np.abs(got[rows] - ref[rows]).max())
    note(f"  max abs err {err:.3e}")
    assert np.isfinite(got).all() and err <= TOL["bf16"]


def _edges(qs):
    """First, last and 16-row boundary rows of every chunk."""
    rows = set()
    for a, b in zip(qs[:-1], qs[1:]):
        rows |= {int(r) for r in (a, b - 1, a + 15, a + 16, (a + b) // 2) if a <= r < b}
    return sorted(rows)


@pytest.mark.parametrize("chunks,hq,hkv,kv,variant", [
    # items of 64 columns: one-column remainders, contexts at the ends of 32-token tiles
    ([(1, 1), (16, 16), (17, 33), (8, 64), (15, 95), (31, 96), (33, 97)], 8, 2, "bf16", (4, 1, 1)),
    ([(3, 31), (4, 32), (5, 33), (9, 160)], 16, 1, "fp8_e4m3", (4, 1, 1)),
    # 64 columns, two waves on halves of the context: odd and even tile counts, chunks that end in either half
    ([(7, 2100), (33, 2049), (40, 40), (1, 33), (2, 64), (3, 65)], 16, 2, "bf16", (8, 1, 2)),
    ([(7, 2100), (33, 2081), (16, 32), (17, 97)], 16, 1, "fp8_e4m3", (8, 1, 2)),
    # 128 columns, the same
    ([(7, 2100), (133, 2049), (90, 90), (1, 33), (92, 124), (153, 165)], 64, 8, "bf16", (8, 2, 2)),
    ([(27, 2100), (33, 2081), (66, 82), (57, 97), (40, 64)], 96, 16, "fp8_e4m3", (8, 2, 2)),
    # 128 columns, four waves: GQA 4 and 5 (columns that cross tokens)
    ([(700, 700), (333, 500), (301, 301)], 32, 8, "bf16", (4, 2, 1)),
    ([(701, 800), (333, 333), (1, 1)], 40, 8, "fp8_e4m3", (4, 2, 1)),
    # 256 columns: GQA 5, a remainder of one token
    ([(1001, 1333), (97, 97), (1, 700)], 60, 12, "bf16", (8, 2, 1)),
    # the largest batch, and on the split context: 155 KiB of LDS, the most a launch takes
    ([(1, 1 + s % 16) for s in range(4096)], 18, 9, "bf16", (8, 2, 1)),
    ([(7, 2100)] + [(1, 1 + s % 16) for s in range(4095)], 3, 1, "bf16", (8, 1, 2)),
    ([(7, 2100)] + [(1, 1 + s % 16) for s in range(4095)], 5, 5, "bf16", (8, 2, 2)),
])
def test_item_widths(gpu_lib, chunks, hq, hkv, kv, variant):
    """Each width of work item the library chooses between, at the ends of its
    tiles and columns; every row is written, edge rows match the oracle."""
    note(f"prefill widths {len(chunks)} chunks {hq}/{hkv} {kv}")
    c_max = max(t for _, t in chunks)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus != 256 or plan(chunks, hq, hkv, c_max, cus)[0] == variant
    w = workloads.make_prefill(chunks, hq, hkv, c_max=c_max, kv_format=kv, seed=31)
    rows = _edges(w.meta["q_start"])
    rows = rows[:: max(1, len(rows) // 60)]
    got = gpu_rows(gpu_lib, w)
    ref = oracle_rows(w, rows)
    err = float(np.abs(got[rows] - ref[rows]).max())
    note(f"  max abs err {err:.3e}")
    assert np.isfinite(got).all() and err <= TOL[kv]


@pytest.mark.parametrize("n,T,hq,hkv,kv", [
    (256, 300, 4, 4, "bf16"),         # items of 64 columns
    (256, 2300, 4, 4, "bf16"),        # the same, the context split between two waves
    (256, 2300, 66, 66, "bf16"),      # of 128, the context split
    (256, 2331, 6, 2, "fp8_e4m3"),    # of 64, split, columns that cross tokens
    (600, 650, 64, 64, "bf16"),       # of 128 to four waves
    (1000, 1011, 64, 64, "fp8_e4m3"), # of 256
])
def test_non_finite_value_reaches_no_further_than_its_tile(gpu_lib, n, T, hq, hkv, kv):
    """A masked probability is 0, and 0 times a value that is not finite is not
    0: a column may meet such values up to the end of the 32-token tile that
    the last of the up to 32 tokens it shares a wave with lies in, and no
    further, however many tokens its work item has.  Earlier rows keep their
    bits; the token's own row shows it."""
    note(f"non-finite value: {n} tokens at {T}, {hq}/{hkv} {kv}")
    w = workloads.make_prefill([(n, T)], hq, hkv, c_max=T, kv_format=kv, seed=37)
    dev = workloads.to_device(w)
    base = gpu_rows(gpu_lib, w, dev)
    assert np.isfinite(base).all()
    for t in (T - 1, T - 40):
        blk, slot = int(w.block_tables[0][t // 16]), t % 16
        keep = dev["v"][0, blk, :, :, slot].clone()
        dev["v"][0, blk, :, :, slot] = 0x7F if kv == "fp8_e4m3" else 0x7FC0
        got = gpu_rows(gpu_lib, w, dev)
        dev["v"][0, blk, :, :, slot] = keep
        clean = 32 * (t // 32) - 31 - (T - n)  # rows before it
        assert clean > 0
        np.testing.assert_array_equal(got[:clean], base[:clean])
        assert np.isnan(got[t - (T - n)]).all()


@pytest.mark.parametrize("chunks,hq,hkv,kv", [
    ([(300, 1900), (33, 64), (70, 70), (1, 33)], 8, 2, "bf16"),
    ([(130, 1501), (40, 40), (5, 2000)], 16, 1, "fp8_e4m3"),
    ([(300, 1900)], 64, 8, "bf16"),
])
def test_split_context_rounds_alike(gpu_lib, chunks, hq, hkv, kv):
    """With a max_context_len above 2,048 two waves share a column's context.
    Both start from the maximum of the first 32 tokens, so probabilities are
    rounded as without the split and the outputs differ by the order of 32-bit
    sums only: one addition per 32-token tile (at most 63) and some 64 further
    units of 2^-24 from exponentials, weights and the division, of values below
    8."""
    note(f"split context: {chunks} {hq}/{hkv} {kv}")
    w = workloads.make_prefill(chunks, hq, hkv, c_max=4096, kv_format=kv, seed=41)
    dev = workloads.to_device(w)
    total_q = int(w.meta["q_start"][-1])
    outs = []
    for longest in (2048, 4096):
        shape = gpu_lib.prefill_shape(w.batch, hq, hkv, w.max_blocks_per_seq, longest, w.num_blocks, total_q,
                                      kv_fp8=kv == "fp8_e4m3", out_fp32=True)
        out = torch.full((total_q, hq, 128), float("nan"), device="cuda")
        gpu_lib.chunked_prefill_attention(dev["q"], dev["k"][0], dev["v"][0], dev["block_tables"],
                                          dev["context_lens"], dev["q_start"], w.scale, out, shape, dev["k_scale"],
                                          dev["v_scale"])
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy())
    assert np.isfinite(outs[0]).all()
    err = float(np.abs(outs[0] - outs[1]).max())
    note(f"  max difference {err:.3e}")
    assert err <= 128 * 2.0 ** -24 * 8.0
