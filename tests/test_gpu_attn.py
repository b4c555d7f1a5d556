"""GPU parity, paged_decode_attn: within 2e-3 of the output's max norm of the CPU checker,
both reading the same quantized bytes (the checker's cache, uploaded)."""
import ctypes as C
import zlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_2605_29639_amd import workloads as W
from helpers import (attn_err, gpu_attention, gpu_fill, oracle_fill, upload_oracle_cache)

TOL = 2e-3   # max |gpu - oracle| <= TOL * max |oracle| over the call's whole output


def oracle_out(wl, oc, osc, seq_lens=None, q=None, q_len=None):
    return oracle.paged_decode_attn(wl.q if q is None else q, oc, osc, wl.mode, wl.block_tables,
                                    wl.seq_lens if seq_lens is None else seq_lens,
                                    wl.q_len if q_len is None else q_len, wl.sm_scale)


def check(wl, chunks=(0,), tol=TOL):
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    errs = []
    for chunk in chunks:
        got = gpu_attention(wl, cache, scales, desc, chunk_tokens=chunk)
        assert np.isfinite(got).all(), "non-finite output (chunk %d)" % chunk
        e = attn_err(got, want)
        errs.append(e)
        assert e <= tol, "chunk %d: err %.3e" % (chunk, e)
    return errs


MODES = [W.MODE_INT8, W.MODE_FP8, W.MODE_BF16, W.MODE_FP8_TENSOR, W.MODE_INT4, W.MODE_INT4_GROUP]


def skip_unsupported(mode, D):
    if mode in (W.MODE_INT4, W.MODE_INT4_GROUP) and D != 128:
        pytest.skip("int4 takes head_dim 128 only")


@pytest.mark.parametrize("mode", MODES)
def test_tiny_config(mode):
    skip_unsupported(mode, 64)
    check(W.tiny(mode), chunks=(0, 64))


CASES = [
    # name, seq_lens, q_len, Hq, Hkv, D, bs
    ("ragged16", [1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 700], 1, 4, 2, 64, 16),
    ("d128_g4", [130, 333, 64, 1000, 5], 1, 32, 8, 128, 16),
    ("g1", [100, 260], 1, 2, 2, 128, 16),
    ("g2", [100, 260], 1, 4, 2, 64, 16),
    ("g8", [90, 515], 1, 16, 2, 128, 16),
    ("g16_bs64", [300, 1029, 64, 2049], 1, 64, 4, 128, 64),
    ("bs32", [257, 33], 1, 8, 2, 64, 32),
    ("bs128", [513, 100], 1, 8, 2, 128, 128),
    ("qlen4_g8", [53, 20, 4, 300, 1025], 4, 16, 2, 128, 16),
    ("qlen4_g4", [260, 7], 4, 8, 2, 64, 16),
    ("qlen2_g16", [100, 400], 2, 32, 2, 128, 64),
    ("qlen3_g16_rowgroups", [100, 130], 3, 32, 2, 64, 16),
    ("qlen16_g4", [100, 16, 77], 16, 4, 1, 128, 16),
    ("bs256", [700, 300, 256], 1, 8, 2, 128, 256),
    ("g64_two_row_groups", [150, 90], 1, 64, 1, 64, 16),
    ("qlen16_g8_four_row_groups", [200, 40], 16, 8, 1, 128, 32),
    # a chunk of a prompt attending over the quantized prefix and itself (causal)
    ("chunk64", [200, 70], 64, 8, 2, 128, 16),
    ("chunk200_bs64", [700], 200, 4, 1, 64, 64),
    ("chunk256", [300, 1029], 256, 16, 2, 128, 16),
    ("chunk40_ragged_row_block", [300, 41], 40, 8, 2, 128, 16),       # 160 rows: 128 + 32
    ("prompt_from_an_empty_cache", [130, 130], 130, 4, 1, 128, 16),    # q_len = the whole sequence
    ("chunk512_bs64_d64", [600, 512], 512, 8, 2, 64, 64),
    ("chunk96_g2_bs256", [700, 300], 96, 4, 2, 128, 256),              # 192 rows, 256-token blocks
    ("chunk130_g1_bs32_d64", [257, 140], 130, 2, 2, 64, 32),           # 130 rows: 128 + 2
    ("chunk140_g2_eight_pairs", [300, 140, 200, 141], 140, 4, 2, 64, 16),  # 8 (seq, head) pairs x 3 row blocks
]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_shapes_and_splits(mode, case):
    name, lens, q_len, Hq, Hkv, D, bs = case
    skip_unsupported(mode, D)
    lens = [max(l, q_len) for l in lens]
    wl = W.custom(name, mode, lens, q_len, Hq, Hkv, D, bs, seed=zlib.crc32(name.encode()) % 1000 + mode)
    check(wl, chunks=(0, 64, 256))


def over_the_flat_list(wl, cache, scales, desc, **kw):
    """The call through the measurement build, kept on the flat list of groups and the reduce."""
    from paper_2605_29639_amd import kvq
    prof = kvq.prof_lib()
    prof.kvq_profile_prefill_kernel(0)
    try:
        return gpu_attention(wl, cache, scales, desc, chunk_tokens=0, L=prof, **kw)
    finally:
        prof.kvq_profile_prefill_kernel(1)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_small_shapes_over_the_flat_list(mode, case):
    """Calls this small mostly give each (sequence, kv head) a workgroup; the flat list and its reduce must
    give the same (the oracle's bound; the two differ by the order of sums and by where f16 is exact)."""
    name, lens, q_len, Hq, Hkv, D, bs = case
    skip_unsupported(mode, D)
    lens = [max(l, q_len) for l in lens]
    wl = W.custom(name, mode, lens, q_len, Hq, Hkv, D, bs, seed=zlib.crc32(name.encode()) % 1000 + mode)
    oc, osc = oracle_fill(wl)
    got = over_the_flat_list(wl, *upload_oracle_cache(wl, oc, osc))
    assert np.isfinite(got).all() and attn_err(got, oracle_out(wl, oc, osc)) <= TOL


@pytest.mark.parametrize("mode,D,G,q_len", [(m, 128, 4, 1) for m in MODES] + [(W.MODE_INT8, 64, 2, 3), (W.MODE_FP8, 64, 8, 4),
                                            (W.MODE_BF16, 64, 1, 1), (W.MODE_INT8, 128, 8, 4), (W.MODE_INT4, 128, 7, 3),
                                            (W.MODE_BF16, 128, 8, 3), (W.MODE_INT4_GROUP, 128, 8, 3), (W.MODE_FP8, 128, 5, 7),
                                            (W.MODE_INT8, 64, 8, 4), (W.MODE_BF16, 64, 8, 4), (W.MODE_FP8_TENSOR, 128, 8, 4)])
@pytest.mark.parametrize("seqs", [1, 40, 130])
def test_a_workgroup_for_each_pair(mode, D, G, q_len, seqs):
    """Contexts from one token to a few groups more than the workgroup has wavefronts, on and around the edges
    of groups (wavefronts without a group, with one, with one more than others); one and two row tiles, rows
    that fill neither, several row groups; up to one pair for each compute unit (whole workgroups)
    and up to two (half ones); against the oracle and the flat list."""
    import ctypes as C
    from paper_2605_29639_amd import kvq
    one_tile = G * q_len <= 16 or mode == W.MODE_INT4_GROUP
    pairs = 2 * seqs * -(-G * q_len // (16 if one_tile else 32))
    whole = 4 if mode == W.MODE_BF16 or (not one_tile and D == 128) else 8
    team = whole if pairs <= 256 else whole // 2
    span = team + (0 if mode == W.MODE_INT4_GROUP and pairs <= 256 else 2)   # (two groups in a row do not pay there)
    lens = [max(q_len, 64 * (i % span) + (0, 1, 63, 17)[i % 4], 1) for i in range(span - 1, span - 1 + seqs)]
    wl = W.custom("pairs", mode, lens, q_len, 2 * G, 2, D, 16, seed=seqs + G)
    oc, osc = oracle_fill(wl)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    waves = kvq.prof_lib().kvq_profile_pair_waves(C.byref(desc), seqs, q_len, 2 * G, max(lens), 0)
    assert waves == (team if pairs <= 512 else 0), (pairs, waves)
    got, want = gpu_attention(wl, cache, scales, desc, chunk_tokens=0), oracle_out(wl, oc, osc)
    assert np.isfinite(got).all() and attn_err(got, want) <= 5e-4
    assert attn_err(got, over_the_flat_list(wl, cache, scales, desc).astype(np.float64)) <= 5e-4


@pytest.mark.parametrize("mode", MODES)
def test_gpu_written_cache_gives_the_same_attention(mode):
    """End to end through both entry points: the library's own cache (bit-identical to the
    checker's, see test_gpu_write) and the uploaded checker's cache give the same output."""
    wl = W.custom("e2e", mode, [200, 77, 1030], 1, 8, 2, 128, 16, seed=12)
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    c1, s1, desc = gpu_fill(wl)
    c2, s2, _ = upload_oracle_cache(wl, oc, osc)
    a = gpu_attention(wl, c1, s1, desc)
    b = gpu_attention(wl, c2, s2, desc)
    assert np.array_equal(a, b)
    assert attn_err(a, want) <= TOL


@pytest.mark.parametrize("q_len", [1, 40])   # 40 tokens x 4 heads: the many-row kernel
@pytest.mark.parametrize("mode", MODES)
def test_stale_bytes_after_the_last_position_are_never_used(mode, q_len):
    """Unwritten slots hold NaN codes / NaN or huge scales; block-table entries past the last
    block are -1.  The output must not change and must stay finite."""
    import torch
    D = 128 if mode in (W.MODE_INT4, W.MODE_INT4_GROUP) else 64
    lens = [max(l, q_len) for l in (37, 100, 64, 3)]
    wl = W.custom("stale", mode, lens, q_len, 4 if q_len == 1 else 8, 2, D, 16, seed=8)
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    live = np.zeros(oc.shape[:1] + oc.shape[3:4], dtype=bool)       # [blk, off]
    for b in range(wl.batch):
        s = wl.slots(b, 0, int(wl.seq_lens[b]))
        live[s // 16, s % 16] = True
    dirty_c, dirty_s = oc.copy(), osc.copy()
    for blk, off in np.argwhere(~live):
        if mode == W.MODE_BF16:   # NaN and infinity bit patterns
            dirty_c[blk, :, :, off, :] = 0x7FC0 if (blk + off) % 2 else 0xFF80
        else:
            dirty_c[blk, :, :, off, :] = 0x80 if mode == W.MODE_INT8 else 0x7F
        if mode in (W.MODE_INT8, W.MODE_INT4, W.MODE_INT4_GROUP):
            dirty_s[blk, :, :, off] = np.nan if (blk + off) % 2 else 3e38
    if mode == W.MODE_FP8:
        dead_blocks = ~live.any(axis=1)
        dirty_s[dead_blocks] = np.nan
    cache, scales, desc = upload_oracle_cache(wl, dirty_c, dirty_s)
    for chunk in (0, 64):
        got = gpu_attention(wl, cache, scales, desc, chunk_tokens=chunk)
        assert np.isfinite(got).all()
        assert attn_err(got, want) <= TOL


def test_run_to_run_determinism():
    wl = W.custom("det", W.MODE_INT8, [900, 333], 1, 8, 2, 128, 16, seed=2)
    cache, scales, desc = gpu_fill(wl)
    a = gpu_attention(wl, cache, scales, desc, chunk_tokens=256)
    b = gpu_attention(wl, cache, scales, desc, chunk_tokens=256)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("mode", MODES[:3])  # (one static scale cannot span these magnitudes)
def test_degenerate_inputs(mode):
    """All-zero V rows carrying the largest weight, zero q, huge and tiny V magnitudes."""
    wl = W.custom("degenerate", mode, [80, 80, 80, 80], 1, 4, 2, 64, 16, seed=21, outliers=False)
    oc, osc = oracle.alloc_cache(mode, wl.num_blocks, 16, 2, 64)
    for b in range(4):
        k, v = wl.kv_rows(b, 0, 80)
        kf, vf = W.bf16_bits_to_f32(k), W.bf16_bits_to_f32(v)
        if b == 0:      # an "attention sink": strongest key, zero value
            kf[0, :] = W.bf16_bits_to_f32(wl.q[0]).reshape(2, 2, 64)[:, 0] * 3
            vf[0] = 0
        if b == 1:      # zero query
            wl.q[1] = 0
        if b == 2:      # V spans 40 binades across tokens
            vf *= (2.0 ** np.linspace(-20, 20, 80)).astype(np.float32)[:, None, None]
        if b == 3:      # everything tiny
            vf *= np.float32(2.0 ** -60)
            kf *= np.float32(2.0 ** -30)
        oracle.kv_quant_write(W.to_bf16_bits(kf), W.to_bf16_bits(vf), wl.slots(b, 0, 80), oc, osc,
                              mode)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    got = gpu_attention(wl, cache, scales, desc)
    assert np.isfinite(got).all()
    for b in range(4):   # per sequence, since their magnitudes differ by design
        assert attn_err(got[b], want[b]) <= TOL, b


def test_empty_batch():
    import torch
    from paper_2605_29639_amd import kvq
    desc = kvq.make_desc(0, 4, 16, 2, 64)
    cache, scales = kvq.alloc_cache(desc)
    q = torch.empty((0, 4, 64), dtype=torch.bfloat16, device="cuda")
    out = torch.empty((0, 4, 64), dtype=torch.float32, device="cuda")
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    kvq.paged_decode_attn(q, cache, scales, desc,
                          torch.empty((0, 4), dtype=torch.int32, device="cuda"),
                          torch.empty(0, dtype=torch.int32, device="cuda"), 1, 0, 0.125, out, ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("seed", range(16))
def test_random_shapes(seed):
    """Shapes nobody picked by hand: batch, lengths, group size, query tokens, block size, head
    size, cache mode and split granule all drawn from a seeded generator."""
    rng = np.random.default_rng(7000 + seed)
    D = int(rng.choice([64, 128]))
    modes = [m for m in MODES if not (m in (W.MODE_INT4, W.MODE_INT4_GROUP) and D != 128)]
    mode = int(rng.choice(modes))
    bs = int(rng.choice([16, 32, 64, 128]))
    Hkv = int(rng.choice([1, 2, 3]))
    G = int(rng.choice([1, 2, 4, 8, 16]))
    q_len = int(rng.choice([1, 1, 2, 3, 4, 8]))
    B = int(rng.integers(1, 10))
    lens = [int(rng.choice([rng.integers(q_len, 70), rng.integers(q_len, 1500),
                            64 * rng.integers(1, 9)])) for _ in range(B)]
    lens = [max(l, q_len) for l in lens]
    chunk = int(rng.choice([0, 64, 128, 512]))
    wl = W.custom("random%d" % seed, mode, lens, q_len, G * Hkv, Hkv, D, bs, seed=seed)
    check(wl, chunks=(chunk,))


@pytest.mark.parametrize("mode,q_len,prefix,batch,spread",
                         [(W.MODE_INT8, 1, 0, 3000, 200), (W.MODE_FP8, 1, 0, 1500, 200),
                          (W.MODE_INT8, 4, 0, 3000, 200), (W.MODE_BF16, 1, 0, 3000, 200),
                          (W.MODE_INT8, 2, 256, 2000, 100), (W.MODE_FP8, 4, 256, 1100, 64)])
def test_thousands_of_short_sequences(mode, q_len, prefix, batch, spread):
    """Far more (sequence, kv head) pairs than wavefronts: every range of the flat list crosses
    many pairs, most pairs lie inside one range and are written without a partial, and the
    per-sequence bookkeeping (lengths, prefix sums) runs over a batch many times the
    wavefront's width.  With a prefix: the same through the shared-prefix entry point."""
    rng = np.random.default_rng(900 + q_len)
    lo = max(q_len, prefix)
    lens = [int(x) for x in rng.integers(lo, lo + spread, size=batch)]
    lens[17] = lo              # the shortest allowed
    lens[batch - 1] = lo + 700  # and a long one at the very end of the list
    wl = W.custom("crowd", mode, lens, q_len, 4, 2, 128, 16, seed=77, shared_prefix=prefix)
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    for hint in ((0,) if prefix == 0 else (prefix, 64, 0)):
        got = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, shared_prefix_tokens=hint)
        assert np.isfinite(got).all()
        e = attn_err(got, want)
        assert e <= TOL, "shared_prefix_tokens %d: err %.3e" % (hint, e)


@pytest.mark.parametrize("mode,D", [(W.MODE_INT8, 128), (W.MODE_FP8, 64), (W.MODE_BF16, 128),
                                    (W.MODE_INT4_GROUP, 128)])
def test_the_largest_query_length(mode, D):
    """q_len at the library's limit (1024 query tokens per sequence): a whole prompt of exactly
    that length, and a chunk of that length over a shorter prefix."""
    wl = W.custom("longest_chunk", mode, [1024, 1500], 1024, 4, 2, D, 16, seed=31 + mode)
    check(wl)


@pytest.mark.parametrize("mode", MODES)
def test_many_query_rows_through_both_kernels(mode):
    """128 and more query rows per kv head take the kernel that shares the dequantization among
    128 rows; the streaming kernels must give the same answer (both within the bound of the
    checker, and close to each other)."""
    from paper_2605_29639_amd import kvq
    wl = W.custom("both", mode, [700, 129, 64], 64, 8, 2, 128, 16, seed=40 + mode)
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    shared = gpu_attention(wl, cache, scales, desc)
    prof = kvq.prof_lib()   # the measurement build can keep such calls on the streaming kernels
    prof.kvq_profile_prefill_kernel(0)
    try:
        streamed = gpu_attention(wl, cache, scales, desc, L=prof)
    finally:
        prof.kvq_profile_prefill_kernel(1)
    assert attn_err(shared, want) <= TOL and attn_err(streamed, want) <= TOL
    assert attn_err(shared, streamed.astype(np.float64)) <= 2e-4


PREFIX_LENS = {
    "ragged": [700, 256, 1500, 333, 257],       # one sequence is nothing but the prefix
    "one": [1000],                              # a single pair per kv head
    "many": [256 + 37 * (i % 9) for i in range(70)],   # more sequences than a wavefront has lanes
    "crowd": [256 + 29 * (i % 5) for i in range(260)],   # more pairs than get a workgroup each
}


@pytest.mark.parametrize("mode", [W.MODE_INT8, W.MODE_FP8, W.MODE_BF16, W.MODE_INT4])
@pytest.mark.parametrize("q_len", [1, 4])
@pytest.mark.parametrize("lens", sorted(PREFIX_LENS))
def test_shared_prefix_is_read_through_stacked_rows(mode, q_len, lens):
    """paged_decode_attn_prefix: sequences that begin with the same physical blocks.  The
    shared positions go through the many-row kernel with all sequences' rows stacked, the rest
    through the streaming kernel, and the reduce merges the two: the output stays within the
    bound of the checker and close to paged_decode_attn's (other order of the fp32 merges; the
    probabilities are rounded to 16 bits against a running maximum that depends on the order),
    with a prefix that is not a multiple of 64, with a sequence that is nothing but the prefix (its
    query rows then mask part of it) and with more sequences than a wavefront has lanes.  A prefix
    longer than the shortest sequence is dropped (on the host if it exceeds max_seq_len, else on the
    device), as is one below 64 tokens or with a single sequence: bit for bit paged_decode_attn's output
    then.  The ranges are given by chunk_tokens, which keeps the prefix; with the automatic split all
    these hints are dropped on the host (the next test has those that are not)."""
    import ctypes as C
    from paper_2605_29639_amd import kvq
    wl = W.custom("prefix", mode, PREFIX_LENS[lens], q_len, 8, 2, 128, 16,
                  seed=90 + mode + q_len, shared_prefix=256)
    assert (wl.block_tables[:, :16] == wl.block_tables[0, :16]).all()
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    shortest = min(PREFIX_LENS[lens])
    plan = (C.c_int64 * 8)()
    for chunk in (0, 128, 512):
        assert kvq.prof_lib().kvq_profile_plan(C.byref(desc), wl.batch, q_len, 8, wl.max_seq_len, chunk, 256, plan) == kvq.OK
        # (with the automatic split so short a prefix is not worth its kernel)
        assert (plan[3] == 4) == (chunk > 0 and lens != "one")
        plain = gpu_attention(wl, cache, scales, desc, chunk_tokens=chunk)
        assert attn_err(plain, want) <= TOL
        for hint in (256, 200, 64, 63, 4096) + ((shortest + 64,) if lens != "one" else ()):
            hinted = gpu_attention(wl, cache, scales, desc, chunk_tokens=chunk,
                                   shared_prefix_tokens=hint)
            used = chunk > 0 and 64 <= hint and hint // 64 * 64 <= shortest and len(PREFIX_LENS[lens]) > 1
            if not used:
                assert np.array_equal(hinted.view(np.uint32), plain.view(np.uint32)), hint
            else:
                assert attn_err(hinted, want) <= TOL, (chunk, hint)
                assert attn_err(hinted, plain.astype(np.float64)) <= 2e-4, (chunk, hint)


@pytest.mark.parametrize("mode,D", [(W.MODE_INT8, 128), (W.MODE_FP8, 128), (W.MODE_BF16, 128), (W.MODE_INT4, 128),
                                    (W.MODE_INT8, 64), (W.MODE_FP8_TENSOR, 64), (W.MODE_BF16, 64)])
def test_a_shared_prefix_is_used_where_it_is_worth_the_launch(mode, D):
    """260 sequences behind 2048 shared tokens keep the hint, in fewer pieces than there is room for; of
    16 sequences, or of 64 tokens, it is dropped on the host: bit for bit paged_decode_attn's output.  A hint that
    was kept is dropped on the device where one sequence is shorter than the prefix: the same results up to
    the order of the merges."""
    from paper_2605_29639_amd import kvq
    pieces = kvq.prof_lib().kvq_profile_prefix_pieces
    for batch, hint, used in ((260, 2048, True), (260, 2000, True), (260, 64, False), (16, 2048, False)):
        wl = W.custom("prefix_pays", mode, [2048 + 5 + 7 * (i % 9) for i in range(batch)], 2, 4, 2, D, 16,
                      seed=190 + mode, shared_prefix=2048)
        oc, osc = oracle_fill(wl)
        cache, scales, desc = upload_oracle_cache(wl, oc, osc)
        assert (pieces(C.byref(desc), batch, 2, 4, wl.max_seq_len, 0, hint) > 0) == used
        plain = gpu_attention(wl, cache, scales, desc)
        hinted = gpu_attention(wl, cache, scales, desc, shared_prefix_tokens=hint)
        if not used:
            assert np.array_equal(hinted.view(np.uint32), plain.view(np.uint32))
            continue
        assert attn_err(hinted, oracle_out(wl, oc, osc)) <= TOL
        assert attn_err(hinted, plain.astype(np.float64)) <= 2e-4
        short = wl.seq_lens.copy()
        short[3] = 700
        plain = gpu_attention(wl, cache, scales, desc, seq_lens=short, max_len=wl.max_seq_len)
        dropped = gpu_attention(wl, cache, scales, desc, seq_lens=short, max_len=wl.max_seq_len,
                                shared_prefix_tokens=hint)
        assert np.isfinite(dropped).all()
        assert attn_err(dropped, plain.astype(np.float64)) <= 2e-4


@pytest.mark.parametrize("mode,batch,hkv,q_len,longest,prefix,pieces,many", [
    (W.MODE_BF16, 91, 4, 3, 4199, 3840, 3, 1), (W.MODE_BF16, 80, 2, 5, 2200, 2048, 5, 1),
    (W.MODE_INT8, 120, 2, 5, 2200, 2048, 3, 0), (W.MODE_FP8, 300, 1, 3, 2200, 2048, 2, 0)])
def test_a_shared_prefix_under_33_to_64_rows(mode, batch, hkv, q_len, longest, prefix, pieces, many):
    """Two row groups of stacked rows, in calls that are the many-row kernel's without the hint and in streaming ones,
    against the oracle on a few sequences and the call without the hint on all."""
    from paper_2605_29639_amd import kvq
    hq = 16 * hkv if q_len == 3 else 8 * hkv
    lens = [longest - 3 * (i % 40) for i in range(batch)]
    wl = W.custom("prefix rows", mode, lens, q_len, hq, hkv, 128, 16, seed=230 + mode, shared_prefix=prefix)
    cache, scales, desc = gpu_fill(wl)
    prof, plan = kvq.prof_lib(), (C.c_int64 * 8)()
    assert prof.kvq_profile_plan(C.byref(desc), batch, q_len, hq, longest, 0, 0, plan) == kvq.OK and plan[0] == many
    assert prof.kvq_profile_prefix_pieces(C.byref(desc), batch, q_len, hq, longest, 0, prefix) == pieces
    hinted = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, shared_prefix_tokens=prefix)
    assert attn_err(hinted, gpu_attention(wl, cache, scales, desc, chunk_tokens=0).astype(np.float64)) <= 2e-4
    seqs = [0, 1, batch - 1]   # (the first one writes the prefix)
    oc, osc = oracle_fill(wl, sequences=seqs)
    rows = np.concatenate([np.arange(b * q_len, (b + 1) * q_len) for b in seqs])
    want = oracle.paged_decode_attn(np.ascontiguousarray(wl.q[rows]), oc, osc, mode,
                                    np.ascontiguousarray(wl.block_tables[seqs]),
                                    np.ascontiguousarray(wl.seq_lens[seqs]), q_len, wl.sm_scale)
    assert attn_err(hinted[rows], want) <= TOL


@pytest.mark.parametrize("mode,D", [(m, 128) for m in MODES if m != W.MODE_INT4_GROUP] +
                         [(W.MODE_INT8, 64), (W.MODE_FP8, 64)])
@pytest.mark.parametrize("lens,q_len", [([2000, 41, 700], 40), ([64, 65, 128, 1], 33), ([5000], 130),
                                        ([8191, 300], 64), ([64, 65, 128, 33, 2048, 129], 33)])
def test_many_query_rows_over_a_split_context(mode, D, lens, q_len):
    """Calls of the many-row kernel with too few row blocks to fill the chip walk the context in
    pieces that a second launch merges: beside contexts too short to cut, of lengths around a
    group's edge; pieces a row, or all of a row block, sees nothing of; row blocks that are not
    full.  (The list without a long context is not cut.)  The bound is the checker's; f16 probabilities give 1e-4 or less."""
    lens = [max(l, q_len) for l in lens]
    wl = W.custom("split", mode, lens, q_len, 8, 2, D, 16, seed=len(lens) + mode)
    errs = check(wl)
    assert max(errs) <= 5e-4


@pytest.mark.parametrize("mode,G,q_len", [(W.MODE_INT8, 8, 5), (W.MODE_INT8, 8, 8), (W.MODE_FP8, 4, 9), (W.MODE_INT4, 11, 3),
                                          (W.MODE_FP8_TENSOR, 6, 10)])
@pytest.mark.parametrize("longest", [2048, 2049])
def test_two_row_tiles_of_a_crowd_of_short_sequences(mode, G, q_len, longest):
    """33 to 64 query rows of a quantized cache: the many-row kernel with a workgroup for every slot of the
    chip and contexts of at most 2048 tokens, the streaming kernel one token further."""
    lens = [longest] + [40 + 29 * (i % 30) for i in range(299)]
    wl = W.custom("tiles", mode, lens, q_len, 2 * G, 2, 128, 16, seed=G + q_len)
    assert max(check(wl)) <= 5e-4


@pytest.mark.parametrize("mode,D,G,q_len", [(W.MODE_INT8, 128, 8, 9), (W.MODE_INT4, 128, 6, 11), (W.MODE_FP8, 128, 8, 15),
                                            (W.MODE_FP8_TENSOR, 64, 8, 13), (W.MODE_BF16, 128, 3, 11),
                                            (W.MODE_BF16, 64, 5, 13), (W.MODE_INT8, 128, 4, 17)])
@pytest.mark.parametrize("lens", [[3000, 20, 64, 700], [40 + 29 * (i % 30) for i in range(300)]],
                         ids=["few", "crowd"])
def test_a_workgroup_of_query_rows_that_is_not_full(mode, D, G, q_len, lens):
    """33 to 127 query rows per kv head where the many-row kernel takes them: row tiles and wavefronts of
    its one workgroup without rows, with a split context and (many pairs) without; a split-K granule
    keeps such calls on the streaming kernel, which must agree."""
    lens = [max(l, q_len) for l in lens]
    wl = W.custom("part", mode, lens, q_len, 2 * G, 2, D, 16, seed=G + q_len)
    errs = check(wl, chunks=(0, 256))
    assert max(errs) <= 5e-4


@pytest.mark.parametrize("mode,D,groups", [(W.MODE_BF16, 64, 33), (W.MODE_INT8, 64, 41), (W.MODE_FP8, 64, 65),
                                           (W.MODE_BF16, 64, 74), (W.MODE_INT8, 128, 18), (W.MODE_BF16, 128, 35),
                                           (W.MODE_INT4_GROUP, 128, 34)])
def test_row_groups_whose_parts_reach_past_them(mode, D, groups):
    """40 query rows, two or three row groups, and so many partials per row that the reduce cuts a row
    group into parts that do not divide it (7 x 5 or 11 x 3 parts of 32 rows, 6 x 3 of 16): the last part
    must stop at the group's last row, the next row is the next group's."""
    wl = W.custom("parts", mode, [64 * groups - 9], 5, 16, 2, D, 16, seed=groups)
    errs = check(wl, chunks=(64, 0))
    assert max(errs) <= 5e-4


@pytest.mark.parametrize("mode,D,G,q_len", [(W.MODE_INT8, 128, 8, 12), (W.MODE_BF16, 64, 8, 13), (W.MODE_INT4, 128, 4, 33),
                                            (W.MODE_FP8, 64, 8, 20)])
@pytest.mark.parametrize("lens", [[2900], [70, 3100] + [70 + i for i in range(20)], [64 * i + 1 for i in range(30)],
                                  [40] * 40 + [2500] + [130] * 60, [65 + i for i in range(130)] + [3000, 1]],
                         ids=["one", "one long", "all lengths", "one long of 101", "the last but one long"])
def test_contexts_are_cut_by_their_lengths(mode, D, G, q_len, lens):
    """The many-row kernel works its pieces out on the device: one long context among short ones, up to
    64 sequences and more, whatever bound on the lengths the call declares (with a bound far above
    them all, short contexts stay whole)."""
    lens = [max(l, q_len) for l in lens]
    wl = W.custom("cut", mode, lens, q_len, 2 * G, 2, D, 16, seed=len(lens) + D)
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    for bound in (max(lens), max(lens) + 77, 20000):
        got = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, max_len=bound)
        assert np.isfinite(got).all(), bound
        assert attn_err(got, want) <= 5e-4, bound


@pytest.mark.parametrize("lens,q_len,G,H,bs", [
    ([700, 655, 799] * 42, 13, 4, 4, 16),                 # 52 rows: a second row tile of four, two wavefronts without any
    ([900, 64, 65, 1, 959] * 40, 1, 65, 2, 64),           # 65 rows, contexts of one token and of whole groups
    ([640] * 60 + [4100], 16, 8, 2, 32),                  # 128 rows, one long context, cut alone
    ([300, 1025, 513] * 4, 290, 4, 4, 16), ([4287], 147, 4, 8, 128), ([3000, 2990] * 2, 257, 8, 1, 256)])
def test_many_rows_of_group_scaled_int4(lens, q_len, G, H, bs):
    """The many-row kernel of group-scaled int4, against the oracle on sequences of every length and against the
    streaming kernel on all (either rounds f16 probabilities: 2^-12 of a row's largest term), under a bound
    far above the lengths, and with a negative softmax scale."""
    from paper_2605_29639_amd import kvq
    lens = [max(l, q_len) for l in lens]
    wl = W.custom("group rows", W.MODE_INT4_GROUP, lens, q_len, G * H, H, 128, bs, seed=q_len + bs)
    cache, scales, desc = gpu_fill(wl)
    prof = kvq.prof_lib()
    assert prof.kvq_profile_group_rows(C.byref(desc), len(lens), q_len, G * H, max(lens), 0) == 1
    assert prof.kvq_profile_group_rows(C.byref(desc), len(lens), q_len, G * H, max(lens), 256) == 0
    for sign, bound in ((1.0, max(lens)), (-1.0, max(lens)), (1.0, 8 * max(lens))):
        wl.__class__ = type("Signed", (type(wl),), {"sm_scale": sign * abs(wl.sm_scale)})
        got = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, max_len=bound)
        want = gpu_attention(wl, cache, scales, desc, chunk_tokens=256, max_len=bound)
        assert np.isfinite(got).all()
        assert attn_err(got, want.astype(np.float64)) <= 5e-4
    if sum(lens) * q_len < 1 << 21:
        wl.__class__ = type("Signed", (type(wl),), {"sm_scale": abs(wl.sm_scale)})
        assert attn_err(gpu_attention(wl, cache, scales, desc, chunk_tokens=0), oracle_out(wl, *oracle_fill(wl))) <= 5e-4


WIDE = {  # lengths, query tokens, query heads, kv heads, declared bound, whether the lengths are long for it[, block size]
    "dead wavefronts": ([2500, 2337, 2100, 2499], 130, 64, 64, 2500, True),
    "a row block of one row": ([2500, 2433, 2369, 2500], 257, 32, 32, 2500, True),
    "cut": ([12000], 512, 32, 8, 12000, True),
    "cut, below the bound": ([9500], 512, 32, 8, 12000, True),
    "just too short": ([2100, 2000, 1800, 1600], 130, 64, 64, 2500, False),
    "just long enough": ([2100, 2000, 1800, 1601], 130, 64, 64, 2500, True),
    "one just too short": ([2500, 2500, 2480, 1216], 130, 64, 64, 2500, False),
    "one just long enough": ([2500, 2500, 2480, 1217], 130, 64, 64, 2500, True),
    "short": ([130, 191, 257, 200], 130, 64, 64, 2500, False),
    # one of the two kernels may cut contexts, the other may not; the merge is launched for both
    "not cut, the other kernel would": ([3000, 2990, 2900, 3000, 2950, 2999, 2937], 300, 16, 2, 3000, True),
    "one long, cut by the other kernel": ([3000, 301, 400, 310, 577, 300, 640], 300, 16, 2, 3000, False),
    "a walk of more table entries than threads": ([40000], 512, 32, 8, 40000, True),   # (four pieces of 626 entries)
    "32-token blocks": ([2500, 2433, 2369, 2500], 257, 32, 32, 2500, True, 32),
    "64-token blocks, cut": ([12000], 512, 32, 8, 12000, True, 64),
    "128-token blocks, walks from inside a block": ([11990], 512, 32, 8, 12000, True, 128),
    "256-token blocks": ([2500, 2337, 2100, 2499], 130, 64, 64, 2500, True, 256),
}


@pytest.mark.parametrize("mode", [m for m in MODES if m != W.MODE_INT4_GROUP])
@pytest.mark.parametrize("case", sorted(WIDE))
def test_workgroups_of_256_rows_against_the_streaming_kernels(mode, case):
    """Where contexts of max_seq_len would fill the chip with workgroups of 256 rows, the lengths decide on the
    device between that kernel and the one of 128 rows (for int8 and e4m3 codes).  Either must agree with the streaming kernels,
    also under a negative softmax scale.  Both sides are within the oracle's bound elsewhere; f16
    probabilities differ by 2^-12 of a row's largest term at most (measured 1e-4)."""
    import ctypes as C
    from paper_2605_29639_amd import kvq
    lens, q_len, hq, hkv, bound, long, bs = (*WIDE[case], 16)[:7]
    groups = [-(-l // 64) for l in lens]
    codes = mode in (W.MODE_INT8, W.MODE_FP8, W.MODE_FP8_TENSOR)
    wl = W.custom("wide", mode, lens, q_len, hq, hkv, 128, bs, seed=len(case))
    cache, scales, desc = gpu_fill(wl)
    prof, out = kvq.prof_lib(), (C.c_int64 * 8)()
    assert prof.kvq_profile_plan(C.byref(desc), len(lens), q_len, hq, bound, 0, 0, out) == kvq.OK and out[0] == 1 + codes
    if codes:
        assert prof.kvq_profile_wide(C.byref(desc), len(lens), q_len, hq, bound, out) == kvq.OK
        assert (sum(groups) >= out[0] and min(groups) >= out[2]) == long
    for sign in (1.0, -1.0):
        signed = type("Signed", (type(wl),), {"sm_scale": sign * abs(wl.sm_scale)})
        wl.__class__ = signed
        got = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, max_len=bound)
        prof.kvq_profile_prefill_kernel(0)
        try:
            want = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, max_len=bound, L=prof)
        finally:
            prof.kvq_profile_prefill_kernel(1)
        assert np.isfinite(got).all()
        assert attn_err(got, want.astype(np.float64)) <= 5e-4


@pytest.mark.parametrize("mode,D", [(W.MODE_INT4, 128), (W.MODE_INT4_GROUP, 128), (W.MODE_INT8, 64), (W.MODE_FP8, 64),
                                    (W.MODE_FP8_TENSOR, 64), (W.MODE_BF16, 64)])
@pytest.mark.parametrize("seqs", [60, 80])
def test_a_granule_makes_few_or_many_wavefronts(mode, D, seqs):
    """A split-K granule of 64 tokens over 960 and over 1280 groups, below and above one wavefront for each of
    1024 SIMDs, where other instances of the one-tile kernels run: the automatic split must agree."""
    wl = W.custom("granule", mode, [449 + b % 64 for b in range(seqs)], 1, 8, 2, D, 16, seed=seqs)
    errs = check(wl, chunks=(64, 0))
    assert max(errs) <= 5e-4


@pytest.mark.parametrize("mode,D", [(m, 128) for m in MODES] + [(W.MODE_BF16, 64), (W.MODE_FP8, 64)])
@pytest.mark.parametrize("q_len", [1, 4, 40])
def test_a_negative_softmax_scale(mode, D, q_len):
    """Smallest dot products first: the kernels that take a row's maximum of the unscaled products must
    turn it round (one and two row tiles, the many-row kernel)."""
    wl = W.custom("negative", mode, [300, 129, 64], q_len, 16, 2, D, 16, seed=q_len)
    scale = -wl.sm_scale
    wl.__class__ = type("Negative", (type(wl),), {"sm_scale": scale})
    assert wl.sm_scale < 0 and max(check(wl)) <= 5e-4


@pytest.mark.parametrize("hq", [8, 16])
@pytest.mark.parametrize("bound", [1100, 60000])
def test_group_scaled_int4_with_one_and_two_wavefronts_per_simd(hq, bound):
    """Up to eight query rows and a long enough list (here by its declared bound) run twice the wavefronts with
    half the rows in a partial's slot; a short list runs the other instance of the kernel."""
    wl = W.custom("per_simd", W.MODE_INT4_GROUP, [1100, 30, 64, 700, 415], 1, hq, 2, 128, 16, seed=hq)
    oc, osc = oracle_fill(wl)
    want = oracle_out(wl, oc, osc)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    got = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, max_len=bound)
    assert np.isfinite(got).all() and attn_err(got, want) <= 5e-4


@pytest.mark.parametrize("G,q_len", [(1, 1), (1, 3), (2, 2), (3, 1), (4, 1), (5, 1)])
@pytest.mark.parametrize("seqs,bound", [(5, None), (5, 60000), (300, None)])
def test_group_scaled_int4_with_four_rows_or_fewer(G, q_len, seqs, bound):
    """Up to four rows take four columns of the tile each (five rows do not): a workgroup for each pair, an even
    split with twice the wavefronts, and more pairs than wavefronts; contexts that end in each quarter
    of a group, so that some of a row's columns see no token at all.  q is large, for
    maxima that differ between a row's columns."""
    lens = [(1100, 30, 64, 700, 415, 5, 17, 33, 49, 129)[i % 10] // (1 if seqs < 10 else 2) + q_len for i in range(seqs)]
    wl = W.custom("banks", W.MODE_INT4_GROUP, lens, q_len, 2 * G, 2, 128, 16, seed=G + q_len)
    scale = 4 * wl.sm_scale
    wl.__class__ = type("Peaked", (type(wl),), {"sm_scale": scale})
    oc, osc = oracle_fill(wl)
    cache, scales, desc = upload_oracle_cache(wl, oc, osc)
    got = gpu_attention(wl, cache, scales, desc, chunk_tokens=0, **({"max_len": bound} if bound else {}))
    assert np.isfinite(got).all() and attn_err(got, oracle_out(wl, oc, osc)) <= 5e-4


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("q_len", [1, 4, 6, 20])
def test_a_peaked_row_of_an_unquantized_cache(D, q_len):
    """A row that attends to one token alone returns that token's V: its probability is 1 to within the
    rounding of the exponent (about 130 here, so 2^-17), numerator and denominator alike, and goes into
    P.V as two bf16 terms whose second is rounded, 2^-17 of it at most and nothing of a value beside a
    power of two.  Cut instead of rounded it would lose 2^-16."""
    import torch
    from paper_2605_29639_amd import kvq
    H, G, L, bs = 2, 8, 700, 16
    desc = kvq.make_desc(W.MODE_BF16, L // bs + 1, bs, H, D)
    cache, scales = kvq.alloc_cache(desc)
    g = torch.Generator(device="cuda")
    g.manual_seed(D + q_len)
    k, v = torch.randn((2, L, H, D), generator=g, device="cuda").to(torch.bfloat16)
    kvq.kv_quant_write(k, v, torch.arange(L, device="cuda"), cache, scales, desc)
    t = torch.randint(0, L - 128, (q_len, H, G), generator=g, device="cuda")
    rows = k.float().permute(1, 0, 2)[torch.arange(H, device="cuda")[None, :, None], t]     # [q_len, H, G, D]
    q = (rows * (1024.0 / D)).to(torch.bfloat16).view(q_len, H * G, D)
    want = v.float().permute(1, 0, 2)[torch.arange(H, device="cuda")[None, :, None], t].view(q_len, H * G, D)
    tables = torch.arange(L // bs + 1, dtype=torch.int32, device="cuda")[None].contiguous()
    lens = torch.tensor([L], dtype=torch.int32, device="cuda")
    out = torch.empty((q_len, H * G, D), device="cuda")
    for chunk in (0, 64, 1024):
        ws = kvq.alloc_workspace(desc, 1, q_len, H * G, L, chunk)
        kvq.paged_decode_attn(q, cache, scales, desc, tables, lens, q_len, L, 1.0 / D ** 0.5, out, ws, chunk_tokens=chunk)
        torch.cuda.synchronize()
        assert float(((out - want).abs() / want.abs().clamp(min=1e-3)).max()) <= 2.0 ** -17, chunk
