"""GPU parity of the shapes outside bf16 x head dimension 64 / 128: fp32 prefill and bf16 prefill
with other head dimensions on the matrix cores, in every split of the work that the launchers
choose, at head dimensions on and between the padded sizes; decoding with the same shapes."""
import numpy as np
import pytest
import torch

import fedattn_inputs as fi
import oracle
import paper_2511_02647_amd as fa
from gpu_util import check, decode, dev, host, prefill, say
from test_gpu_parity import rand_block

pytestmark = pytest.mark.gpu
BF16, F32 = torch.bfloat16, torch.float32

# Which launch a layout takes on 256 CUs is checked by tests/test_host_rules.py: those called by a launch's name take it.
# (lengths, Hq, Hkv), fp32: the keys of 16 query rows of a head split over a workgroup, few workgroups and more than are resident at
# once; heads sharing a workgroup (at least 1536 workgroups on 256 CUs).  Ragged ends, an empty and
# a one-token segment, groups of 1, 2 and 4 heads per KV head.
LAYOUTS = {"narrow": ([70, 0, 63, 1, 258], 4, 1), "split": ([500, 33, 484], 16, 8), "shared": ([3101, 2, 3137], 32, 8)}


@pytest.mark.parametrize("layout", sorted(LAYOUTS))
@pytest.mark.parametrize("D", [8, 40, 64, 88, 128, 136, 256])
def test_f32_prefill(layout, D):
    lens, Hq, Hkv = LAYOUTS[layout]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(seg[-1])
    q, k, v = rand_block(41, total, Hq, Hkv, D, bf16=False)
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=200)
    for sync, causal in [(0, True), (1, True), (1, False)]:
        what = "f32 %s D=%d sync=%d causal=%d" % (layout, D, sync, causal)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=F32, causal=causal, sync_override=sync)
        ref = oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=bool(sync), causal=causal)
        check(got[rows, heads], ref, F32, what)


@pytest.mark.parametrize("D", [8, 24, 32, 56, 64, 96, 104, 128])
def test_f32_prefill_ends_of_key_slices(D):
    """Walks that end on, before and behind a 16-key slice and leave one to four wavefronts without one, every row checked."""
    lens, Hq, Hkv = [1, 15, 16, 17, 0, 31, 33, 48, 63, 64, 65, 80, 129], 3, 1
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(44, int(seg[-1]), Hq, Hkv, D, bf16=False)
    for sync, causal in [(0, True), (1, True), (0, False), (1, False)]:
        what = "f32 slice ends D=%d sync=%d causal=%d" % (D, sync, causal)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=F32, causal=causal, sync_override=sync)
        check(got, oracle.attend_block(q, k, v, seg, is_sync=bool(sync), causal=causal), F32, what)


# one head per workgroup with split keys, on short and long walks (head dimensions beyond 128: 4-wave workgroups, in an
# order if causal); 4-wave workgroups, one tile each, heaviest first (the other launches: test_bf16_prefill_every_launch)
BF16_LAYOUTS = {"short": ([70, 0, 63, 1, 258], 4, 1), "long": ([1100, 0, 1003], 6, 3), "four": ([3101, 2, 3137], 32, 8)}


@pytest.mark.parametrize("layout", sorted(BF16_LAYOUTS))
@pytest.mark.parametrize("D", [8, 40, 72, 96, 120, 160, 184, 200, 256])
def test_bf16_prefill_other_head_dims(layout, D):
    """The weights enter the second product exactly (three bf16 parts), so the error is that of fp32
    arithmetic plus the rounding of the output to bf16, half a unit in the last place: 2^-9 of the value."""
    lens, Hq, Hkv = BF16_LAYOUTS[layout]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(seg[-1])
    q, k, v = rand_block(43, total, Hq, Hkv, D)
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=200)
    for sync, causal in [(0, True), (1, True), (1, False)]:
        what = "bf16 %s D=%d sync=%d causal=%d" % (layout, D, sync, causal)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=BF16, causal=causal, sync_override=sync)
        ref = oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=bool(sync), causal=causal)
        check(got[rows, heads], ref, BF16, what)
        assert np.all(np.abs(got[rows, heads] - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5), what   # twice half a unit: values at a binade's edge


@pytest.mark.parametrize("chunk", [1, 20, 64])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_keep_lists_with_and_without_workspace(chunk, causal, dtype):
    seg = np.array([0, 130, 130, 321, 402], dtype=np.int32)
    Hq, Hkv, D = 4, 2, 72
    q, k, v = rand_block(42, 402, Hq, Hkv, D, bf16=dtype == BF16)
    flags = (np.random.default_rng(7).random(int(fi.chunk_counts(np.diff(seg), chunk).sum())) < 0.4).astype(np.uint8)
    ref = oracle.attend_block(q, k, v, seg, is_sync=True, causal=causal, keep_tok=oracle.expand_keep_chunks(flags, seg, chunk))
    say("keep-list chunk=%d causal=%d" % (chunk, causal))
    got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=1, block=0, dtype=dtype, causal=causal, keep_chunks=flags, chunk_tokens=chunk)
    check(got, ref, dtype, "keep-list chunk=%d" % chunk)
    # without a workspace the flags are read by the general kernel
    p = fa.make_params(4, Hq, Hkv, D, 1, dtype, causal=causal)
    tq = dev(q, dtype)
    out = torch.full_like(tq, float("nan"))
    fa.fedattn_prefill(p, 0, tq, dev(k, dtype), dev(v, dtype), out, seg, keep_chunks=torch.from_numpy(flags).to("cuda"), chunk_tokens=chunk)
    torch.cuda.synchronize()
    check(host(out), ref, dtype, "keep-list chunk=%d, no workspace" % chunk)


@pytest.mark.parametrize("dtype,D", [(BF16, d) for d in (8, 40, 80, 96, 120, 160, 200, 256)] + [(F32, d) for d in (8, 64, 72, 128, 136, 256)])
@pytest.mark.parametrize("lens,Hq,Hkv", [([200, 77, 130], 8, 2), ([64], 3, 1), ([700, 0, 1, 333, 64, 65], 12, 2), ([40, 1500], 40, 2)])
def test_decode_other_shapes(dtype, D, lens, Hq, Hkv):
    """One chunk and many per segment, an empty segment, one to 120 query columns; with and without a workspace."""
    N = len(lens)
    cap = np.asarray(lens, dtype=np.int32) + 3
    seg = np.concatenate([[0], np.cumsum(cap)]).astype(np.int32)
    lens = np.asarray(lens, dtype=np.int32)
    _, kc, vc = rand_block(50, int(seg[-1]), Hkv, Hkv, D, bf16=dtype == BF16)
    q, _, _ = rand_block(51, N, Hq, Hkv, D, bf16=dtype == BF16)
    p = fa.make_params(N, Hq, Hkv, D, 0, dtype)
    for sync, rl in [(0, None), (1, None), (1, lens // 2)]:
        what = "decode %s D=%d lens=%s %d/%d sync=%d remote=%s" % (dtype, D, lens.tolist(), Hq, Hkv, sync, rl is not None)
        say(what)
        ref = oracle.decode_step(q, kc, vc, seg, lens, is_sync=bool(sync), remote_lens=rl)
        got = decode(q, kc, vc, seg, lens, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=dtype, remote_lens=rl, sync_override=sync)
        check(got, ref, dtype, what)
        if dtype == BF16:   # fp32 arithmetic, output rounded to bf16 (see above)
            assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5), what
        tq = dev(q, dtype)
        out = torch.full_like(tq, float("nan"))
        fa.fedattn_decode(p, 0, tq, dev(kc, dtype), dev(vc, dtype), out, seg, lens, remote_lens=rl, sync_override=sync)
        torch.cuda.synchronize()
        check(host(out), ref, dtype, what + ", no workspace")


@pytest.mark.parametrize("dtype,D", [(F32, 64), (BF16, 96)])
def test_decode_other_shapes_fused_blocks_equal_single_calls(dtype, D):
    N, Hq, Hkv, M, cap = 3, 8, 2, 5, 300
    seg = (np.arange(N + 1) * cap).astype(np.int32)
    lens = np.array([300, 20, 129], dtype=np.int32)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    mk = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float32).to(dtype)
    q, k, v = mk(M, N, Hq, D), mk(M, N * cap, Hkv, D), mk(M, N * cap, Hkv, D)
    p = fa.make_params(N, Hq, Hkv, D, 2, dtype)
    one, many = torch.zeros_like(q), torch.zeros_like(q)
    need = fa.fedattn_workspace_bytes(p, fa.FEDATTN_OP_DECODE, N * cap)
    ws = torch.full((4 * (need + 256),), 255, dtype=torch.uint8, device="cuda")
    say("decode %s D=%d fused blocks" % (dtype, D))
    for b in range(M):
        fa.fedattn_decode(p, b, q[b], k[b], v[b], one[b], seg, lens, workspace=ws)
    fa.fedattn_decode_blocks_fused(p, 0, M, q, k, v, many, q[0].numel(), k[0].numel(), seg, lens, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(one, many)


# sync blocks that are taken as pairs, also under a keep-list: 256 of them
PAIRS = {"ragged": ([500, 512, 497, 490], 32, 8), "even": ([512, 512, 512, 512], 32, 8), "one": ([2030], 32, 8)}
PAIRS_DIMS = [64, 96, 128]


@pytest.mark.parametrize("layout", sorted(PAIRS))
@pytest.mark.parametrize("D", PAIRS_DIMS)
@pytest.mark.parametrize("chunk", [0, 64, 7])
def test_bf16_prefill_in_pairs(layout, D, chunk):
    lens, Hq, Hkv = PAIRS[layout]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(seg[-1])
    q, k, v = rand_block(46, total, Hq, Hkv, D)
    flags = keep = None
    if chunk:
        flags = (np.random.default_rng(8).random(int(fi.chunk_counts(np.diff(seg), chunk).sum())) < 0.5).astype(np.uint8)
        keep = oracle.expand_keep_chunks(flags, seg, chunk)
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=150)
    what = "pairs %s D=%d chunk=%d" % (layout, D, chunk)
    say(what)
    got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=BF16, sync_override=1, keep_chunks=flags, chunk_tokens=chunk)
    check(got[rows, heads], oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=True, keep_tok=keep), BF16, what)


@pytest.mark.parametrize("dtype,Hq,Hkv,D,tiles", [(BF16, 4, 1, 64, 32), (BF16, 1, 1, 64, 32), (BF16, 2, 1, 128, 64), (BF16, 3, 1, 96, 32), (F32, 1, 1, 64, 16)])
@pytest.mark.parametrize("extra", [0, 1])
def test_prefill_with_as_many_query_tiles_as_listed_and_one_more(dtype, Hq, Hkv, D, tiles, extra):
    """512 query tiles (of 32, 64 or 16 rows) are listed by the host, more are found in the segment tables."""
    lens = [tiles * 300, 0, tiles * 3 - 5, tiles * 209 + extra]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(45, int(seg[-1]), Hq, Hkv, D, bf16=dtype == BF16)
    rows, heads = fi.sample_rows(seg, Hq, 96, fi.DEFAULT_SEED, salt=D, tile=tiles, max_boundary_rows=150)
    for sync, causal in [(0, True), (1, True), (1, False)]:
        what = "%d tiles D=%d sync=%d causal=%d" % (512 + extra, D, sync, causal)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=dtype, causal=causal, sync_override=sync)
        check(got[rows, heads], oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=bool(sync), causal=causal), dtype, what)


# bf16 with head dimension 64 / 128: ragged layouts, named after the launch of their causal sync block, with empty and
# one-token segments
PLAN_LAYOUTS = {"split": ([70, 0, 63, 1, 258], 4, 1), "split-long": ([1, 1999, 33], 2, 1), "eight-short": ([100, 1, 0, 301, 33], 64, 16),
                "eight": ([129, 0, 700, 1, 1203], 16, 4), "eight-pairs": ([578, 866, 0, 1, 502], 32, 8), "four": ([3101, 2, 3137], 32, 8)}


@pytest.mark.parametrize("layout", sorted(PLAN_LAYOUTS))
@pytest.mark.parametrize("D,scale", [(128, 0.0), (64, 0.0), (128, 0.2), (64, 0.3)])
def test_bf16_prefill_launches(layout, D, scale):
    lens, Hq, Hkv = PLAN_LAYOUTS[layout]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(60, int(seg[-1]), Hq, Hkv, D)
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=200)
    for sync, causal in [(0, True), (1, True), (1, False)]:
        what = "bf16 %s D=%d scale=%.1f sync=%d causal=%d" % (layout, D, scale, sync, causal)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=BF16, causal=causal, sync_override=sync, scale=scale)
        ref = oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=bool(sync), causal=causal, scale=scale if scale else None)
        check(got[rows, heads], ref, BF16, what)


# (launch, sync, causal, lengths, Hq, Hkv, head dimensions): every launch of a bf16 prefill block in every mode that reaches
# it, at every padded head dimension that has it
ALL_D = (32, 40, 64, 72, 120, 128)
LAUNCHES = [("eight", 1, False, [1, 0, 160, 181, 168, 199], 32, 8, ALL_D), ("eight", 0, True, [67, 36, 0, 82, 99, 1], 32, 8, ALL_D),
            ("eight", 1, True, [214, 1, 259, 0, 262, 263], 32, 8, ALL_D), ("eight-pairs", 0, True, [1249, 1276, 1260, 1275, 1, 0], 12, 4, ALL_D),
            ("eight-pairs", 1, True, [578, 866, 0, 1, 502], 32, 8, ALL_D),
            ("eight-pairs", 1, True, [0, 2136, 1885, 1745, 1, 2311], 8, 2, (64, 72, 120, 128)),    # 255 tiles: one without a partner
            ("four", 1, False, [378, 340, 392, 1, 0, 363], 32, 8, ALL_D + (160, 224)),
            ("four", 0, True, [967, 965, 1, 0, 1050, 955], 24, 8, ALL_D + (192,)), ("four", 1, True, [1101, 1062, 1075, 1192, 0, 1], 24, 8, ALL_D + (256,)),
            ("four-ordered", 0, True, [34, 60, 50, 48, 0, 1], 32, 8, (32, 40, 72, 120, 160, 184)),
            ("four-ordered", 0, True, [450, 1, 574, 569, 541, 0], 24, 8, (64, 128)), ("four-ordered", 1, True, [47, 48, 48, 0, 44, 1], 32, 8, (128, 208, 256)),
            ("split", 1, False, [676, 1, 0, 784, 1894, 645], 1, 1, ALL_D), ("split", 0, True, [139, 72, 94, 0, 1, 194], 8, 2, ALL_D),
            ("split", 1, True, [134, 119, 117, 129, 1, 0], 8, 8, ALL_D)]


@pytest.mark.parametrize("launch,sync,causal,lens,Hq,Hkv,D", [x[:6] + (d,) for x in LAUNCHES for d in x[6]])
def test_bf16_prefill_every_launch(launch, sync, causal, lens, Hq, Hkv, D):
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(61, int(seg[-1]), Hq, Hkv, D)
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=200)
    for scale in (0.0, 0.2) if D in (64, 128) else (0.0,):     # folded into the query operand or not
        what = "bf16 launch %s D=%d sync=%d causal=%d scale=%.1f" % (launch, D, sync, causal, scale)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=BF16, causal=causal, sync_override=sync, scale=scale)
        ref = oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=bool(sync), causal=causal, scale=scale if scale else None)
        check(got[rows, heads], ref, BF16, what)
        if D not in (64, 128):
            assert np.all(np.abs(got[rows, heads] - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5), what   # as above


# several blocks in one launch: pairs of tiles, in 8-wave workgroups (few) and 4-wave ones (at least two per CU)
@pytest.mark.parametrize("lens,Hq,Hkv", [([130, 0, 70, 133], 8, 2), ([700, 1, 350, 333], 32, 8)])
@pytest.mark.parametrize("dtype,D", [(BF16, 72), (BF16, 120), (BF16, 200), (F32, 40), (F32, 128)])
def test_prefill_blocks_other_shapes(lens, Hq, Hkv, dtype, D):
    M, H = 4, 2
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    blocks = [rand_block(62 + b, int(seg[-1]), Hq, Hkv, D, bf16=dtype == BF16) for b in range(M)]
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=100)
    for causal in (True, False):
        p = fa.make_params(len(lens), Hq, Hkv, D, H, dtype, causal=causal)
        tq, tk, tv = (torch.stack([dev(b[i], dtype) for b in blocks]) for i in range(3))
        out = torch.full_like(tq, float("nan"))
        what = "prefill_blocks %s D=%d %d/%d causal=%d" % (dtype, D, Hq, Hkv, causal)
        say(what)
        fa.fedattn_prefill_blocks(p, 0, M, tq, tk, tv, out, tq[0].numel(), tk[0].numel(), seg)
        torch.cuda.synchronize()
        for b in range(M):
            ref = oracle.attend_rows(*blocks[b], seg, rows, heads, is_sync=oracle.is_sync_block(H, b), causal=causal)
            check(host(out[b])[rows, heads], ref, dtype, what)


# more chunks than a wavefront has lanes, rows past the 4096 where a workgroup's share grows, chunks longer than
# a segment, kept last chunks that end inside a tile; as many participants as there can be
COMPACTION = {"long": [4500, 0, 1, 70, 511, 512, 513, 4096], "many": [1 + 5 * (i % 7) for i in range(fa.FEDATTN_MAX_PARTICIPANTS)]}


@pytest.mark.parametrize("layout", sorted(COMPACTION))
@pytest.mark.parametrize("chunk", [1, 3, 513, 64, 128, 8192])
def test_keep_list_compaction(layout, chunk):
    seg = np.concatenate([[0], np.cumsum(COMPACTION[layout])]).astype(np.int32)
    Hq, Hkv, D = 2, 1, 64
    q, k, v = rand_block(44, int(seg[-1]), Hq, Hkv, D)
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=chunk, tile=64, max_boundary_rows=200)
    n_flags = int(fi.chunk_counts(np.diff(seg), chunk).sum())
    for share in (0.4, 1.0):
        flags = (np.random.default_rng(8).random(n_flags) < share).astype(np.uint8)
        kt = oracle.expand_keep_chunks(flags, seg, chunk)
        for causal in (True, False):
            what = "compaction %s chunk=%d share=%.1f causal=%d" % (layout, chunk, share, causal)
            say(what)
            got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=1, block=0, dtype=BF16, causal=causal, keep_chunks=flags, chunk_tokens=chunk)
            ref = oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=True, causal=causal, keep_tok=kt)
            check(got[rows, heads], ref, BF16, what)


@pytest.mark.parametrize("lens", [[1 + 5 * (i % 7) for i in range(fa.FEDATTN_MAX_PARTICIPANTS)], [300, 0, 1, 64, 65, 130, 17, 16, 90], [33, 70, 1, 129]])
@pytest.mark.parametrize("D", [24, 96, 128])
@pytest.mark.parametrize("chunk,share", [(1, 0.1), (20, 0.6), (64, 0.5), (1, 0.0)])
def test_f32_keep_lists_of_short_tiles(lens, D, chunk, share):
    """Lists of none to 127 tiles of 1 to 64 rows: empty slices left out (from four participants on, from eight with chunks of a tile and more) or walked."""
    Hq, Hkv = 2, 1
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(49, int(seg[-1]), Hq, Hkv, D, bf16=False)
    flags = (np.random.default_rng(9).random(int(fi.chunk_counts(np.diff(seg), chunk).sum())) < share).astype(np.uint8)
    keep = oracle.expand_keep_chunks(flags, seg, chunk)
    for causal in (True, False):
        what = "f32 short tiles N=%d D=%d chunk=%d share=%.1f causal=%d" % (len(lens), D, chunk, share, causal)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=1, block=0, dtype=F32, causal=causal, keep_chunks=flags, chunk_tokens=chunk)
        check(got, oracle.attend_block(q, k, v, seg, is_sync=True, causal=causal, keep_tok=keep), F32, what)


@pytest.mark.parametrize("dtype,D", [(BF16, 128), (BF16, 64), (BF16, 72), (F32, 64)])
@pytest.mark.parametrize("chunk", [1, 20, 64])
@pytest.mark.parametrize("tail", [1, 31, 32, 33])
def test_kept_tiles_load_only_kept_rows(dtype, D, chunk, tail):
    """Listed tiles with 1 to 33 valid rows, last in their participant's list: what follows them in memory (rows of a
    participant that shares nothing, unwritten workspace, the end of K and V) is NaN and must not reach anybody."""
    lens = [64 + tail, 45, 70, 64 + tail]
    Hq, Hkv = 8, 2
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(46, int(seg[-1]), Hq, Hkv, D, bf16=dtype == BF16)
    first = np.concatenate([[0], np.cumsum(fi.chunk_counts(np.diff(seg), chunk))])
    flags = np.ones(int(first[-1]), dtype=np.uint8)
    flags[first[1]:first[2]] = 0              # participant 1 shares nothing
    if chunk == 1:                            # `tail` rows of the others, from anywhere
        for n in (0, 2, 3):
            flags[first[n]:first[n + 1]] = 0
            flags[first[n] + np.random.default_rng(n).choice(lens[n], min(tail, lens[n]), replace=False)] = 1
    kt = oracle.expand_keep_chunks(flags, seg, chunk)
    kn, vn = k.copy(), v.copy()
    kn[seg[1]:seg[2]] = vn[seg[1]:seg[2]] = np.nan
    others = np.r_[seg[0]:seg[1], seg[2]:seg[4]]
    for causal in (True, False):
        what = "kept tiles %s D=%d chunk=%d tail=%d causal=%d" % (dtype, D, chunk, tail, causal)
        ref = oracle.attend_block(q, k, v, seg, is_sync=True, causal=causal, keep_tok=kt)
        say(what)
        got = prefill(q, k, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=1, block=0, dtype=dtype, causal=causal, keep_chunks=flags, chunk_tokens=chunk)
        check(got, ref, dtype, what)
        got = prefill(q, kn, vn, seg, Hq=Hq, Hkv=Hkv, D=D, H=1, block=0, dtype=dtype, causal=causal, keep_chunks=flags, chunk_tokens=chunk)
        check(got[others], ref[others], dtype, what + ", participant 1 NaN")


@pytest.mark.parametrize("dtype,D", [(BF16, 128), (BF16, 64), (BF16, 72), (F32, 64)])
@pytest.mark.parametrize("lens", [[64], [512], [576], [2048], [2112], [9000], [1, 0, 130], [65, 300, 7], [700, 1, 64, 65]])
def test_decode_merge_inside_the_launch(dtype, D, lens):
    """Chunk counts on both sides of the merge's batches of eight and of its limit, local and sync blocks in turn over one
    workspace full of ones; a second call finds the first one's partials and counters, a third another order of blocks."""
    N, Hq, Hkv, M = len(lens), 8, 2, 4
    lens = np.asarray(lens, dtype=np.int32)
    seg = np.concatenate([[0], np.cumsum(lens + 2)]).astype(np.int32)
    p = fa.make_params(N, Hq, Hkv, D, 2, dtype)
    q = np.stack([rand_block(70 + b, N, Hq, Hkv, D, bf16=dtype == BF16)[0] for b in range(M)])
    kv = [rand_block(80 + b, int(seg[-1]), Hkv, Hkv, D, bf16=dtype == BF16)[1:] for b in range(M)]
    tq, tk, tv = dev(q, dtype), dev(np.stack([k for k, _ in kv]), dtype), dev(np.stack([v for _, v in kv]), dtype)
    ws = torch.full((fa.fedattn_workspace_bytes(p, fa.FEDATTN_OP_DECODE, int(seg[-1])),), 255, dtype=torch.uint8, device="cuda")
    for first in (0, 0, 1):
        what = "decode merge %s D=%d lens=%s first=%d" % (dtype, D, lens.tolist(), first)
        say(what)
        out = torch.full_like(tq, float("nan"))
        fa.fedattn_decode_blocks(p, first, M, tq, tk, tv, out, tq[0].numel(), tk[0].numel(), seg, lens, workspace=ws)
        torch.cuda.synchronize()
        for b in range(M):
            ref = oracle.decode_step(q[b], kv[b][0], kv[b][1], seg, lens, is_sync=oracle.is_sync_block(2, first + b))
            check(host(out[b]), ref, dtype, what)


@pytest.mark.parametrize("D,Hq", [(64, 16), (128, 32), (128, 64), (256, 32), (72, 64)])
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_decode_sync_blocks_that_fill_the_chip(dtype, D, Hq):
    """Enough (chunk, KV head) pairs that the launches take more columns per workgroup (fp32: 16, 32 or 64) and
    longer chunks (bf16); ragged, empty and one-row segments, rows that only their own participant sees."""
    lens = np.array([900, 700, 1, 1300, 650, 1000, 0, 777], dtype=np.int32)
    N, Hkv = len(lens), 8
    seg = np.concatenate([[0], np.cumsum(lens + 1)]).astype(np.int32)
    q, _, _ = rand_block(90, N, Hq, Hkv, D, bf16=dtype == BF16)
    _, kc, vc = rand_block(91, int(seg[-1]), Hkv, Hkv, D, bf16=dtype == BF16)
    for rl in (None, lens - lens // 3):
        say("decode sync %s D=%d Hq=%d remote=%s" % (dtype, D, Hq, rl is not None))
        got = decode(q, kc, vc, seg, lens, Hq=Hq, Hkv=Hkv, D=D, H=1, block=0, dtype=dtype, remote_lens=rl)
        ref = oracle.decode_step(q, kc, vc, seg, lens, is_sync=True, remote_lens=rl)
        check(got, ref, dtype, "decode sync D=%d Hq=%d" % (D, Hq))


# what a masked key holds must not reach the rows that do not see it: layouts for every tile kernel of the shapes outside
# bf16 x 64 / 128 (fp32: keys split, few and many workgroups, and heads sharing tiles; bf16: split, 8-wave and 4-wave launches)
HIDDEN = [("narrow", F32, 64), ("narrow", F32, 40), ("split", F32, 128), ("split", F32, 256), ("shared", F32, 32), ("short", BF16, 72),
          ("short", BF16, 96), ("eight", BF16, 72), ("eight-pairs", BF16, 72), ("local-pairs", BF16, 72), ("long", BF16, 160), ("four", BF16, 40), ("four", BF16, 256)]
HIDDEN_LAYOUTS = dict(LAYOUTS, **BF16_LAYOUTS, **{"eight": ([214, 1, 259, 0, 262, 263], 32, 8), "eight-pairs": ([578, 1, 502, 0, 866], 32, 8), "local-pairs": ([1249, 1276, 1260, 1275, 1, 0], 12, 4)})   # the poisoned token is in a second walk


@pytest.mark.parametrize("layout,dtype,D", HIDDEN)
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_values_of_masked_keys_do_not_reach_other_rows(layout, dtype, D, bad):
    lens, Hq, Hkv = HIDDEN_LAYOUTS[layout]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(47, int(seg[-1]), Hq, Hkv, D, bf16=dtype == BF16)
    t = int(seg[2]) + lens[2] // 2                       # a token inside participant 2's segment
    vn = v.copy()
    vn[t, 0, D // 2 + 1] = bad                           # seen through KV head 0 only
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=100)
    near = np.arange(max(0, t - 130), min(int(seg[-1]), t + 40))     # every row of the query tiles around it, first and last head
    rows = np.concatenate([rows, near, near])
    heads = np.concatenate([heads, np.zeros_like(near), np.full_like(near, Hq - 1)])
    for sync in (0, 1):
        what = "hidden value %s D=%d %s sync=%d bad=%s" % (layout, D, dtype, sync, bad)
        say(what)
        got = prefill(q, k, vn, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=dtype, sync_override=sync)[rows, heads]
        sees = (rows >= t) & (heads < Hq // Hkv) & ((sync == 1) | (rows < seg[3]))
        ref = oracle.attend_rows(q, k, v, seg, rows, heads, is_sync=bool(sync))
        check(got[~sees], ref[~sees], dtype, what)
        assert sees.any() and not np.isfinite(got[sees][:, D // 2 + 1]).any(), what


@pytest.mark.parametrize("layout,dtype,D", [("narrow", F32, 40), ("split", F32, 88), ("short", BF16, 72), ("eight", BF16, 72), ("long", BF16, 168)])
def test_an_infinite_key_element_beside_the_padding(layout, dtype, D):
    """A score of minus infinity is a weight of zero, also where the tile pads the head dimension."""
    lens, Hq, Hkv = HIDDEN_LAYOUTS[layout]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = rand_block(48, int(seg[-1]), Hq, Hkv, D, bf16=dtype == BF16)
    q[:, :, D - 1] = -1.0
    t = int(seg[2]) + 5
    kn, kf = k.copy(), k.copy()
    kn[t, :, D - 1], kf[t, :, D - 1] = np.inf, 2.0 ** 100
    rows, heads = fi.sample_rows(seg, Hq, 64, fi.DEFAULT_SEED, salt=D, tile=32, max_boundary_rows=100)
    for sync, causal in [(0, True), (1, True), (1, False)]:
        what = "infinite key %s D=%d %s sync=%d causal=%d" % (layout, D, dtype, sync, causal)
        say(what)
        got = prefill(q, kn, v, seg, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=dtype, causal=causal, sync_override=sync)
        check(got[rows, heads], oracle.attend_rows(q, kf, v, seg, rows, heads, is_sync=bool(sync), causal=causal), dtype, what)


@pytest.mark.parametrize("dtype,D", [(F32, 64), (F32, 40), (F32, 256), (BF16, 72), (BF16, 96), (BF16, 200)])
@pytest.mark.parametrize("lens,Hq,Hkv", [([60, 40, 50], 4, 2), ([200, 77, 130], 8, 2), ([700, 90, 1, 333, 64, 65], 12, 2), ([40, 1500, 9], 40, 2)])
def test_decode_private_rows_stay_private(dtype, D, lens, Hq, Hkv):
    """Merged in the launch (one chunk, several) and by the combine kernel; participant 1's private rows are NaN, or a
    key of its segment has an infinite element that gives every query a score of minus infinity."""
    N, lens = len(lens), np.asarray(lens, dtype=np.int32)
    seg = np.concatenate([[0], np.cumsum(lens + 3)]).astype(np.int32)
    _, kc, vc = rand_block(52, int(seg[-1]), Hkv, Hkv, D, bf16=dtype == BF16)
    q, _, _ = rand_block(53, N, Hq, Hkv, D, bf16=dtype == BF16)
    rl = np.maximum(lens - 7, 0).astype(np.int32)
    q[:, :, D - 1] = -1.0
    others = np.arange(N) != 1
    for what, poison in (("V", np.nan), ("V", np.inf), ("K", np.inf)):
        kn, vn, kf = kc.copy(), vc.copy(), kc.copy()
        if what == "V":
            vn[seg[1] + rl[1]:seg[1] + lens[1]] = poison
        else:
            kn[seg[1] + 3, :, D - 1], kf[seg[1] + 3, :, D - 1] = np.inf, 2.0 ** 100
        for sync in (0, 1):
            name = "private rows %s D=%d lens=%s %d/%d %s=%s sync=%d" % (dtype, D, lens.tolist(), Hq, Hkv, what, poison, sync)
            say(name)
            got = decode(q, kn, vn, seg, lens, Hq=Hq, Hkv=Hkv, D=D, H=0, block=0, dtype=dtype, remote_lens=rl, sync_override=sync)
            ref = oracle.decode_step(q, kf, vc, seg, lens, is_sync=bool(sync), remote_lens=rl)
            sane = others if what == "V" else np.ones(N, dtype=bool)
            check(got[sane], ref[sane], dtype, name)
            if what == "V":
                assert not np.isfinite(got[1]).any(), name
