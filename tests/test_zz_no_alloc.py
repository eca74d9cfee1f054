"""fedattn_decode_static (the decode entry point that allocates nothing and works in the
library's built-in scratch array) against fedattn_decode with a caller's workspace: two calls
in a row on one GPU, the second on a smaller problem, local and sync blocks.  Both entry
points run the same kernels, so the outputs must be bit-identical; the oracle bar is checked
as well."""
import gc

import numpy as np
import pytest
import torch

import fedattn_inputs as fi
import oracle
import paper_2511_02647_amd as fa
from gpu_util import check, dev, host, say

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


def _case(seed, N, cap, lens, Hq, Hkv, D):
    g = np.random.default_rng(seed)
    mk = lambda *s: fi.round_to_bf16(g.standard_normal(s).astype(np.float32))
    seg = (np.arange(N + 1) * cap).astype(np.int32)
    return seg, np.asarray(lens, dtype=np.int32), mk(N, Hq, D), mk(N * cap, Hkv, D), mk(N * cap, Hkv, D)


def test_decode_static_matches_decode_with_a_workspace():
    Hq, Hkv, D = 8, 2, 128
    cases = [_case(901, 6, 1500, [1500, 1, 700, 1333, 64, 65], Hq, Hkv, D),   # several chunks per segment
             _case(902, 3, 200, [200, 77, 130], Hq, Hkv, D)]                  # smaller problem, same array
    for ci, (seg, lens, q, kc, vc) in enumerate(cases):
        N = len(lens)
        p = fa.make_params(N, Hq, Hkv, D, 2, BF16)
        tq, tk, tv = dev(q, BF16), dev(kc, BF16), dev(vc, BF16)
        ws = torch.empty(fa.fedattn_workspace_bytes(p, fa.FEDATTN_OP_DECODE, int(seg[-1])), dtype=torch.uint8, device="cuda")
        prompt = np.minimum(lens, 100).astype(np.int32)
        for block, rl in [(0, None), (1, None), (1, prompt)]:
            sync = oracle.is_sync_block(2, block)
            want = torch.full_like(tq, float("nan"))
            fa.fedattn_decode(p, block, tq, tk, tv, want, seg, lens, remote_lens=rl, workspace=ws)
            got = torch.full_like(tq, float("nan"))
            say("decode_static call %d block %d (%s) remote=%s" % (ci, block, "sync" if sync else "local", rl is not None))
            gc.collect()       # tensors of earlier tests must not be released while we watch the allocator
            before, reserved = torch.cuda.memory_allocated(), torch.cuda.memory_reserved()
            fa.fedattn_decode_static(p, block, tq, tk, tv, got, seg, lens, remote_lens=rl)
            torch.cuda.synchronize()
            assert torch.cuda.memory_allocated() <= before and torch.cuda.memory_reserved() == reserved
            assert torch.equal(got, want), "static-scratch decode differs from the workspace decode (call %d, block %d)" % (ci, block)
            ref = oracle.decode_step(q, kc, vc, seg, lens, is_sync=sync, remote_lens=rl)
            check(host(got), ref, BF16, "decode_static call %d block %d remote=%s" % (ci, block, rl is not None))


def test_decode_static_rejects_problems_beyond_its_array():
    N, Hq, Hkv, D = 128, 64, 8, 128
    p = fa.make_params(N, Hq, Hkv, D, 1, BF16)
    seg = (np.arange(N + 1) * 64).astype(np.int32)
    assert fa.fedattn_workspace_bytes(p, fa.FEDATTN_OP_DECODE, int(seg[-1])) > fa.FEDATTN_STATIC_SCRATCH_BYTES
    t = torch.zeros(N, Hq, D, dtype=BF16, device="cuda")
    kv = torch.zeros(N * 64, Hkv, D, dtype=BF16, device="cuda")
    with pytest.raises(fa.FedAttnError) as e:
        fa.fedattn_decode_static(p, 0, t, kv, kv, torch.empty_like(t), seg, np.full(N, 64, np.int32))
    assert e.value.status == fa.FEDATTN_EWORKSPACE and "scratch" in str(e.value)
    torch.cuda.synchronize()


# (segment lengths, Hq, Hkv, D): partials of all KV heads beyond the built-in array; those of one head's columns beyond
# it (pieces of 64 columns, of 48); local blocks beyond it
PIECES = {"heads": ([65, 0, 1, 130] * 8, 32, 8, 128), "columns": ([70 + n % 60 for n in range(127)] + [0], 16, 4, 256),
          "few-columns": ([64 + n % 65 for n in range(128)], 4, 1, 256), "local": ([20 + n for n in range(128)], 64, 8, 256)}


@pytest.mark.parametrize("shape", sorted(PIECES))
@pytest.mark.parametrize("dtype", [torch.float32, BF16])
def test_decode_in_pieces(shape, dtype):
    """fp32 and bf16 with other head dimensions: blocks whose partials exceed the built-in array run in pieces, with a
    workspace (never larger than the array) and without one alike."""
    lens, Hq, Hkv, D = PIECES[shape]
    D = D if dtype == torch.float32 else D - 24
    N, lens = len(lens), np.asarray(lens, dtype=np.int32)
    seg = np.concatenate([[0], np.cumsum(lens + 1)]).astype(np.int32)
    g = np.random.default_rng(903)
    mk = lambda *s: (fi.round_to_bf16 if dtype == BF16 else (lambda x: x))(g.standard_normal(s).astype(np.float32))
    q, kc, vc = mk(N, Hq, D), mk(int(seg[-1]), Hkv, D), mk(int(seg[-1]), Hkv, D)
    p = fa.make_params(N, Hq, Hkv, D, 2, dtype)
    need = fa.fedattn_workspace_bytes(p, fa.FEDATTN_OP_DECODE, int(seg[-1]))
    assert need == fa.FEDATTN_STATIC_SCRATCH_BYTES      # the whole block would take more
    tq, tk, tv = dev(q, dtype), dev(kc, dtype), dev(vc, dtype)
    ws = torch.full((2 * need,), 255, dtype=torch.uint8, device="cuda")
    for block, rl in [(0, None), (1, None), (1, lens // 2)]:
        what = "decode pieces %s %s block %d remote=%s" % (shape, dtype, block, rl is not None)
        say(what)
        ref = oracle.decode_step(q, kc, vc, seg, lens, is_sync=oracle.is_sync_block(2, block), remote_lens=rl)
        outs = [torch.full_like(tq, float("nan")) for _ in range(4)]
        fa.fedattn_decode(p, block, tq, tk, tv, outs[0], seg, lens, remote_lens=rl, workspace=ws[:need])
        fa.fedattn_decode(p, block, tq, tk, tv, outs[1], seg, lens, remote_lens=rl, workspace=ws)
        fa.fedattn_decode_blocks_fused(p, block, 1, tq, tk, tv, outs[2], tq.numel(), tk.numel(), seg, lens, remote_lens=rl, workspace=ws)
        fa.fedattn_decode_static(p, block, tq, tk, tv, outs[3], seg, lens, remote_lens=rl)
        torch.cuda.synchronize()
        check(host(outs[0]), ref, dtype, what)
        for o in outs[1:]:
            assert torch.equal(o, outs[0]), what


def test_decode_pieces_of_several_blocks_and_more_heads_than_pieces_have_room_for():
    lens, Hq, Hkv, D = PIECES["heads"]
    N, M, lens = len(lens), 3, np.asarray(lens, dtype=np.int32)
    seg = np.concatenate([[0], np.cumsum(lens + 1)]).astype(np.int32)
    p = fa.make_params(N, Hq, Hkv, D, 2, torch.float32)
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    mk = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, k, v = mk(M, N, Hq, D), mk(M, int(seg[-1]), Hkv, D), mk(M, int(seg[-1]), Hkv, D)
    ws = torch.full((2 * fa.FEDATTN_STATIC_SCRATCH_BYTES,), 255, dtype=torch.uint8, device="cuda")   # two blocks in flight
    one, many = torch.zeros_like(q), torch.zeros_like(q)
    say("decode pieces, fused blocks")
    for b in range(M):
        fa.fedattn_decode_static(p, 1, q[b], k[b], v[b], one[b], seg, lens)
    fa.fedattn_decode_blocks_fused(p, 1, M, q, k, v, many, q[0].numel(), k[0].numel(), seg, lens, sync_override=1, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(one, many)
    # 17000 KV heads: no room for chunk counters beside the partials; one row per participant, so the output is V
    N, H = 128, 17000
    p = fa.make_params(N, H, H, 8, 0, torch.float32)
    seg = np.arange(N + 1, dtype=np.int32)
    q, k, v = mk(N, H, 8), mk(N, H, 8), mk(N, H, 8)
    say("decode, 17000 KV heads")
    for call in (lambda o: fa.fedattn_decode(p, 0, q, k, v, o, seg, np.ones(N, np.int32), workspace=ws),
                 lambda o: fa.fedattn_decode_static(p, 0, q, k, v, o, seg, np.ones(N, np.int32))):
        out = torch.full_like(q, float("nan"))
        call(out)
        torch.cuda.synchronize()
        assert torch.allclose(out, v, rtol=1e-6, atol=0)
