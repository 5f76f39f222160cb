"""The entry point that allocates nothing (cocktail_decode_attention_static) against cocktail_decode_attention.

Collected last on purpose (the file name sorts behind the other test files): it is the only test that uses the
workspace built into the library, and a failure here must not hide the parity tests.
"""
import numpy as np
import pytest
import torch

import workloads
import paper_2503_23294_amd as ck
from paper_2503_23294_amd import _lib

TOL = 2e-3      # max_d |a - b| / max_d |b| per (sequence, query head): the bar of the parity tests


def _prepare(w, workers, dev):
    shape = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = np.concatenate(workloads.chunk_bits(w))
    plan = ck.cocktail_plan(shape, w.seq_lens, bits, workers)
    cache = ck.PackedCache(plan, dev)
    k, v = workloads.kv_flat(w, 0)
    ck.cocktail_reorder_quantize(cache, torch.from_numpy(k).to(dev), torch.from_numpy(v).to(dev), ragged=True)
    q = torch.from_numpy(workloads.query(w, 0)).to(dev)
    return cache, q


@pytest.mark.gpu
@pytest.mark.parametrize("rep", [1, 4, 8, 16])
def test_static_workspace_entry_point_matches_the_regular_one(rep):
    assert torch.cuda.is_available(), "this test needs the MI355X"
    dev = torch.device("cuda:0")
    # two calls in a row on the library's one workspace, the second with a smaller input: whatever the first
    # call left there must not leak into the second
    big = workloads.small(f"static_big_r{rep}", 3, 2 * rep, 2, [5000, 2100, 3300], 64, 32, mix=(0.2, 0.4, 0.4),
                          seed_offset=800 + rep)
    small = workloads.small(f"static_small_r{rep}", 1, 2 * rep, 2, [64 * 3 + 11], 32, 32, mix=(0.3, 0.3, 0.4),
                            seed_offset=810 + rep)
    for w, workers in ((big, 48), (small, 5)):
        print(f"[no-alloc] {w.name}", flush=True)
        cache, q = _prepare(w, workers, dev)
        assert int(cache.plan.sizes.workspace_bytes) <= _lib.STATIC_WORKSPACE_BYTES
        ref, ref_lse = ck.cocktail_decode_attention(cache, q)
        ck.cocktail_decode_check(cache)
        out = torch.full_like(ref, float("nan"))
        lse = torch.full_like(ref_lse, float("nan"))
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        ck.cocktail_decode_attention_static(cache, q, 0.0, out, lse)
        assert torch.cuda.memory_allocated() == before
        ck.cocktail_decode_check(cache, static_workspace=True)      # also waits for the stream
        a, b = out.float(), ref.float()
        err = ((a - b).abs().amax(dim=2) / b.abs().amax(dim=2)).max().item()
        assert np.isfinite(err) and err <= TOL, f"{w.name}: max relative deviation {err:.3e}"
        assert torch.allclose(lse, ref_lse, rtol=0, atol=1e-4 * max(1.0, float(ref_lse.abs().max())))
        # the regular entry point still works after it, on its own workspace
        again, _ = ck.cocktail_decode_attention(cache, q)
        torch.cuda.synchronize()
        err = ((again.float() - b).abs().amax(dim=2) / b.abs().amax(dim=2)).max().item()
        assert err <= TOL


@pytest.mark.gpu
@pytest.mark.parametrize("rep,kv_heads,batch,tokens,chunk", [(8, 8, 128, 64, 16), (62, 32, 8, 50, 256)])
def test_static_workspace_beyond_16_mib_is_as_good_as_the_callers(rep, kv_heads, batch, tokens, chunk):
    """Plans that need more than COCKTAIL_STATIC_WORKSPACE_BYTES and are accepted (five to eight heads per wave: no
    pools, the same bits; twin sets, with pools): the same as on a workspace of the caller's, in calls that follow each other."""
    dev = torch.device("cuda:0")
    w = workloads.small(f"static_r{rep}", batch, rep * kv_heads, kv_heads, [tokens] * batch, chunk, 32,
                        mix=(0.25, 0.25, 0.25, 0.25), seed_offset=820 + rep)
    print(f"[no-alloc] {w.name}", flush=True)
    shape = ck.make_shape(w.batch, w.num_q_heads, w.num_kv_heads, w.head_dim, w.chunk_size, w.group_size)
    bits = np.tile(np.array([2, 4, 8, 16], np.uint8), batch) if tokens == 4 * chunk else np.zeros(0, np.uint8)
    cache = ck.PackedCache(ck.cocktail_plan(shape, w.seq_lens, bits, 2048), dev)
    assert _lib.STATIC_WORKSPACE_BYTES < int(cache.plan.sizes.workspace_bytes) <= 24 << 20, cache.plan.sizes.workspace_bytes
    ck.cocktail_reorder_quantize(cache, *(torch.from_numpy(x).to(dev) for x in workloads.kv_flat(w, 0, threads=8)), ragged=True)
    q = torch.from_numpy(workloads.query(w, 0)).to(dev)
    ref, ref_lse = ck.cocktail_decode_attention(cache, q)
    for _ in range(2):
        out, lse = torch.full_like(ref, float("nan")), torch.full_like(ref_lse, float("nan"))
        ck.cocktail_decode_attention_static(cache, q, 0.0, out, lse)
        ck.cocktail_decode_check(cache, static_workspace=True)
        assert torch.isfinite(lse).all() and torch.allclose(lse, ref_lse, rtol=0, atol=1e-4 * max(1.0, float(ref_lse.abs().max())))
        a, b = out.float(), ref.float()
        assert ((a - b).abs().amax(dim=2) / b.abs().amax(dim=2)).max().item() <= TOL
        assert rep != 8 or torch.equal(out, ref) and torch.equal(lse, ref_lse)


def test_static_workspace_entry_point_rejects_plans_beyond_its_size():
    """Host-side check, before any HIP call: runs without a GPU."""
    import ctypes as C
    sh = ck.make_shape(1, 1, 1, 128, 4096, 32)
    plan = ck.cocktail_plan(sh, [4096 * 640], np.full(640, 4, np.uint8), 1 << 15)   # 40960 blocks: a partial per worker
    assert int(plan.sizes.workspace_bytes) > _lib.STATIC_WORKSPACE_BYTES
    cache = _lib.Cache()
    cache.plan_host = plan.blob.ctypes.data
    cache.plan_dev = 4096
    L = _lib.lib()
    assert L.cocktail_decode_attention_static(C.byref(sh), 16, C.byref(cache), 0.0, 16, None, None) == _lib.ENOSPACE
    assert b"built-in" in L.cocktail_last_error()
    assert L.cocktail_decode_attention_static(C.byref(sh), None, C.byref(cache), 0.0, 16, None, None) == _lib.EINVAL


@pytest.mark.parametrize("rep,accepted", [(8, True), (4, False)])
def test_static_workspace_holds_the_partial_states_of_eight_heads_per_wave(rep, accepted):
    """Plans with eight heads per wave have 2048 workers, 1024 more than their workspace was sized for at first: what needs
    up to 24 MiB is not refused.  q is misaligned, so that the call ends with an error in any case, also on a GPU."""
    import ctypes as C
    sh = ck.make_shape(84, 8 * rep, 8, 128, 64, 32)
    bits = np.tile(np.repeat(np.array([2, 4, 8, 16], np.uint8), 4), sh.batch)
    plan = ck.cocktail_plan(sh, [16 * 64] * sh.batch, bits, 2048 if rep == 8 else 8192)
    need = int(plan.sizes.workspace_bytes)
    assert _lib.STATIC_WORKSPACE_BYTES < need <= 24 << 20, need
    cache = _lib.Cache()
    cache.plan_host = plan.blob.ctypes.data
    cache.plan_dev = 4096
    L = _lib.lib()
    rc = L.cocktail_decode_attention_static(C.byref(sh), 8, C.byref(cache), 0.0, 16, None, None)
    assert rc != 0 and (rc != _lib.ENOSPACE) == accepted, rc


@pytest.mark.parametrize("rep,kv_heads,accepted", [(62, 32, True), (13, 32, False)])
def test_static_workspace_holds_the_partial_states_of_twin_sets(rep, kv_heads, accepted):
    """Sets of query heads that are planned as twins have more partial states than sets that are cut one after the other (62
    heads in sets of two: 12.7 MiB then, 17 MiB as twins): such a plan is not refused.  A ratio without sets keeps the common
    limit.  q is misaligned, so that the call ends with an error in any case, also on a GPU."""
    import ctypes as C
    sh = ck.make_shape(8 if accepted else 6, kv_heads * rep, kv_heads, 128, 256, 32)
    plan = ck.cocktail_plan(sh, [50] * sh.batch if accepted else [50 * 64] * sh.batch,
                            [] if accepted else np.full(12 * sh.batch, 4, np.uint8), 2048 if accepted else 1 << 15)
    need = int(plan.sizes.workspace_bytes)
    assert _lib.STATIC_WORKSPACE_BYTES < need <= 24 << 20, need
    cache = _lib.Cache()
    cache.plan_host = plan.blob.ctypes.data
    cache.plan_dev = 4096
    rc = _lib.lib().cocktail_decode_attention_static(C.byref(sh), 8, C.byref(cache), 0.0, 16, None, None)
    assert rc != 0 and (rc != _lib.ENOSPACE) == accepted, rc
