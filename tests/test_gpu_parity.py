"""Device library vs the float64 oracle, on the GPU, through the C ABI.

Every step compares block tables, refcounts and the free ring bit-exactly and
attention outputs / pool contents within the stated tolerances (see twin.py).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import OracleError, Status
from paper_2607_10987_amd import kvstate as kv
from twin import Twin, close, to_np

pytestmark = pytest.mark.gpu


def small_shape(dtype="f32", B=2, dh=16, L=1, d=32, hq=2, hkv=1):
    return synth.ModelShape("small", L, d, hq, hkv, dh, B, dtype)


def test_tiny_workload(gpu_available):
    """The 256-token / 2-agent / compose / 8-decode workload, float32, in full."""
    wl = synth.WORKLOADS["tiny"]
    tw = Twin(wl.shape, n_blocks=64, max_pos=512, wl="tiny")
    root = tw.materialize(wl.context)
    a1, a2 = tw.fork(root, wl.agents)
    tw.attend([a1, a2], wl.suffix)
    # [shared 0..255 | agent 1 256..287 | agent 2 256..287 shifted by +32]
    c = tw.compose([(root, 0, 256), (a1, 256, 288), (a2, 256, 288)])
    for _ in range(wl.decode):
        tw.attend([c], 1)
    n = kv.kv_state_info(tw.gpu.h, c)["n_blocks"]
    hdr, ohdr, buf, pay = tw.pack(c, 0, n)
    u = tw.unpack(hdr, ohdr, buf, pay, rerotated_from=c)
    tw.attend([u, a1], 3)
    tw.close()


def test_allocator_hand_trace_on_device(gpu_available):
    tw = Twin(small_shape(), n_blocks=8, max_pos=64, wl="trace")
    s0 = tw.materialize(5)
    s1, s2 = tw.fork(s0, 2)
    tw.attend([s1], 1)
    tw.attend([s2, s0], 2)
    tw.release(s1)
    s3 = tw.compose([(s2, 0, 5), (s0, 4, 7)])
    assert kv.kv_read_block_table(tw.gpu.h, s3) == [0, 1, 7, 3]
    assert tw.evict(5) == 2
    with pytest.raises(kv.KVError) as e:
        kv.kv_fork(tw.gpu.h, s2, 1)
    assert e.value.status == kv.KV_ERR_EVICTED
    tw.close()


def test_evict_truncate_on_device(gpu_available):
    """Truncation to the shared prefix, then a resume of a truncated state:
    tables, refcounts, ring and the attention output match the oracle."""
    tw = Twin(small_shape(), n_blocks=16, max_pos=64, wl="trunc")
    s0 = tw.materialize(4)
    c1, c2 = tw.fork(s0, 2)
    tw.attend([c1], 3)
    tw.attend([c2], 1)
    s3 = tw.materialize(3)
    assert tw.evict_truncate(3) == (1, 2)
    assert kv.kv_read_block_table(tw.gpu.h, c1) == [0, 1]
    with pytest.raises(kv.KVError) as e:
        kv.kv_fork(tw.gpu.h, s3, 1)
    assert e.value.status == kv.KV_ERR_EVICTED
    tw.attend([c1, c2], 2)
    # a shared partial tail: both holders keep only the whole shared blocks
    r = tw.materialize(5)
    k, = tw.fork(r, 1)
    tw.attend([k], 1)
    kv.kv_pin(tw.gpu.h, c1, 1)
    tw.orc.pin(tw.sid[c1], True)
    kv.kv_pin(tw.gpu.h, c2, 1)
    tw.orc.pin(tw.sid[c2], True)
    tw.evict_truncate(0)
    tw.attend([r, k], 1)
    tw.close()


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_sequences_on_device(gpu_available, seed):
    rng = np.random.default_rng(seed)
    order = rng.permutation(40)
    tw = Twin(small_shape(B=4), n_blocks=40, max_pos=96, max_states=10, seed=seed,
              wl="random", order=order)
    handles = []
    for step in range(40):
        live = [h for h in handles if tw.orc.states[tw.sid[h]].status == "ACTIVE"]
        op = int(rng.integers(0, 8)) if live else 0
        try:
            if op == 0:
                handles.append(tw.materialize(int(rng.integers(1, 12)),
                                              pos0=int(rng.integers(0, 20))))
            elif op == 1:
                handles += tw.fork(live[rng.integers(len(live))], int(rng.integers(1, 3)))
            elif op == 2:
                k = int(rng.integers(1, min(3, len(live)) + 1))
                pick = list(rng.choice(len(live), k, replace=False))
                tw.attend([live[i] for i in pick], int(rng.integers(1, 7)))
            elif op == 3:
                segs = []
                for _ in range(int(rng.integers(1, 4))):
                    h = live[rng.integers(len(live))]
                    n = kv.kv_state_info(tw.gpu.h, h)["n_tokens"]
                    a = int(rng.integers(0, n))
                    segs.append((h, a, int(rng.integers(a + 1, n + 1))))
                handles.append(tw.compose(segs))
            elif op == 4:
                h = live[rng.integers(len(live))]
                nb = kv.kv_state_info(tw.gpu.h, h)["n_blocks"]
                b0 = int(rng.integers(0, nb))
                hdr, ohdr, buf, pay = tw.pack(h, b0, nb)
                handles.append(tw.unpack(hdr, ohdr, buf, pay,
                                         rerotated_from=h if h in tw.rerot else None))
            elif op == 5:
                tw.evict(int(rng.integers(0, 40)))
            elif op == 6:
                tw.evict_truncate(int(rng.integers(0, 40)))
            else:
                tw.release(live[rng.integers(len(live))])
        except kv.KVError as e:
            # the oracle must refuse the same call with the same status; its
            # state is unchanged, so the device tables must still match
            assert e.status in (kv.KV_ERR_OOM, kv.KV_ERR_CAPACITY), e
            tw.check_meta()
    tw.close()


def test_bf16_llama_shape_two_layers(gpu_available):
    """8B-shaped heads (32 q / 8 kv, dh 128, B 16), 2 layers, ragged lengths."""
    shape = synth.LLAMA8B_SHAPE
    shape = synth.ModelShape("8b-l2", 2, shape.d_model, shape.n_q_heads, shape.n_kv_heads,
                             shape.head_dim, shape.block_size, "bf16")
    tw = Twin(shape, n_blocks=160, max_pos=2048, wl="mid")
    root = tw.materialize(1000)                    # 1000 mod 16 = 8: partial tail
    kids = tw.fork(root, 3)
    tw.attend(kids, 100)                           # copy-on-write of the shared tail
    for _ in range(3):
        tw.attend(kids, 1)                         # batched decode
    c = tw.compose([(root, 0, 1000), (kids[0], 1000, 1100), (kids[1], 1000, 1100)])
    tw.attend([c], 1)
    hdr, ohdr, buf, pay = tw.pack(c, 2, 40)
    tw.unpack(hdr, ohdr, buf, pay, rerotated_from=c)
    tw.close()


def test_bf16_70b_heads_two_layers(gpu_available):
    """70B-shaped heads (d_model 8192, 64 q / 8 kv heads: 8 query heads per KV
    head, dh 128, blocks of 32), 2 layers, element by element: a ragged
    materialize, batched decode of four forks (token rows staged in two
    column chunks of the decode-size projection), a 40-token append of two
    of them, a compose and a pack / unpack of it."""
    base = synth.LLAMA70B_SHAPE
    shape = synth.ModelShape("70b-l2", 2, base.d_model, base.n_q_heads, base.n_kv_heads,
                             base.head_dim, base.block_size, "bf16")
    tw = Twin(shape, n_blocks=64, max_pos=512, max_states=12, wl="70b")
    root = tw.materialize(300)                     # 300 mod 32 = 12: partial tail
    kids = tw.fork(root, 4)
    for _ in range(2):
        tw.attend(kids, 1)
    tw.attend(kids[:2], 40)
    c = tw.compose([(root, 0, 300), (kids[0], 300, 342), (kids[3], 300, 302)])
    tw.attend([c], 1)
    nb = kv.kv_state_info(tw.gpu.h, c)["n_blocks"]
    hdr, ohdr, buf, pay = tw.pack(c, 0, nb)
    tw.unpack(hdr, ohdr, buf, pay, rerotated_from=c)
    tw.close()


def test_pack_unpack_bit_exact_round_trips(gpu_available):
    for dtype in ("f32", "bf16"):
        shape = small_shape(dtype, B=4, dh=32, L=3, hq=4, hkv=2)
        order = np.random.default_rng(5).permutation(32)
        tw = Twin(shape, n_blocks=32, max_pos=128, wl="rt" + dtype, order=order)
        # a seeded payload: both sides hold identical stored values
        hdr, ohdr, buf, pay = tw.synthetic_transfer(5, 18, 7, tag=1)
        u = tw.unpack(hdr, ohdr, buf, pay)
        hdr2, ohdr2, buf2, pay2 = tw.pack(u, 0, 5)
        # device bytes equal the oracle's values exactly (zero-filled tail slots)
        got = to_np(buf2.view(tw.tdt)).reshape(pay2.shape)
        assert np.array_equal(got, pay2)
        # device pack o unpack o pack is the identity on bytes, through a permuted pool
        v = kv.kv_unpack(tw.gpu.h, hdr2, buf2)
        buf3 = torch.empty_like(buf2)
        kv.kv_pack(tw.gpu.h, v, 0, 5, buf3)
        torch.cuda.synchronize()
        assert torch.equal(buf3, buf2)
        tw.close()


def test_pack_unpack_pinned_host_tier(gpu_available):
    """Pack to / unpack from pinned host memory (the host tier of a state):
    the same bytes as through device memory, and a round trip through the
    host gives back the same blocks.  Pageable host memory is rejected before
    anything is enqueued."""
    shape = small_shape("bf16", B=4, dh=32, L=3, hq=4, hkv=2)
    tw = Twin(shape, n_blocks=48, max_pos=128, wl="hosttier")
    hdr, ohdr, buf, pay = tw.synthetic_transfer(5, 18, 7, tag=3)
    u = tw.unpack(hdr, ohdr, buf, pay)
    hdr_d, _, dev_buf, _ = tw.pack(u, 0, 5)          # device pack, checked against the oracle
    host = torch.empty(dev_buf.numel(), dtype=torch.uint8, pin_memory=True)
    hdr_h = kv.kv_pack(tw.gpu.h, u, 0, 5, host)
    torch.cuda.synchronize()
    assert torch.equal(host, dev_buf.cpu())
    assert bytes(hdr_h) == bytes(hdr_d)
    v = kv.kv_unpack(tw.gpu.h, hdr_h, host)
    again = torch.empty_like(dev_buf)
    kv.kv_pack(tw.gpu.h, v, 0, 5, again)
    torch.cuda.synchronize()
    assert torch.equal(again, dev_buf)
    before = kv.kv_pool_counts(tw.gpu.h)
    page = torch.empty(dev_buf.numel(), dtype=torch.uint8)  # pageable
    with pytest.raises(kv.KVError) as e:
        kv.kv_pack(tw.gpu.h, u, 0, 5, page)
    assert e.value.status == kv.KV_ERR_ARG
    with pytest.raises(kv.KVError) as e:
        kv.kv_unpack(tw.gpu.h, hdr_h, page)
    assert e.value.status == kv.KV_ERR_ARG
    assert kv.kv_pool_counts(tw.gpu.h) == before
    tw.close()


def test_error_codes_on_device(gpu_available):
    tw = Twin(small_shape(B=2), n_blocks=4, max_pos=16, max_states=3, wl="err")
    x = torch.zeros((16, 32), dtype=torch.float32, device="cuda")
    o = torch.zeros((1, 16, 32), dtype=torch.float32, device="cuda")
    with pytest.raises(kv.KVError) as e:
        kv.kv_materialize(tw.gpu.h, x, 9, 0, o)
    assert e.value.status == kv.KV_ERR_OOM
    assert kv.kv_pool_counts(tw.gpu.h)["free_blocks"] == 4
    s = tw.materialize(4)
    with pytest.raises(kv.KVError) as e:
        kv.kv_attend(tw.gpu.h, [s], x, 13, o)
    assert e.value.status == kv.KV_ERR_CAPACITY
    for k, code in ((0, kv.KV_ERR_ARG), (3, kv.KV_ERR_CAPACITY)):
        with pytest.raises(kv.KVError) as e:
            kv.kv_fork(tw.gpu.h, s, k)
        assert e.value.status == code
    with pytest.raises(kv.KVError) as e:
        kv.kv_attend(tw.gpu.h, [s, s], x, 1, o)
    assert e.value.status == kv.KV_ERR_ARG
    buf = torch.empty(2 * tw.s.block_bytes, dtype=torch.uint8, device="cuda")
    with pytest.raises(kv.KVError) as e:
        kv.kv_pack(tw.gpu.h, s, 0, 2, buf, dst_bytes=2 * tw.s.block_bytes - 1)
    assert e.value.status == kv.KV_ERR_BUFSIZE
    hdr = kv.kv_pack(tw.gpu.h, s, 0, 2, buf)
    for field, val, code in (("magic", 1, kv.KV_ERR_BAD_HEADER),
                             ("model_id", 99, kv.KV_ERR_INCOMPATIBLE),
                             ("n_tokens", 5, kv.KV_ERR_BAD_HEADER)):
        h2 = kv.kv_pack_header.from_buffer_copy(hdr)
        setattr(h2, field, val)
        with pytest.raises(kv.KVError) as e:
            kv.kv_unpack(tw.gpu.h, h2, buf)
        assert e.value.status == code
    h2 = kv.kv_pack_header.from_buffer_copy(hdr)
    h2.cfg.block_size = 4
    with pytest.raises(kv.KVError) as e:
        kv.kv_unpack(tw.gpu.h, h2, buf)
    assert e.value.status == kv.KV_ERR_INCOMPATIBLE
    with pytest.raises(kv.KVError) as e:
        kv.kv_unpack(tw.gpu.h, hdr, buf, src_bytes=hdr.payload_bytes - 1)
    assert e.value.status == kv.KV_ERR_BUFSIZE
    kv.kv_release(tw.gpu.h, s)
    with pytest.raises(kv.KVError) as e:
        kv.kv_pack(tw.gpu.h, s, 0, 1, buf)
    assert e.value.status == kv.KV_ERR_EVICTED
    kv.kv_sync(tw.gpu.h)
    tw.close()


def test_buffer_checks_before_any_launch(gpu_available):
    """The C ABI checks every device buffer before it launches anything:
    host memory and misaligned pointers are KV_ERR_ARG, an allocation that
    ends before the bytes the call needs is KV_ERR_BUFSIZE.  Exercised
    through kv_set_weights (which launches nothing) with raw addresses that
    bypass the binding's own tensor checks, and through the binding."""
    import ctypes
    import os
    shape = small_shape("bf16", B=16, dh=128, L=2, d=256, hq=4, hkv=2)
    tw = Twin(shape, n_blocks=8, max_pos=64, wl="bufchk")
    h = tw.gpu.h
    per = shape.qkv_cols * shape.d_model
    host = (ctypes.c_uint16 * (2 * per))()
    hip = ctypes.CDLL("libamdhip64.so.7", mode=os.RTLD_NOLOAD | os.RTLD_GLOBAL)
    base, size = ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipMemGetAddressRange(ctypes.byref(base), ctypes.byref(size),
                                     ctypes.c_void_p(tw.w_dev.data_ptr())) == 0
    near_end = (base.value + size.value - 4096) & ~15
    for ptr, code in ((ctypes.addressof(host), kv.KV_ERR_ARG),
                      (tw.w_dev.data_ptr() + 2, kv.KV_ERR_ARG),
                      (near_end, kv.KV_ERR_BUFSIZE)):
        assert kv.lib().kv_set_weights(h, ptr, per) == code
    # the binding refuses what the library would, before calling it
    with pytest.raises(kv.KVError) as e:
        kv.kv_set_weights(h, tw.w_dev.float(), per)
    assert e.value.status == kv.KV_ERR_ARG
    with pytest.raises(kv.KVError) as e:
        kv.kv_set_weights(h, tw.w_dev.reshape(-1)[:per], per)
    assert e.value.status == kv.KV_ERR_BUFSIZE
    # the weights set at construction are still in use: the pool works
    s = tw.materialize(20)
    tw.attend([s], 3)
    tw.close()


def test_bf16_fanout_decode_sixteen_agents(gpu_available):
    """16 agents x 4 query heads share a context: 64 query vectors per KV head in
    the shared units, private tails per agent, block boundaries crossed."""
    base = synth.LLAMA8B_SHAPE
    shape = synth.ModelShape("8b-l2", 2, base.d_model, base.n_q_heads, base.n_kv_heads,
                             base.head_dim, base.block_size, "bf16")
    tw = Twin(shape, n_blocks=200, max_pos=1200, max_states=24, wl="fan16", check_kv=False)
    root = tw.materialize(1030)                    # a ragged shared tail
    kids = tw.fork(root, 16)
    tw.attend(kids, 7)                             # copy-on-write of the shared tail
    for _ in range(2):
        tw.attend(kids, 1)
    tw.attend(kids[3:9], 1)                        # a sub-batch with longer histories
    tw.attend([root] + kids[:2], 1)
    tw.close()


def test_bf16_ragged_edges(gpu_available):
    """8B-shaped heads, 2 layers, at sizes that leave partial tiles in every
    kernel: a one-token state (decode-path kernels over a single key),
    prefills of 33 and 300 tokens (partial 256-row projection and 64-token
    attention tiles), decode batches of 3, 5 and 17 (17 agents x 4 query heads
    = 68 query vectors per KV head: four wavefronts of the MFMA decode path
    share each unit, and 17 token rows for the projection), appends of 2 x 33
    rows and of 70 rows behind 301 cached tokens, a three-segment compose and
    a pack / unpack of the result."""
    base = synth.LLAMA8B_SHAPE
    shape = synth.ModelShape("8b-l2", 2, base.d_model, base.n_q_heads, base.n_kv_heads,
                             base.head_dim, base.block_size, "bf16")
    tw = Twin(shape, n_blocks=220, max_pos=700, max_states=40, wl="ragged")
    one = tw.materialize(1)
    a = tw.materialize(33, pos0=5)
    b = tw.materialize(300)
    tw.attend([one, a, b], 1)
    kids = tw.fork(b, 17)
    tw.attend(kids, 1)                             # copy-on-write of b's partial tail
    tw.attend(kids[:5], 1)
    tw.attend([a, one], 33)
    tw.attend(kids[5:7], 70)
    c = tw.compose([(one, 0, 2), (a, 3, 30), (kids[0], 100, 302)])
    tw.attend([c], 1)
    nb = kv.kv_state_info(tw.gpu.h, c)["n_blocks"]
    hdr, ohdr, buf, pay = tw.pack(c, 0, nb)
    tw.unpack(hdr, ohdr, buf, pay, rerotated_from=c)
    tw.close()


def test_bf16_decode_batch_one_multichunk(gpu_available):
    """A batch of one decodes over its keys in chunks of its own (here 256 keys:
    decode steps over 1030 and 1031 keys span five, the last one ragged), so the
    split-key partials and their merge are compared with the oracle element by
    element; a batch of two over the same state and a fork of it is cut
    otherwise, then appends 3 tokens each (6 token rows: the decode-size
    projection with rows of two sequences)."""
    base = synth.LLAMA8B_SHAPE
    shape = synth.ModelShape("8b-l2", 2, base.d_model, base.n_q_heads, base.n_kv_heads,
                             base.head_dim, base.block_size, "bf16")
    tw = Twin(shape, n_blocks=160, max_pos=1100, max_states=8, wl="chunks")
    s = tw.materialize(1029)
    tw.attend([s], 1)
    tw.attend([s], 1)
    kid = tw.fork(s, 1)[0]
    tw.attend([s, kid], 1)
    tw.attend([s, kid], 3)      # 6 token rows, 3 per sequence, through the decode-size projection
    tw.close()


def test_api_maxima_on_device(gpu_available):
    """The largest calls the interface accepts: a fork into KV_MAX_FORK
    children, one attend over a batch of KV_MAX_BATCH states (each one
    copy-on-writes the shared partial tail), a compose of KV_MAX_SEGMENTS
    one-token segments with distinct shifts."""
    assert kv.KV_MAX_FORK == kv.KV_MAX_BATCH == kv.KV_MAX_SEGMENTS == 64
    tw = Twin(small_shape(B=4), n_blocks=200, max_pos=128, max_states=80, wl="max")
    root = tw.materialize(10)
    kids = tw.fork(root, kv.KV_MAX_FORK)
    tw.attend(kids, 1)
    c = tw.compose([(k, 10, 11) for k in kids[:kv.KV_MAX_SEGMENTS]])
    tw.attend([c], 2)
    with pytest.raises(kv.KVError) as e:
        kv.kv_fork(tw.gpu.h, root, kv.KV_MAX_FORK + 1)
    assert e.value.status in (kv.KV_ERR_ARG, kv.KV_ERR_CAPACITY)
    kv.kv_sync(tw.gpu.h)
    tw.close()
