"""Allocator kernels at their edges, mirrored on the oracle through ``Twin``
(tables, refcounts, ring and counters exact after every call): a full batch
that leaves one shared tail in one call (the last member appends in place),
requests of several wavefronts' blocks, mixed with requests that need none,
and releases of states on both sides of the wide form, whole and truncated.
A host that is wrong about a tail's holders is told so.
"""
import pytest
import torch

import synth
from paper_2607_10987_amd import kvstate as kv
from twin import Twin

pytestmark = pytest.mark.gpu


def small():
    return synth.ModelShape("meta", 1, 16, 1, 1, 16, 2, "f32")


def test_full_batch_leaves_one_tail(gpu_available):
    tw = Twin(small(), n_blocks=700, max_pos=64, max_states=70, wl="meta", check_kv=False)
    root = tw.materialize(5)                  # a half-full tail
    kids = tw.fork(root, 63)
    tw.attend(kids + [root], 1)               # 63 copies, then the last holder in place
    tw.attend(kids[:40], 4)                   # two or three new blocks each
    tw.attend(kids[30:50] + [root], 1)        # some need a block, some do not
    tw.evict(0)
    tw.close()


@pytest.mark.parametrize("n", [256, 1536, 1538, 4100])
def test_release_of_long_states(gpu_available, n):
    """n / 2 blocks: one round of the narrow form, its most (768 blocks), one
    block more, several rounds of the wide form."""
    tw = Twin(small(), n_blocks=n // 2 + 400, max_pos=n + 300, max_states=12, wl=f"rel{n}",
              check_kv=False)
    root = tw.materialize(n)
    kids = tw.fork(root, 3)
    tw.attend(kids, 129)                      # 64 or 65 blocks in one request
    tw.evict_truncate(tw.orc.allocated() - 70)
    tw.evict(tw.orc.allocated() - 1)
    tw.evict(0)
    tw.close()


def test_append_in_place_to_a_tail_that_a_later_member_leaves(gpu_available):
    """The device's check of the host's copy-on-write decisions takes the
    requests in their order.  The first member's tail entry is made to name a
    block that another state and the second member hold: the host appends to it
    in place, which the other state would see; that the second member's copy
    then leaves it does not make it private."""
    s, B, P, n = small(), 2, 40, 3
    cfg = kv.make_cfg(s.n_layers, s.d_model, s.n_q_heads, s.n_kv_heads, s.head_dim, B, "f32", 16, 8)
    pool = kv.Pool(cfg, P, kv.kv_scratch_bytes(cfg, 16, 2, 16))
    w = torch.randn(1, s.qkv_cols, s.d_model, device="cuda")
    pool.set_weights(w, w[0].numel())
    x = torch.randn(n, s.d_model, device="cuda")
    o = torch.empty(1, n, s.n_q_heads * s.head_dim, device="cuda")
    own, root = (kv.kv_materialize(pool.h, x, n, 0, o) for _ in range(2))
    kid = kv.kv_fork(pool.h, root, 1)[0]

    def attend(states):
        xa = torch.randn(len(states), s.d_model, device="cuda")
        kv.kv_attend(pool.h, states, xa, 1, torch.empty(1, len(states), 1, o.shape[-1],
                                                        device="cuda"))

    # metadata: header (256 bytes), refcounts, ring, then the tables
    align = lambda v: -(-v // 256) * 256
    off = align(align(256 + 4 * P) + 4 * P)
    tables = pool.meta_t[off:off + 8 * 8 * 4].view(torch.int32).view(8, 8)
    slot = own & 0xFFFFFFFF
    assert tables[slot, :2].tolist() == kv.kv_read_block_table(pool.h, own)
    tables[slot, 1] = kv.kv_read_block_table(pool.h, root)[1]
    torch.cuda.synchronize()
    attend([own, kid])
    with pytest.raises(kv.KVError) as e:
        kv.kv_sync(pool.h)
    assert e.value.status == kv.KV_ERR_INTERNAL
    pool.close()
