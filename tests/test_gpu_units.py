"""GPU parity of the split-key attention where members diverge inside a chunk.

The work plan cuts a chunk at the block where the members of a group diverge;
each case is mirrored on the float64 oracle through ``Twin`` (outputs within
the tolerance stated there).  The cases put the divergence at the edges: in
the first block of the context, right at and right after a chunk border, a
fork of a fork inside one chunk, members whose histories share nothing, key
counts that end one key into a block, and units on both sides of the 32 query
vectors that separate the two kernels.
"""
import ctypes

import numpy as np
import pytest
import torch

import synth
from oracle import apply_rope, attention_rows, project_q
from paper_2607_10987_amd import kvstate as kv
from twin import Twin, close, to_np

pytestmark = pytest.mark.gpu


def shape8b(L=2):
    b = synth.LLAMA8B_SHAPE
    return synth.ModelShape("8b", L, b.d_model, b.n_q_heads, b.n_kv_heads, b.head_dim,
                            b.block_size, "bf16")


def context(tw, n, tag):
    nb = -(-n // tw.s.block_size)
    return tw.unpack(*tw.synthetic_transfer(nb, n, 0, tag=tag))


@pytest.mark.parametrize("n_ctx,agents,T", [
    (5, 9, 1),        # every member copies the only block: nothing shared
    (16, 17, 1),      # one whole block shared, below the shared-keys threshold or above it
    (1023, 20, 1),    # the new token completes the last block
    (1024, 20, 1),    # the new token opens a block
    (1041, 33, 1),    # 132 query vectors: eight wavefronts
    (2100, 8, 4),     # 128 query vectors of 4 tokens each
    (1701, 3, 7),     # appends over a ragged shared tail
    (1610, 1, 32),    # a batch of one, tokens crossing several blocks
    (90, 3, 5),       # too short a context for the split-key path
])
def test_divergence_inside_a_chunk(gpu_available, n_ctx, agents, T):
    shape = shape8b()
    tw = Twin(shape, n_blocks=-(-n_ctx // 16) + agents * 8 + 8, max_pos=n_ctx + 128,
              max_states=agents + 4, wl="units", check_kv=False)
    root = context(tw, n_ctx, 5)
    kids = tw.fork(root, agents)
    tw.attend(kids, T)
    tw.attend(kids, 1)
    tw.attend(kids[::2], T)                 # histories of different lengths
    tw.attend(kids, 1)
    tw.close()


def test_nested_forks_and_unrelated_members(gpu_available):
    """A fork of a fork that diverges in the same chunk, next to states of
    other contexts, one of them shorter than the others' common part."""
    tw = Twin(shape8b(), n_blocks=400, max_pos=2600, max_states=60, wl="nest", check_kv=False)
    root = context(tw, 1900, 6)
    branches = tw.fork(root, 3)
    tw.attend(branches, 20)
    leaves = [k for b in branches for k in tw.fork(b, 4)]
    other = context(tw, 40, 7)
    others = tw.fork(other, 5)
    tw.attend(leaves, 1)
    tw.attend(leaves + others, 1)           # 17 members: 68 query vectors, groups of 12 and 5
    tw.attend(leaves[:5] + others[:3], 3)
    tw.attend(others + leaves[::3] + [root], 1)
    tw.close()


@pytest.mark.parametrize("n_ctx,agents,T", [
    (63, 10, 16),     # less than a tile shared: a workgroup per sequence
    (64, 11, 16),     # one whole tile shared by four sequences; a last workgroup of three
    (200, 9, 32),     # two sequences a workgroup, a whole token group each
    (1000, 21, 3),    # 21 sequences of 3 tokens in one workgroup
    (130, 33, 2),     # the most sequences per workgroup, and one left over
])
def test_packed_appends(gpu_available, n_ctx, agents, T):
    """More than 128 query vectors of several sequences of few tokens: rows of
    whole sequences share a workgroup.  Twice from a common context (the
    second time over private tails), then with members of other contexts."""
    tw = Twin(shape8b(16), n_blocks=-(-n_ctx // 16) * 2 + agents * 12 + 16, max_pos=n_ctx + 128,
              max_states=agents + 8, wl="packed", check_kv=False)
    root = context(tw, n_ctx, 8)
    kids = tw.fork(root, agents)
    tw.attend(kids, T)
    tw.attend(kids, T)
    other = context(tw, n_ctx // 2 + 1, 9)
    pair = tw.fork(other, 2)
    tw.attend(kids[:agents - 2] + pair, T)
    tw.close()


@pytest.mark.parametrize("hq,T", [(32, 20), (64, 9)])
def test_packed_appends_that_share_little(gpu_available, hq, T):
    """Packs are decided one by one: three forks of one context are taken as
    one, members of unrelated contexts (63 to 411 keys, the last one alone in
    its pack) in workgroups of their own of the same launch, and so are forks
    whose private part outweighs the common one."""
    shape = synth.ModelShape("8b-s", 16, 512, hq, 8, 128, 16, "bf16")
    tw = Twin(shape, n_blocks=400, max_pos=700, max_states=40, wl="little", check_kv=False)
    roots = [context(tw, n, 20 + i) for i, n in enumerate((411, 63, 64, 200, 130))]
    forks = tw.fork(roots[0], 3)
    tw.attend(forks + roots[1:], T)                  # 3 | 3 | 1 at either T
    tw.attend(roots[1:] + forks, T)                  # no pack shares anything but the last
    short = tw.fork(roots[1], 4)
    tw.attend(short, 130)                            # 130 private keys after 63 common ones
    tw.attend(short + forks, T)
    tw.close()


def area_for(cfg, agents, T, keys, groups):
    """The largest work area in which the call takes its wide form in layer
    groups of `groups` layers (asked of the library), and the form's path."""
    out = (ctypes.c_int64 * 8)()
    f = kv.lib().kvs_query_append
    f.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32,
                  ctypes.c_size_t, ctypes.c_void_p]
    lo, hi, found = 0, 1 << 32, None
    while hi - lo > 256:                       # layers per group grow with the area
        mid = (lo + hi) // 2
        assert f(ctypes.byref(cfg), agents, T, keys, mid, out) == 0
        if out[0] <= groups:
            lo = mid
            if out[0] == groups and out[2] == 1:
                found = (mid, out[3])
        else:
            hi = mid
    return found


@pytest.mark.parametrize("L,hq,hkv,n_ctx,agents,T,path", [
    (4, 4, 1, 2100, 24, 1, 3),                 # split-key decode: units and late masks
    (4, 8, 1, 2100, 16, 1, 3),
    (32, 32, 8, 600, 9, 20, 2),                # packed appends: the packs' shared keys
])
@pytest.mark.parametrize("part", [1, 3])
def test_layer_groups_of_the_wide_forms(gpu_available, L, hq, hkv, n_ctx, agents, T, path, part):
    """What the first layer group works out once serves the later ones: a
    quarter or three quarters of the layers at once, against the float64
    oracle."""
    shape = synth.ModelShape("8b-g", L, 512, hq, hkv, 128, 16, "bf16")
    groups = part * L // 4
    cfg = kv.make_cfg(L, 512, hq, hkv, 128, 16, "bf16", n_ctx + 128, agents + 4)
    area, got = area_for(cfg, agents, T, n_ctx + 2 * T, groups)
    assert got == path
    tw = Twin(shape, n_blocks=-(-n_ctx // 16) + agents * 8 + 8, max_pos=n_ctx + 128,
              max_states=agents + 4, wl="lgw", check_kv=False, scratch_bytes=area)
    kids = tw.fork(context(tw, n_ctx, 31), agents)
    kv.kv_profile_enable(tw.gpu.h, True)
    for i in range(2):
        tw.attend(kids, T)
        prof = kv.kv_profile_read(tw.gpu.h)
        n = -(-L // groups)
        assert prof["attn_decode" if T == 1 else "attn"][0] == n, prof
        assert prof["merge"][0] == (n if path == 3 else 0), prof
    tw.close()


def test_full_batch_over_one_large_chunk(gpu_available):
    """64 agents x 4 query heads over 10111 keys, 32 layers of 8 KV heads: the
    chunk that would hold all keys has more block ids (64 members x 640) than
    the plan kernel's LDS takes.  Outputs of three members in the first and the
    last layer against the float64 oracle's attention over the keys and values
    that the device stored (tolerances of ``Twin``)."""
    L, d, hq, hkv, dh, B, n_ctx, A = 32, 256, 32, 8, 128, 16, 10110, 64
    cols, nb = (hq + 2 * hkv) * dh, -(-10110 // 16)
    cfg = kv.make_cfg(L, d, hq, hkv, dh, B, "bf16", 10240, 70)
    pool = kv.Pool(cfg, nb + A * 2 + 4, kv.kv_scratch_bytes(cfg, A, A, n_ctx + 2))
    gen = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    w = normal(L, cols, d) * d ** -0.5
    pool.set_weights(w, cols * d)
    h = kv.kv_pack_header()
    h.magic, h.version, h.model_id, h.cfg = kv.KV_PACK_MAGIC, kv.KV_PACK_VERSION, cfg.model_id, cfg
    h.n_tokens, h.n_blocks, h.block_bytes = n_ctx, nb, L * 2 * hkv * B * dh * 2
    h.payload_bytes = nb * h.block_bytes
    root = kv.kv_unpack(pool.h, h, normal(nb, L, 2, hkv, B, dh))
    kids = kv.kv_fork(pool.h, root, A)
    for step in range(2):                  # a private tail of one key, then of two
        x = normal(A, d)
        o = torch.empty((L, A, 1, hq * dh), dtype=torch.bfloat16, device="cuda")
        kv.kv_attend(pool.h, kids, x, 1, o)
        kv.kv_sync(pool.h)
        assert torch.isfinite(o).all()
        n = n_ctx + step + 1
        pos = np.full(hq, n - 1)
        for layer in (0, L - 1):
            q = project_q(to_np(x), to_np(w[layer]), hq, hkv, dh)
            for m in (0, 37, 63):
                table = kv.kv_read_block_table(pool.h, kids[m])
                t = pool.blocks_view()[table, layer].permute(1, 2, 0, 3, 4)
                k, v = (to_np(u.reshape(hkv, -1, dh)[:, :n]) for u in t)
                qr = apply_rope(q[m][:, None, :], np.full(1, n - 1), 10000.0)[:, 0, :]
                want = attention_rows(qr, k, v, pos, np.arange(n), np.arange(hq) // (hq // hkv))
                close(to_np(o[layer, m, 0]), want.reshape(-1), "bf16", f"layer {layer} agent {m}")
    pool.close()
