"""Non-finite values stay with the tokens that see them.

One agent of a batch gets inputs whose queries, keys and values overflow or
are NaN.  The outputs of every other agent must be what they are beside a
finite neighbour, bit for bit, on each attention path that takes several
agents in one workgroup or unit.
"""
import pytest
import torch

from paper_2607_10987_amd import kvstate as kv

pytestmark = pytest.mark.gpu

TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


class Agents:
    """A pool with one cached context of N(0, 1) keys and values."""

    def __init__(self, L, hq, hkv, dh, dt, n_ctx, agents, T, d=256, B=16):
        self.L, self.d, self.q, self.dt = L, d, hq * dh, TORCH[dt]
        self.gen = torch.Generator(device="cuda").manual_seed(3)
        cols, nb, n = (hq + 2 * hkv) * dh, -(-n_ctx // B), n_ctx + 4 * T
        cfg = kv.make_cfg(L, d, hq, hkv, dh, B, dt, n, 3 * agents + 8)
        self.pool = kv.Pool(cfg, nb + 3 * agents * (-(-3 * T // B) + 2) + 8,
                            kv.kv_scratch_bytes(cfg, agents * T, agents, n))
        self.w = self.normal(L, cols, d) * d ** -0.5
        self.pool.set_weights(self.w, cols * d)
        h = kv.kv_pack_header()
        h.magic, h.version, h.model_id, h.cfg = (kv.KV_PACK_MAGIC, kv.KV_PACK_VERSION,
                                                 cfg.model_id, cfg)
        blocks = self.normal(nb, L, 2, hkv, B, dh)
        h.n_tokens, h.n_blocks = n_ctx, nb
        h.block_bytes = blocks[0].numel() * blocks.element_size()
        h.payload_bytes = nb * h.block_bytes
        self.root = kv.kv_unpack(self.pool.h, h, blocks)
        self.agents, self.T = agents, T

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device="cuda", dtype=self.dt)

    def append(self, kids, x):
        o = torch.empty((self.L, len(kids), x.shape[1], self.q), dtype=self.dt, device="cuda")
        kv.kv_attend(self.pool.h, kids, x, x.shape[1], o)
        kv.kv_sync(self.pool.h)
        return o


def spoil(x, agent):
    """The agent's last token overflows, the one before (if any) is NaN."""
    y = x.clone()
    y[agent, -1] = 3e38
    if x.shape[1] > 1:
        y[agent, -2] = float("nan")
    return y


@pytest.mark.parametrize("L,hq,hkv,n_ctx,agents,T,what", [
    (32, 32, 8, 200, 9, 29, "packed: two agents a workgroup share a wavefront's rows"),
    (32, 32, 8, 130, 9, 32, "packed: a wavefront's rows are of one agent"),
    (32, 32, 8, 70, 11, 5, "packed: many agents a wavefront, one tile shared"),
    (32, 32, 8, 40, 11, 5, "packed launch, a workgroup per agent: less than a tile shared"),
    (32, 64, 8, 130, 8, 11, "packed: eight query heads"),
    (2, 32, 8, 2100, 8, 4, "split-key: appends"),
    (2, 32, 8, 1041, 33, 1, "split-key: decode, shared units and private tails"),
    (2, 32, 8, 700, 3, 70, "prefill: a workgroup per agent"),
    (1, 4, 2, 60, 3, 9, "portable (two query heads per KV head)"),
])
def test_agents_are_isolated(gpu_available, L, hq, hkv, n_ctx, agents, T, what):
    p = Agents(L, hq, hkv, 128, "bf16", n_ctx, agents, T)
    x, x2 = p.normal(agents, T, p.d), p.normal(agents, T, p.d)
    clean, kids = kv.kv_fork(p.pool.h, p.root, agents), kv.kv_fork(p.pool.h, p.root, agents)
    bad = agents // 2
    rest = [i for i in range(agents) if i != bad]
    a, b = p.append(clean, x), p.append(kids, spoil(x, bad))
    assert bool(torch.isfinite(a).all())
    assert bool(torch.isnan(b[:, bad, -1]).any()), "the spoiled inputs took no effect"
    same = torch.equal(a[:, rest], b[:, rest])
    assert same, what
    # a second append, over the private keys that hold the values
    a, b = p.append(clean, x2), p.append(kids, x2)
    same = torch.equal(a[:, rest], b[:, rest])
    assert same, what
    p.pool.close()


@pytest.mark.parametrize("hq,hkv,dh,dt", [(4, 2, 64, "f32"), (3, 1, 48, "f32"), (2, 2, 256, "f32"),
                                          (5, 1, 64, "bf16"), (3, 3, 112, "bf16"),
                                          (6, 2, 128, "bf16")])
@pytest.mark.parametrize("n_before,T,at", [(0, 20, 9), (5, 33, 32), (200, 7, 3), (300, 1, 0)])
def test_later_tokens_do_not_reach_earlier_ones(gpu_available, hq, hkv, dh, dt, n_before, T, at):
    """The portable attention: token `at` has infinite values (and finite
    queries and keys: input channel 0 feeds only the values).  Tokens before it
    keep their outputs, those from it on are not finite.  Up to the order of
    sums, which may differ in the tile of keys that holds the values: float32
    arithmetic within 2e-5, one bf16 rounding of it within 2^-8 of the value."""
    L, d, B = 2, 64, 16
    q, dtype, cols = hq * dh, TORCH[dt], (hq + 2 * hkv) * dh
    gen = torch.Generator(device="cuda").manual_seed(11)
    w = (torch.randn(L, cols, d, generator=gen, device="cuda") * d ** -0.5).to(dtype)
    w[:, :, 0] = 0
    w[:, (hq + hkv) * dh:, 0] = 16
    cfg = kv.make_cfg(L, d, hq, hkv, dh, B, dt, 400, 4)
    pool = kv.Pool(cfg, 64, kv.kv_scratch_bytes(cfg, 400, 1, 400))
    pool.set_weights(w, cols * d)
    x0 = torch.randn(max(n_before, 1), d, generator=gen, device="cuda").to(dtype)
    x = torch.randn(1, T, d, generator=gen, device="cuda").to(dtype)
    x0[:, 0] = x[:, :, 0] = 0
    bad = x.clone()
    bad[0, at, 0] = 3e38

    def outputs(xi):
        if n_before == 0:
            o = torch.empty((L, T, q), dtype=dtype, device="cuda")
            kv.kv_release(pool.h, kv.kv_materialize(pool.h, xi, T, 0, o))
            return o
        o0 = torch.empty((L, n_before, q), dtype=dtype, device="cuda")
        s = kv.kv_materialize(pool.h, x0, n_before, 0, o0)
        o = torch.empty((L, 1, T, q), dtype=dtype, device="cuda")
        kv.kv_attend(pool.h, [s], xi, T, o)
        kv.kv_release(pool.h, s)
        return o[:, 0]

    a, b = outputs(x).double(), outputs(bad).double()
    assert bool(torch.isfinite(a).all())
    # (the projection of head_dim 128 may store NaN for overflowing values)
    got = b[:, at:]
    assert bool((got == float("inf")).all() if dh != 128 else (~torch.isfinite(got)).all())
    err = (a[:, :at] - b[:, :at]).abs()
    bound = 2e-5 + (2.0 ** -8 * a[:, :at].abs() if dt == "bf16" else 0.0)
    assert bool((err <= bound).all()), float(err.max())
    pool.close()
