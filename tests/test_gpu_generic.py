"""GPU parity of the portable fp32 path at the edges of its tiles: 16 rotation
pairs, 16 or 64 token rows, 16 contraction indices per wavefront, 16 query
vectors, 16 keys, 1 to 16 wavefronts.  Every case is mirrored on the float64
oracle through ``Twin`` (its tolerances): head dimensions on both sides of each
template bound and not a multiple of 32, d_model that is not a multiple of 4
(element-wise loads), block sizes that are not powers of two, one to three
query heads per KV head, and enough layers for the 64-row tiles.
"""
import pytest

import synth
from twin import Twin

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,d,hq,hkv,dh,B,dt,ctx,agents,T", [
    (1, 64, 2, 1, 16, 1, "f32", 1, 2, 1),
    (1, 30, 3, 1, 48, 5, "f32", 17, 3, 5),
    (2, 131, 4, 4, 64, 7, "bf16", 33, 2, 16),
    (1, 256, 4, 2, 80, 16, "f32", 300, 4, 2),
    (2, 100, 2, 2, 128, 16, "f32", 128, 1, 65),
    (1, 96, 6, 2, 144, 3, "bf16", 40, 3, 7),
    (1, 70, 3, 3, 256, 64, "f32", 65, 2, 15),
    (2, 256, 6, 2, 128, 16, "bf16", 300, 3, 7),   # three query heads per KV head
    (40, 36, 4, 2, 32, 4, "f32", 97, 2, 33),
    (40, 34, 4, 2, 32, 4, "bf16", 66, 3, 40),
])
def test_portable_path(gpu_available, L, d, hq, hkv, dh, B, dt, ctx, agents, T):
    shape = synth.ModelShape("gen", L, d, hq, hkv, dh, B, dt)
    n = -(-ctx // B) + agents * (-(-(T + 4) // B) + 3) + 4
    tw = Twin(shape, n_blocks=n, max_pos=ctx + T + 40, max_states=agents + 3, wl="gen")
    root = tw.materialize(ctx, pos0=2)
    kids = tw.fork(root, agents)
    tw.attend(kids, T)
    tw.attend(kids, 1)
    tw.attend(kids[:1], 3)
    tw.close()
