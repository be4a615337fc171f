"""What lvx_workspace_bytes asks for, evaluated on the CPU: a workspace sized for a call serves every call with fewer tokens."""
import ctypes as C
import random

import pytest

import paper_2512_04677_amd as lvx


def stage(heads, head_dim, ffn, n_layers, fp8):
    """A stage that only its sizes matter of, and what its pointers point to."""
    y = head_dim // 6 * 2
    rope = lvx.rope_desc(heads, head_dim, (head_dim - 2 * y, y, y), 1e4, 30, 52)
    blocks, blocks8 = (lvx.BlockWeights * n_layers)(), (lvx.BlockWeightsFp8 * n_layers)()
    b8 = C.cast(blocks8, C.POINTER(lvx.BlockWeightsFp8)) if fp8 else None
    return lvx.Stage(n_layers, ffn, 0, 0, rope, C.cast(blocks, C.POINTER(lvx.BlockWeights)), b8, 0, 0), (blocks, blocks8)


# heads, head_dim, FFN width, FP8, tokens of two chunks of which the shorter one's attention may be split, or was once sized as if it were
PAIRS = [(40, 128, 13824, True, 1536, 3072), (24, 128, 8192, True, 2560, 5120), (40, 128, 13824, True, 1500, 3000), (40, 128, 13824, False, 1536, 2304),
         (32, 128, 8192, True, 2048, 3072), (32, 128, 8192, True, 1536, 1537), (12, 128, 6144, True, 4096, 4097), (40, 64, 5120, False, 1152, 1153)]


@pytest.mark.parametrize("heads,head_dim,ffn,fp8,few,many", PAIRS)
def test_workspace_of_a_longer_chunk_serves_a_shorter_one(heads, head_dim, ffn, fp8, few, many):
    lib = lvx.load()
    s, keep = stage(heads, head_dim, ffn, 8, fp8)
    for n_ctx in (64, 77):
        assert 0 < lib.lvx_workspace_bytes(C.byref(s), few, n_ctx) <= lib.lvx_workspace_bytes(C.byref(s), many, n_ctx)


def test_workspace_never_shrinks_with_the_tokens():
    lib = lvx.load()
    rng = random.Random(6)
    for _ in range(300):
        heads, head_dim = 2 * rng.randint(1, 24), rng.choice([64, 128])
        s, keep = stage(heads, head_dim, 128 * rng.randint(2, 110), rng.randint(1, 8), rng.random() < 0.5)
        n_ctx = rng.randint(1, 600)
        # all lengths near the multiples of a workgroup's queries, some between
        tokens = sorted({128 * i + j for i in range(1, 50) for j in (-1, 0, 1, 2)} | {rng.randint(1, 8000) for _ in range(50)})
        sizes = [lib.lvx_workspace_bytes(C.byref(s), n, n_ctx) for n in tokens]
        assert sizes[0] > 0 and all(a <= b for a, b in zip(sizes, sizes[1:])), (heads, head_dim)
