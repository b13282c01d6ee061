"""The affinity's block shapes, row widths and work distribution at the edges where they
can go wrong: rows that end inside a 128-byte chunk, images that end inside a block."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_05718_amd as mpm
from parity import check_nearest, check_stage, to64

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def clustered(rng, n, D, k=6, sigma=0.3):
    cent = rng.standard_normal((k, D))
    return cent[rng.integers(0, k, n)] + sigma * rng.standard_normal((n, D))


def store(x64, dtype):
    return torch.from_numpy(np.asarray(x64, np.float32)).to(TORCH_DT[dtype])


def packed(imgs):
    off = np.concatenate([[0], np.cumsum([len(i) for i in imgs])]).astype(np.int32)
    return torch.cat(imgs).to(DEV), torch.from_numpy(off).to(DEV), max(len(i) for i in imgs)


def check_merge(imgs, dtype, m):
    """nb, map and merged rows of a packed merge against the oracle, image by image."""
    off = m.y_off.cpu().numpy()
    nb, maps, y = m.nb.cpu().numpy(), m.map.cpu().numpy(), to64(m.y[: off[-1]])
    for b, img in enumerate(imgs):
        n = len(img)
        if n == 0:
            assert off[b + 1] == off[b] and np.all(maps[b] == -1)
            continue
        check_stage(to64(img), dtype, nb[b, :n], maps[b], y[off[b]:off[b + 1]])


# Rows of 16 bytes to 1 KB that end at, one piece before and one piece past a 128-byte
# chunk, and inside a 32-byte matrix step.
@pytest.mark.parametrize("dtype,D", [("bf16", D) for D in (8, 56, 72, 120, 136, 200, 520)] +
                                    [("f32", D) for D in (4, 28, 36, 60, 100, 260)])
def test_rows_of_any_width(dtype, D):
    """Dense and packed rows that are no whole number of chunks: small blocks (one
    image) and large ones (nine ragged images, the last ending with the buffer)."""
    rng = np.random.default_rng(D)
    print(f"rows of {D} {dtype}", flush=True)
    one = [store(clustered(rng, 300, D, k=40), dtype)]
    nb = mpm.argmax(one[0][None].to(DEV))
    torch.cuda.synchronize()
    check_nearest(to64(one[0]), nb[0].cpu().numpy())
    imgs = [store(clustered(rng, n, D, k=40), dtype) for n in (513, 1, 256, 700, 2, 255, 640, 0, 257)]
    x, off, N = packed(imgs)
    m = mpm.merge(x, off, N=N)
    torch.cuda.synchronize()
    check_merge(imgs, dtype, m)
