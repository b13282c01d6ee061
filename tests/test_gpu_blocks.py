"""The affinity's block shapes, row widths and work distribution at the edges where they
can go wrong: rows that end inside a 128-byte chunk, images that end inside a block."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_05718_amd as mpm
from parity import check_nearest, check_stage, to64
from work_shares import deferred

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


# Images that end at, before and past a block, several images per XCD share or several shares
# per image, empty images: (values a row, sizes, block rows picked for bf16 and f32 on 256 CUs).
WORK_CASES = {
    "one_image": (64, [1500], (64, 64)),
    "three_images": (64, [1024, 129, 897], (128, 64)),
    "uneven_shares": (64, [300, 0, 513, 256, 1, 128, 640, 257, 384, 0, 511, 127], (128, 64)),
    "many_small": (64, [65, 64, 1, 0, 63, 2] * 20, (64, 64)),
    "counted_limit": (32, [130, 1] * 256, (128, 128)),          # 512 images, the most counted one by one
    "past_counted_limit": (32, [130, 1] * 256 + [40], (128, 128)),
    "long_and_short": (64, [2300] + [30] * 9 + [1700], (128, 128)),
    "large_blocks": (32, [4096, 3300], (256, 256)),
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", list(WORK_CASES))
def test_work_distribution(dtype, name):
    """Ragged packed batches on the automatic pick, dense or packed, equal those on the
    forced full schedule: same neighbours, maps and merged rows; sampled images against
    the oracle."""
    D, ns, picks = WORK_CASES[name]
    rng = np.random.default_rng(len(ns) + D)
    rows = mpm.affinity_block_rows(len(ns), max(ns), D, TORCH_DT[dtype], packed=True)
    print(f"work distribution {name} {dtype}: rows {rows}", flush=True)
    if torch.cuda.get_device_properties(DEV).multi_processor_count == 256:
        assert rows == picks[dtype == "f32"]
    imgs = [store(clustered(rng, n, D, k=max(1, n // 6)), dtype) for n in ns]
    x, off, N = packed(imgs)
    m = mpm.merge(x, off, N=N)
    f = mpm.merge(x, off, N=N, schedule="full")
    torch.cuda.synchronize()
    total = int(m.y_off[-1])
    assert torch.equal(m.y_off, f.y_off) and torch.equal(m.map, f.map)
    assert torch.equal(m.y[:total], f.y[:total])
    nb, fb = m.nb.cpu().numpy(), f.nb.cpu().numpy()
    for b, n in enumerate(ns):
        assert np.array_equal(nb[b, :n], fb[b, :n]), b
        if n and b in (0, 1, 2, len(ns) - 1):
            check_nearest(to64(imgs[b]), nb[b, :n])


@pytest.mark.parametrize("B,N,D", [(1, 1500, 64), (5, 1024, 768), (24, 1024, 384), (9, 900, 192), (48, 200, 64)])
def test_picked_blocks_equal_full(B, N, D):
    """Dense batches: nearest neighbours and cosines of the automatic pick are bit for bit
    those of the full schedule on 256 x 256 blocks."""
    rng = np.random.default_rng(B * N)
    x = torch.stack([store(clustered(rng, N, D, k=20), "bf16") for _ in range(B)]).to(DEV)
    print(f"picked blocks B={B} N={N} D={D}: {mpm.affinity_block_rows(B, N, D, torch.bfloat16)} rows", flush=True)
    nb, best = mpm.argmax(x, with_best=True)
    fn, fb = mpm.argmax(x, with_best=True, schedule="full")
    torch.cuda.synchronize()
    assert torch.equal(nb, fn) and torch.equal(best.view(torch.int32), fb.view(torch.int32))


# float32 batches on either side of each line of the pick: small blocks at most four a CU,
# two rounds of middling blocks, one round of large ones, several rounds; two row widths that
# end inside a chunk.
@pytest.mark.parametrize("B,N,D", [(16, 512, 64), (17, 512, 64), (32, 1024, 36), (24, 990, 64), (1, 4096, 20)])
def test_picked_blocks_equal_small_f32(B, N, D):
    """Neighbours and cosines of a float32 batch do not depend on the blocks: bit for bit
    those of the same images one by one (64 x 64 blocks), image 0 also against the oracle."""
    rng = np.random.default_rng(B * N + D)
    x = torch.stack([store(clustered(rng, N, D, k=20), "f32") for _ in range(B)]).to(DEV)
    print(f"picked blocks f32 B={B} N={N} D={D}: {mpm.affinity_block_rows(B, N, D, torch.float32)} rows", flush=True)
    nb, best = mpm.argmax(x, with_best=True)
    for b in sorted({0, B // 2, B - 1}):
        one, cos = mpm.argmax(x[b:b + 1].contiguous(), with_best=True)
        torch.cuda.synchronize()
        assert torch.equal(nb[b], one[0]) and torch.equal(best[b].view(torch.int32), cos[0].view(torch.int32)), b
    check_nearest(to64(x[0].cpu()), nb[0].cpu().numpy())


# Tiles within, at and past the 16 lanes of a row; pieces short of the lanes, at four a lane
# and one past; an empty and a one-token image.
@pytest.mark.parametrize("dtype,D", [("bf16", 8), ("bf16", 512), ("bf16", 520), ("f32", 60), ("f32", 260)])
def test_cosines_of_packed_rows(dtype, D):
    rng = np.random.default_rng(D)
    ns = [1100, 0, 1, 64, 1025]
    print(f"cosines {dtype} D={D} ns={ns}", flush=True)
    x = torch.from_numpy(rng.standard_normal((sum(ns), D)).astype(np.float32)).to(TORCH_DT[dtype])
    off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    nb, best = mpm.argmax(x.to(DEV), torch.from_numpy(off).to(DEV), N=max(ns), with_best=True)
    only = mpm.argmax(x.to(DEV), torch.from_numpy(off).to(DEV), N=max(ns))
    torch.cuda.synchronize()
    nb, only, best = nb.cpu().numpy(), only.cpu().numpy(), best.cpu().numpy()
    for b, n in enumerate(ns):
        assert np.array_equal(nb[b, :n], only[b, :n])
        if n == 1:
            assert nb[b, 0] == -1 and best[b, 0] == -np.inf
        if n < 2:
            continue
        x64 = to64(x[off[b]:off[b + 1]])
        for i in (0, 1, 15, 16, 63, n // 2, n - 1):
            # float32 sums of D products and two float32 norms: below 3 (D + 4) 2^-24.
            assert abs(best[b, i] - oracle.cosine(x64, i, int(nb[b, i]))) <= 3 * (D + 4) * 2.0 ** -24


# One image, the most whose counts are added to the offsets directly, one more.
@pytest.mark.parametrize("B", [1, 2, 256, 257])
def test_offsets_in_an_unprepared_workspace(B):
    """Offsets, maps and sources of an insertion in a workspace and an offsets buffer that hold
    anything, twice in a row, equal those of the neighbours' own compaction (whose offsets are
    a second launch); some images empty."""
    from paper_2604_05718_amd import _lib, api

    rng = np.random.default_rng(B)
    ns = [int(n) for n in rng.integers(0, 70, B)]
    ns[0], ns[-1], N = 70, 70, 70
    print(f"offsets B={B}", flush=True)
    x = store(clustered(rng, sum(ns), 32, k=300), "bf16").to(DEV)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)).to(DEV)
    want = mpm.pair_compact(mpm.argmax(x, off, N=N), x_off=off)
    ws = torch.full((mpm.workspace_bytes(B, N),), 0xA5, dtype=torch.uint8, device=DEV)
    for _ in range(2):
        m = torch.full((B, N), -9, dtype=torch.int32, device=DEV)
        y_off = torch.full((B + 1,), 12345, dtype=torch.int32, device=DEV)
        _lib.check("mpm_affinity_compact", _lib.load().mpm_affinity_compact(
            api._p(x), api._p(off), None, B, N, 32, api._dt(x), 0, api._p(m), api._p(y_off), api._p(ws), ws.numel(), None,
            None, api._stream()))
        torch.cuda.synchronize()
        assert torch.equal(y_off, want[2]) and torch.equal(m, want[0])
        src = api.ws_view(ws, B, N, "src")
        for b in (0, B // 2, B - 1):
            c = int(y_off[b + 1] - y_off[b])
            assert torch.equal(src[b, :c], want[1][b, :c])


@pytest.mark.parametrize("D", [64, 1024])
def test_packed_pick_of_the_shortest_images(D):
    """Images of at most 64 tokens run the small blocks, packed (a guessed length is at least
    one token) or dense, however many they are."""
    for B in (1, 8, 31, 2000):
        for N in (1, 2, 64):
            print(f"pick of short images B={B} N={N} D={D}", flush=True)
            dense, packed = (mpm.affinity_block_rows(B, N, D, torch.bfloat16, packed=p) for p in (False, True))
            assert dense == packed == 64


# Images of one 256-row block, fewer than half of the slots: whole blocks, or (float32, and
# bfloat16 rows of at least six chunks) half blocks only; odd counts, 128 (halves on every
# slot) and one more; rows that end inside a chunk cannot have the schedule forced.
@pytest.mark.parametrize("dtype,B,N,D", [("f32", 7, 2, 768), ("f32", 128, 40, 32), ("f32", 129, 256, 48),
                                         ("bf16", 5, 200, 768), ("bf16", 63, 130, 384), ("bf16", 64, 256, 320),
                                         ("bf16", 128, 129, 416), ("f32", 1, 1, 64),
                                         ("f32", 1, 328, 192), ("bf16", 2, 665, 768),   # two and three blocks: whole
                                         ("bf16", 135, 76, 384), ("f32", 136, 76, 64)])  # not two slots for every block
def test_single_block_images_on_the_symmetric_schedule(dtype, B, N, D):
    """Neighbours and cosines, dense and packed, are those of the full schedule bit for bit."""
    rng = np.random.default_rng(B * N + D)
    print(f"single blocks {dtype} B={B} N={N} D={D}", flush=True)
    x = torch.stack([store(clustered(rng, N, D), dtype) for _ in range(B)]).to(DEV)
    off = torch.arange(0, (B + 1) * N, N, dtype=torch.int32, device=DEV)
    nf, bf = mpm.argmax(x, with_best=True, schedule="full")
    for args in (dict(), dict(x_off=off, N=N)):
        nb, best = mpm.argmax(x.view(B * N, D) if args else x, with_best=True, schedule="symmetric", **args)
        torch.cuda.synchronize()
        assert torch.equal(nb, nf) and torch.equal(best.view(torch.int32), bf.view(torch.int32))
    if N > 1:
        check_nearest(to64(x[B // 2].cpu()), nf[B // 2].cpu().numpy())


# Rows of one, four, five, 32 and 33 16-byte pieces (one, four and sixteen lanes a row), of
# more and fewer partial tiles than the lanes take together; more rows than the launch has
# lanes for (taken in turn), most of them past their image's end.
@pytest.mark.parametrize("dtype,D,ns", [(dt, p * (8 if dt == "bf16" else 4), [1300, 0, 1, 65, 300])
                                        for dt in ("bf16", "f32") for p in (1, 4, 5, 32, 33)] +
                                       [("bf16", 8, [1500] + [3, 0, 1, 40] * 700), ("f32", 100, [2000] + [2, 0, 1] * 50),
                                        ("bf16", 8, [5200, 1]), ("bf16", 256, [2200] * 2), ("f32", 16, [600] * 60)])
def test_cosines_of_narrow_rows(dtype, D, ns):
    rng = np.random.default_rng(D + len(ns))
    print(f"cosines of narrow rows {dtype} D={D} images {len(ns)}", flush=True)
    x = torch.from_numpy(rng.standard_normal((sum(ns), D)).astype(np.float32)).to(TORCH_DT[dtype])
    off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    args = (x.to(DEV), torch.from_numpy(off).to(DEV), max(ns))
    nb, best = mpm.argmax(*args, with_best=True)
    only = mpm.argmax(*args)
    torch.cuda.synchronize()
    nb, only, best = nb.cpu().numpy(), only.cpu().numpy(), best.cpu().numpy()
    for b, n in enumerate(ns):
        assert np.array_equal(nb[b, :n], only[b, :n]), b
        x64 = to64(x[off[b]:off[b + 1]])
        for i in sorted({0, 1, 15, 63, n // 2, n - 1}):
            if not 0 <= i < n:
                continue
            if n == 1:
                assert nb[b, 0] == -1 and best[b, 0] == -np.inf
                continue
            # float32 sums of D products and two float32 norms: below 3 (D + 4) 2^-24.
            assert abs(best[b, i] - oracle.cosine(x64, i, int(nb[b, i]))) <= 3 * (D + 4) * 2.0 ** -24, (b, i)


# Rows whose last chunk ends in its first half (computed as half a chunk), at its middle, one
# piece past it and at its end, on one chunk and on three; forced schedules where the width
# allows them, each block shape against the small blocks bit for bit.
@pytest.mark.parametrize("dtype,D", [(dt, (c * 128 + e) // (2 if dt == "bf16" else 4)) for dt in ("bf16", "f32")
                                     for c in (0, 2) for e in (16, 48, 64, 80, 112)])
def test_half_chunks(dtype, D):
    rng = np.random.default_rng(D)
    print(f"half chunks {dtype} D={D}", flush=True)
    x = torch.stack([store(clustered(rng, 700, D, k=20), dtype) for _ in range(33)]).to(DEV)
    nb, best = mpm.argmax(x, with_best=True)
    for b in (0, 16, 32):
        one, cos = mpm.argmax(x[b:b + 1].contiguous(), with_best=True)
        torch.cuda.synchronize()
        assert torch.equal(nb[b], one[0]) and torch.equal(best[b].view(torch.int32), cos[0].view(torch.int32))
    check_nearest(to64(x[0].cpu()), nb[0].cpu().numpy())
    for schedule in ("full", "symmetric") if D * x.element_size() % 64 == 0 else ():
        fn, fb = mpm.argmax(x, with_best=True, schedule=schedule)
        torch.cuda.synchronize()
        assert torch.equal(nb, fn) and torch.equal(best.view(torch.int32), fb.view(torch.int32)), schedule


@pytest.mark.parametrize("B,N,D,packed,rows", [(16, 1024, 16, False, 256), (16, 1024, 48, False, 256),
                                               (16, 1024, 64, False, 128), (64, 1024, 8, False, 256)])
def test_pick_of_narrow_f32_rows(B, N, D, packed, rows):
    """Dense float32 rows of at most a chunk and a half: a single round of full 256-row blocks,
    and several rounds of symmetric ones, where they are faster; equal to the small blocks."""
    if torch.cuda.get_device_properties(DEV).multi_processor_count != 256:
        pytest.skip("the picks are for a 256-CU device")
    print(f"narrow f32 pick B={B} N={N} D={D} packed={packed}", flush=True)
    assert mpm.affinity_block_rows(B, N, D, torch.float32, packed=packed) == rows
    rng = np.random.default_rng(B + D)
    ns = [int(v) for v in rng.integers(int(0.8 * N), int(0.9 * N), B)] if packed else [N] * B
    x = torch.cat([store(clustered(rng, n, D, k=40), "f32") for n in ns]).to(DEV)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)).to(DEV)
    args = (x, off, N) if packed else (x.view(B, N, D),)
    nb, small = mpm.argmax(*args), mpm.argmax(*args, schedule="full_64")
    torch.cuda.synchronize()
    for b in range(B):
        assert torch.equal(nb[b, :ns[b]], small[b, :ns[b]]), b


# Fewer images than XCDs: large blocks (one image whose last round runs as half blocks, two
# images, a part of a round), ragged small and middling blocks with a slot for each item.
@pytest.mark.parametrize("dtype,D,ns,N", [("bf16", 64, [5835], 5835), ("bf16", 64, [4500], 5400),
                                          ("bf16", 64, [3700, 3650], 4096), ("f32", 64, [4096, 3300], 4096),
                                          ("f32", 64, [1288, 80], 1288), ("bf16", 384, [2000, 100, 100], 2000),
                                          ("bf16", 64, [3, 1704, 0, 90, 1], 1704)])
def test_few_images(dtype, D, ns, N):
    rng = np.random.default_rng(sum(ns))
    rows = mpm.affinity_block_rows(len(ns), N, D, TORCH_DT[dtype], packed=True)
    print(f"few images {dtype} D={D} ns={ns} N={N}: {rows} rows", flush=True)
    imgs = [store(clustered(rng, n, D, k=40), dtype) for n in ns]
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)).to(DEV)
    x = torch.cat(imgs).to(DEV)
    nb = {s: mpm.argmax(x, off, N=N, schedule=s) for s in ("auto", "full", "symmetric", "full_64")}
    torch.cuda.synchronize()
    for b, n in enumerate(ns):
        for s in ("full", "symmetric", "full_64"):
            assert torch.equal(nb["auto"][b, :n], nb[s][b, :n]), (b, s)
    b = int(np.argmax(ns))
    check_nearest(to64(imgs[b]), nb["auto"][b, :ns[b]].cpu().numpy())


# Batches whose items lie far apart: counted ones with runs of more than 64 images without an
# item of the slot's, empty images at either end, 512 images and one less; batches past the
# counted limit, most of whose items lie past their image's end (more than 64 of a slot's in a
# row), the last image the only long one.
SPARSE = {
    "counted_runs": [300] + [0] * 90 + [600] + [1, 0, 2] * 100 + [0] * 60 + [900] + [0] * 20,
    "counted_limit": [0] + [3] * 500 + [0] * 5 + [700, 1, 0, 513, 0, 0],
    "below_the_limit": [40, 0, 1] * 170 + [900],
    "past_the_limit": [1400] + [0, 5, 0, 1, 70] * 130 + [1300],
    "last_long": [0] * 600 + [1, 1500],
}


@pytest.mark.parametrize("dtype,D", [("bf16", 32), ("f32", 16), ("bf16", 72)])
@pytest.mark.parametrize("name", list(SPARSE))
def test_items_far_apart(name, dtype, D):
    """Every schedule gives the same neighbours as the small blocks; the long images and some
    short ones against the oracle; the window (every item a band) too."""
    ns = SPARSE[name]
    rng = np.random.default_rng(len(ns))
    print(f"items far apart {name} {dtype} D={D}: {len(ns)} images", flush=True)
    x = store(clustered(rng, sum(ns), D, k=60), dtype).to(DEV)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)).to(DEV)
    N = max(ns)
    nb = {s: mpm.argmax(x, off, N=N, schedule=s) for s in ("full_64", "auto", "full", "symmetric")}
    torch.cuda.synchronize()
    keep = torch.arange(N, device=DEV)[None, :] < torch.diff(off)[:, None]
    for s in ("auto", "full", "symmetric"):
        assert torch.equal(nb[s][keep], nb["full_64"][keep]), s
    offh = off.cpu().numpy()
    for b in sorted(set(np.argsort(ns)[-2:].tolist() + [1, len(ns) // 2])):
        if ns[b]:
            check_nearest(to64(x[offh[b]:offh[b + 1]].cpu()), nb["auto"][b, :ns[b]].cpu().numpy())
    # A window over the whole grid is the dense method.
    one = mpm.merge(x, off, N=N)
    for rows in (128, 256) if D * x.element_size() % 64 == 0 else (0,):
        m = mpm.merge_local(x, N, N, x_off=off, N=N, block_rows=rows)
        torch.cuda.synchronize()
        assert torch.equal(m.y_off, one.y_off) and torch.equal(m.map, one.map)


@pytest.mark.parametrize("B,N,D,packed,used", [(500, 400, 384, False, "symmetric"), (900, 256, 64, False, "full"),
                                               (64, 1024, 768, False, "symmetric")])
def test_pick_of_large_batches(B, N, D, packed, used):
    """Batches of many rounds run the large blocks where they are faster; neighbours equal to
    the small blocks' (a sample of the images against the oracle)."""
    if torch.cuda.get_device_properties(DEV).multi_processor_count != 256:
        pytest.skip("the picks are for a 256-CU device")
    print(f"pick of a large batch B={B} N={N} D={D} packed={packed}", flush=True)
    assert mpm.affinity_block_rows(B, N, D, torch.bfloat16, packed=packed) == 256
    if not packed:
        assert mpm.affinity_schedule_used(B, N, D, torch.bfloat16) == used
    g = torch.Generator(device=DEV).manual_seed(B + D)
    ns = [int(v) for v in np.random.default_rng(B).integers(int(0.8 * N), int(0.9 * N), B)] if packed else [N] * B
    x = torch.randn((sum(ns), D), generator=g, device=DEV).to(torch.bfloat16)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)).to(DEV)
    args = (x, off, N) if packed else (x.view(B, N, D),)
    nb, small = mpm.argmax(*args), mpm.argmax(*args, schedule="full_64")
    torch.cuda.synchronize()
    keep = torch.arange(N, device=DEV)[None, :] < torch.diff(off)[:, None]
    assert torch.equal(nb[keep], small[keep])
    o = off.cpu().numpy()
    for b in (0, B - 1):
        check_nearest(to64(x[o[b]:o[b + 1]].cpu()), nb[b, :ns[b]].cpu().numpy())


def test_plans_are_what_runs():
    """affinity_plan agrees with the older queries where they apply, and with the partials a
    call leaves: exactly the slots of its block rows are written, full or symmetric; the same
    for the windowed blocks of any row width."""
    from paper_2604_05718_amd import _lib

    rng = np.random.default_rng(3)
    shapes = [(1, 700, 64, "bf16"), (9, 900, 192, "bf16"), (64, 1024, 72, "bf16"), (16, 1024, 40, "bf16"),
              (30, 1000, 52, "f32"), (64, 1024, 64, "bf16"), (3, 300, 24, "bf16")]
    for B, N, D, dtype in shapes:
        for packed in (False, True):
            dt = TORCH_DT[dtype]
            used, rows = mpm.affinity_plan(B, N, D, dt, packed=packed)
            print(f"plan B={B} N={N} D={D} {dtype} packed={packed}: {used} {rows}", flush=True)
            assert rows == mpm.affinity_block_rows(B, N, D, dt, packed=packed)
            assert (used == "full_64") == (rows == 64) and (rows != 128 or used == "symmetric")
            if D * (2 if dtype == "bf16" else 4) % 64 == 0:
                if not packed:
                    assert used == mpm.affinity_schedule_used(B, N, D, dt)
                for s in ("full", "symmetric", "full_64"):
                    assert mpm.affinity_plan(B, N, D, dt, s, packed)[0] == s
            x = store(clustered(rng, B * N, D, k=50), dtype).to(DEV)
            off = torch.arange(0, (B + 1) * N, N, dtype=torch.int32, device=DEV) if packed else None
            ws = torch.full((mpm.workspace_bytes(B, N),), 0x5A, dtype=torch.uint8, device=DEV)
            mpm.affinity(x if packed else x.view(B, N, D), off, N, ws=ws)
            wl = torch.full_like(ws, 0x5A)
            mpm.merge_local(x if packed else x.view(B, N, D), 32, 3, x_off=off, N=N if packed else None, ws=wl)
            torch.cuda.synchronize()
            o, T = _lib.workspace_offsets(B, N), (N + 63) // 64
            for w, width in ((ws, rows), (wl, mpm.local_tile_rows(B, N, D, dt, 32, 3))):
                pi = w[o["pi"]:o["pi"] + 4 * B * T * N].view(torch.int32).view(B, T, N)
                tiles = (N + width - 1) // width
                assert not bool((pi[:, :tiles] == 0x5A5A5A5A).any()) and bool((pi[:, tiles:] == 0x5A5A5A5A).all())


# Rows that are no whole number of 64 bytes cannot have a schedule forced: batches whose pick is
# each kind of 256-row block, dense and packed, with deferred diagonal blocks and without, images
# counted one by one and not.
@pytest.mark.parametrize("dtype,B,N,D,packed,plan,halves",
                         [("bf16", 64, 1024, 200, False, ("symmetric", 256), True),
                          ("bf16", 16, 1024, 200, False, ("full", 256), False),
                          ("f32", 46, 1924, 212, False, ("symmetric", 256), True),
                          ("bf16", 16, 1024, 136, True, ("full", 256), False),
                          ("bf16", 12, 1600, 200, True, ("symmetric", 256), True),
                          ("bf16", 16, 4096, 24, True, ("symmetric", 256), True),
                          ("f32", 2, 4096, 28, True, ("symmetric", 256), True)])
def test_large_blocks_of_odd_rows(dtype, B, N, D, packed, plan, halves):
    for seed in range(50):  # the first ragged lengths that leave blocks to the half-block launch
        rng = np.random.default_rng(B * D + seed)
        ns = [int(v) for v in rng.integers(int((0.55 if B >= 16 else 0.85) * N), N + 1, B)] if packed else [N] * B
        if packed and B >= 16:
            ns[0], ns[B // 2], ns[-1] = 0, N, 1
        groups = dict() if B >= 8 else dict(groups=1, slots=256)  # few images: the chip's slots in one group
        if not halves or any(deferred(ns, **groups)):
            break
    print(f"large blocks of odd rows {dtype} B={B} N={N} D={D} packed={packed}", flush=True)
    if torch.cuda.get_device_properties(DEV).multi_processor_count == 256:
        assert mpm.affinity_plan(B, N, D, TORCH_DT[dtype], packed=packed) == plan
    if plan[0] == "symmetric":
        assert any(deferred(ns, **groups)) == halves
    g = torch.Generator(device=DEV).manual_seed(B + D)
    cent = torch.randn((200, D), generator=g, device=DEV)
    x = cent[torch.randint(0, 200, (sum(ns),), generator=g, device=DEV)]
    x = (x + 0.3 * torch.randn((sum(ns), D), generator=g, device=DEV)).to(TORCH_DT[dtype])
    o = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    off = torch.from_numpy(o).to(DEV)
    m = mpm.merge(x, off, N=N) if packed else mpm.merge(x.view(B, N, D))
    # Image by image: the small blocks, whatever the batch runs.
    nb = m.nb
    sample = sorted({1, B // 4, B // 2, B - 2} | set(rng.integers(0, B, 6).tolist()))
    for b in sample:
        if ns[b] == 0:
            continue
        img = x[o[b]:o[b + 1]].contiguous()
        one = mpm.argmax(img[None])
        torch.cuda.synchronize()
        assert torch.equal(nb[b, :ns[b]], one[0]), b
    for b in {1, B // 2} if N * N * D < 1e9 else {1}:
        check_nearest(to64(x[o[b]:o[b + 1]].cpu()), nb[b, :ns[b]].cpu().numpy())


@pytest.mark.parametrize("B,N,D", [(64, 1024, 96), (300, 400, 32), (20, 700, 224)])
def test_given_norms_of_half_chunks(B, N, D):
    """Two insertions on rows that end inside a chunk, the second on given norms and counted
    ragged images: neighbours, maps and merged rows of sampled images against the oracle."""
    rng = np.random.default_rng(N + D)
    print(f"given norms of half chunks B={B} N={N} D={D}", flush=True)
    x = torch.stack([store(clustered(rng, N, D, k=40), "bf16") for _ in range(B)])
    m1 = mpm.merge(x.to(DEV), want_inv=True)
    m2 = mpm.merge(m1.y, m1.y_off, N=N, x_inv=m1.y_inv)
    torch.cuda.synchronize()
    o1, o2 = m1.y_off.cpu().numpy(), m2.y_off.cpu().numpy()
    for b in sorted({0, 7, B // 2, B - 1}):
        y1 = to64(m1.y[o1[b]:o1[b + 1]].cpu())
        s1 = check_stage(to64(x[b]), "bf16", m1.nb[b].cpu().numpy(), m1.map[b].cpu().numpy(), y1)
        check_stage(y1, "bf16", m2.nb[b, :s1.count].cpu().numpy(), m2.map[b].cpu().numpy(), to64(m2.y[o2[b]:o2[b + 1]].cpu()))
