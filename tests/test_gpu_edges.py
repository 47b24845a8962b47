"""Parity at the edges of the kernels' tiles, walks and dispatch rules, against the CPU oracle.

Bars: prefix lengths and slots bit-exact; extend attention within max-abs 1e-4 (fp32 sums of at most some hundred values of
order one) and 2e-2 (bf16 probabilities and results: half a unit in the last place is 2^-9 of a value, values of up to 5)."""
import threading

import numpy as np
import pytest
import torch

from harness import out_to_f64, to_torch
from paper_2407_00023_amd import workloads as W

TOL = {"f32": 1e-4, "bf16": 2e-2, "bf16_kv8": 2e-2}


@pytest.fixture(scope="module")
def pa(gpu_device):
    from paper_2407_00023_amd import binding
    return binding


def _path(rng, edges, vocab=1000):
    """A cached trunk cut into nodes with these edge lengths, by a sequence that leaves it at every cut."""
    trunk = rng.integers(0, vocab, sum(edges)).astype(np.int32)
    cached = [(trunk, np.arange(len(trunk), dtype=np.int32))]
    for i, c in enumerate(np.cumsum(edges)[:-1]):
        cached.append((np.append(trunk[:c], (trunk[c] + 1) % vocab).astype(np.int32),
                       np.append(np.arange(c), 100000 + i).astype(np.int32)))
    return trunk, cached


# None: as many requests as there are prompts below (5 to 49), 16 workgroups each; 65: 15, 256: 4; 257, 300: one, windows of 1,024
# positions; 1025: of 512.  Paths around
# the walk's limits: 4 nodes whatever their length, 16 while they hold 128 tokens on average; swept by one workgroup up to 4,096
# tokens, by several beyond; in the end windows, more of them than workgroups
@pytest.mark.gpu
@pytest.mark.parametrize("B", [None, 65, 256, 257, 300, 1025])
@pytest.mark.parametrize("edges", [[1], [1, 1, 1], [1, 1, 1, 1], [2, 1, 3, 1, 5], [127] * 5, [128] * 5, [128] * 15, [128] * 16,
                                   [200] * 17, [1023, 1, 1, 1021], [4096], [4097], [3000, 1500, 700], [2048] * 6, [1, 1, 1, 1, 9000],
                                   [700] * 4 + [3] * 500],
                         ids=lambda e: f"{len(e)}x{e[0]}")
def test_match_at_the_limits_of_walk_sweep_and_window(pa, gpu_device, edges, B):
    import oracle
    rng = np.random.default_rng(len(edges) + edges[0])
    trunk, cached = _path(rng, edges)
    n, cuts = len(trunk), np.cumsum(edges)
    prompts = [np.zeros(0, np.int32), trunk, np.append(trunk, np.int32(7))]
    # ends and mismatches at the first and last token of edges, and around multiples of a wave, a sweep and a window
    at = {0, 1, n // 2, n - 1} | {int(c) + d for c in (cuts[0], cuts[-1] - edges[-1], cuts[len(cuts) // 2]) for d in (-1, 0, 1)}
    at |= {k + d for k in (64, 512, 1024, 2048, 4096) for d in (-1, 0)}
    for c in sorted(x for x in at if 0 <= x < n):
        wrong = trunk.copy()
        wrong[c] = (wrong[c] + 500) % 1000
        prompts += [trunk[:c], wrong]
    prompts = (prompts * 210)[:B] if B else prompts
    toks = np.concatenate(prompts).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([len(p) for p in prompts])]).astype(np.int32)
    pl_ref, si_ref = oracle.match_prefixes(cached, toks, off)
    tree = pa.Tree()
    for c in cached:
        tree.insert(*c)
    tree.upload()
    print(f"[case] match path {edges[:4]}... B {len(prompts)}", flush=True)
    pl, si = pa.match_prefixes(tree, torch.from_numpy(toks).to(gpu_device), torch.from_numpy(off).to(gpu_device))
    pl, si = pl.cpu().numpy(), si.cpu().numpy()
    np.testing.assert_array_equal(pl, pl_ref)
    for r in range(len(prompts)):
        np.testing.assert_array_equal(si[off[r]:off[r] + pl_ref[r]], si_ref[off[r]:off[r] + pl_ref[r]])


def _same_hash_blocks(n=128):
    """Two blocks of n tokens whose path hashes are equal behind any common beginning: a Thue-Morse sequence of two token ids and
    its complement.  The hashes differ by (difference of the ids) x prod_i (base^(2^i) - 1), a multiple of 2^64 for n = 128
    and ids 2^29 apart; checked here with the library's base."""
    import os
    import re
    src = open(os.path.join(os.path.dirname(W.__file__), "csrc", "common.h")).read()
    base = int(re.search(r"kPathHashBase = (0x[0-9A-Fa-f]+)", src).group(1), 16)
    tm = np.array([bin(i).count("1") & 1 for i in range(n)], np.int32)
    x, y = (tm << 29).astype(np.int32), ((1 - tm) << 29).astype(np.int32)
    h = [0, 0]
    for k, block in enumerate((x, y)):
        for t in block:
            h[k] = (h[k] * base + int(t) + 1) % 2 ** 64
    assert h[0] == h[1]
    return x, y


def _insert_cuts(cached, seq, cuts, slot0):
    """seq cut into nodes at `cuts`, by sequences that leave it there."""
    cached.append((seq, np.arange(slot0, slot0 + len(seq), dtype=np.int32)))
    for c in cuts:
        cached.append((np.append(seq[:c], np.int32(5000 + len(cached))), np.append(np.arange(slot0, slot0 + c), 10 ** 6 + len(cached)).astype(np.int32)))


# Two paths with the same hash at some depth.  "same depth": a node begins there on both, a long edge on one, short ones on the
# other, cut just past the end of the first window, so that the long edge, where it hides the other node in the index, reaches
# over the next window's nodes.  "inside an edge": on one path the depth lies inside an edge of some windows' length, behind
# which short edges go on, and the other's node reaches past that edge's end.
@pytest.mark.gpu
@pytest.mark.parametrize("B", [2, 65, 256, 257, 1025])
@pytest.mark.parametrize("kind", ["same depth", "inside an edge"])
@pytest.mark.parametrize("swap", [False, True])
def test_match_on_paths_with_colliding_hashes(pa, gpu_device, kind, swap, B):
    import oracle
    rng = np.random.default_rng(5)
    x, y = _same_hash_blocks()
    if swap:
        x, y = y, x
    edges = [200] * 4 + [3] * 3 + [12]   # the walk stops at 809, short of the blocks
    head, tail = rng.integers(0, 4000, sum(edges)).astype(np.int32), rng.integers(0, 4000, 7000).astype(np.int32)
    at = len(head) + len(x)
    long_path, cut_path = np.concatenate([head, x, tail]), np.concatenate([head, y, tail])
    cached = []
    if kind == "same depth":
        _insert_cuts(cached, long_path, list(np.cumsum(edges)) + [at], 0)
        _insert_cuts(cached, cut_path, [at] + list(range(1030, 4000, 50)), 20000)
    else:
        _insert_cuts(cached, long_path, list(np.cumsum(edges)) + [at + 300], 0)
        _insert_cuts(cached, cut_path, list(range(at + 2500, at + 5500, 50)), 20000)
    prompts = [cut_path, long_path]
    for cut in (at - 1, at, at + 1, 1024, 1030, 1031, 2048, at + 2499, at + 2500, at + 2600, 4096):
        for path in (cut_path, long_path):
            wrong = path.copy()
            wrong[cut] = 4999
            prompts += [path[:cut], wrong]
    prompts = (prompts * 24)[:B]
    toks = np.concatenate(prompts).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([len(p) for p in prompts])]).astype(np.int32)
    pl_ref, si_ref = oracle.match_prefixes(cached, toks, off)
    tree = pa.Tree()
    for c in cached:
        tree.insert(*c)
    tree.upload()
    print(f"[case] colliding hashes, {kind}, swapped {swap}, B {B}", flush=True)
    t, o = torch.from_numpy(toks).to(gpu_device), torch.from_numpy(off).to(gpu_device)
    for _ in range(4):
        pl, si = pa.match_prefixes(tree, t, o)
        pl, si = pl.cpu().numpy(), si.cpu().numpy()
        np.testing.assert_array_equal(pl, pl_ref)
        for r in range(len(prompts)):
            np.testing.assert_array_equal(si[off[r]:off[r] + pl_ref[r]], si_ref[off[r]:off[r] + pl_ref[r]])


@pytest.mark.gpu
def test_captured_matches_beside_eager_ones(pa, gpu_device):
    """Graphs with a match of several workgroups per request, replayed while other matches run on other streams; then a graph
    with more captured calls than the library keeps buffers for.  Every replay is compared, with eager work in between."""
    import oracle
    rng = np.random.default_rng(11)
    trunk, cached = _path(rng, [700] * 4 + [3] * 500)
    tree = pa.Tree()
    for c in cached:
        tree.insert(*c)
    tree.upload()

    def batch(B, seed):
        cuts = np.random.default_rng(seed).integers(0, len(trunk), B)
        prompts = [np.append(trunk[:c], np.int32(2000)) for c in cuts]
        toks, off = np.concatenate(prompts).astype(np.int32), np.concatenate([[0], np.cumsum(cuts + 1)]).astype(np.int32)
        pl, si = oracle.match_prefixes(cached, toks, off)
        assert np.array_equal(pl, cuts)
        b = dict(t=torch.from_numpy(toks).to(gpu_device), o=torch.from_numpy(off).to(gpu_device), want=(pl, si), off=off)
        b["len"], b["slot"] = torch.full((B,), -1, dtype=torch.int32, device=gpu_device), torch.full_like(b["t"], -1)
        return b

    def check(b, pl, si):
        pl, si, off = pl.cpu().numpy(), si.cpu().numpy(), b["off"]
        np.testing.assert_array_equal(pl, b["want"][0])
        for r in range(len(pl)):
            np.testing.assert_array_equal(si[off[r]:off[r] + pl[r]], b["want"][1][off[r]:off[r] + pl[r]])

    run = lambda b: pa.match_prefixes(tree, b["t"], b["o"], b["len"], b["slot"])
    batches = [batch(B, B) for B in (40, 128, 200, 256)]
    streams = [torch.cuda.Stream() for _ in batches]
    for b in batches:
        run(b)
    torch.cuda.synchronize()
    graphs = []
    for b in batches[:2]:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            run(b)
    for k in range(10):
        print(f"[case] captured matches beside eager ones, round {k}", flush=True)
        for b in batches:
            b["len"].fill_(-1), b["slot"].fill_(-1)
        torch.cuda.synchronize()
        for i, b in enumerate(batches):
            with torch.cuda.stream(streams[i]):
                for _ in range(1 if i < 2 else 40):
                    graphs[i].replay() if i < 2 else run(b)
        torch.cuda.synchronize()
        for b in batches:
            check(b, b["len"], b["slot"])
    small, many = batch(3, 1), 130
    pls = torch.full((many, 3), -1, dtype=torch.int32, device=gpu_device)
    sis = torch.full((many, len(small["t"])), -1, dtype=torch.int32, device=gpu_device)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for k in range(many):
            pa.match_prefixes(tree, small["t"], small["o"], pls[k], sis[k])
    for _ in range(3):
        pls.fill_(-1), sis.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        for k in range(many):
            check(small, pls[k], sis[k])


def _items(ws, B, rows, D):
    """The item records of a work list, 12 ints each: behind the header, the tile table and the member table (extend_plan.h)."""
    up = lambda n: -(-n // 256) * 256
    own = min(rows, B * (48 if D == 128 else 64)) // 32 + B if 1 < B <= 256 else 0
    at = 256 + up(8 * (-(-rows // 128) + B + own)) + (up(32 * B) if B <= 256 else 0)
    return ws[at:at + 48 * ws[4:8].view(torch.int32).item()].view(torch.int32).reshape(-1, 12).tolist()


def _extend(pa, dev, dtype, P, E, Hq, Hkv, D, page, common=0, seed=0, tiles=None, kv_more=0, cut=None, direct=None, louder_from=None,
            records=None):
    """Largest error against the oracle for requests with P[r] cached tokens, the first `common` of them the same for all.
    tiles: how many row tiles the work list has to hold; kv_more: how many more keys than it has the call is told of (1,000,000: it
    builds a list whatever the batch); cut, direct: whether any tile has to be cut into parts, and the call to go without a list;
    louder_from: the key of every request from which on keys are 48 times as large (no common tokens then); records: a list that gets
    the item records of the work list."""
    import oracle
    rng = np.random.default_rng(seed)
    P, E = np.asarray(P, np.int32), np.asarray(E, np.int32)
    B, el = len(P), "f32" if dtype == "f32" else "bf16"
    npages = -(-common // page) + sum(-(-int(p - common) // page) for p in P)
    nslots = (npages + 3) * page
    order, cur = rng.permutation(npages + 3), 0

    def take(n):
        nonlocal cur
        k = -(-n // page)
        pages, cur = order[cur:cur + k], cur + k
        return (pages[:, None] * page + np.arange(page)).reshape(-1)[:n].astype(np.int32)

    head = take(common)
    slots = [np.concatenate([head, take(int(p) - common)]) for p in P]
    off = np.concatenate([[0], np.cumsum(P + E)]).astype(np.int32)
    eo = np.concatenate([[0], np.cumsum(E)]).astype(np.int32)
    si = np.full(off[-1], -1, np.int32)
    for r in range(B):
        si[off[r]:off[r] + P[r]] = slots[r]
    backed = np.unique(np.concatenate(slots))
    ss = np.random.SeedSequence(seed + 17).spawn(5)
    mk = lambda s, n, h: W._normal(s, n * h * D, el).reshape(n, h, D)
    T = int(eo[-1])
    q, k, v, pk, pv = mk(ss[0], T, Hq), mk(ss[1], T, Hkv), mk(ss[2], T, Hkv), mk(ss[3], len(backed), Hkv), mk(ss[4], len(backed), Hkv)
    if louder_from is not None:
        assert common == 0 and el == "bf16"
        fk, fpk = W.bf16_bits_to_f32(k).copy(), W.bf16_bits_to_f32(pk).copy()
        for r in range(B):
            fk[eo[r] + max(louder_from - P[r], 0):eo[r + 1]] *= 48
            fpk[np.searchsorted(backed, slots[r][louder_from:])] *= 48
        k, pk = W.f32_to_bf16_bits(fk), W.f32_to_bf16_bits(fpk)
    tdt, kv8 = (torch.float32 if dtype == "f32" else torch.bfloat16), dtype == "bf16_kv8"
    kw = dict(page_size=page, num_slots=nslots, kv8=kv8)
    pool = torch.zeros(pa.kv_pool_bytes(nslots, Hkv, D, tdt, page, kv8), dtype=torch.uint8, device=dev)
    tt = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    pa.append_kv(pool, tt(backed), to_torch(pk, el, dev), to_torch(pv, el, dev), **kw)
    print(f"[case] extend {dtype} P {P[:6]} E {E[:6]} Hq {Hq} Hkv {Hkv} D {D} page {page} common {common}", flush=True)
    told = int((P + E).max()) + kv_more
    ws = torch.zeros(pa.extend_workspace_bytes(B, T, told, Hq, Hkv, D, tdt), dtype=torch.uint8, device=dev)
    out = pa.extend_attention(to_torch(q, el, dev), to_torch(k, el, dev), to_torch(v, el, dev), pool, tt(si), tt(off), tt(P), tt(E),
                              tt(eo), D ** -0.5, max_kv_len=told, workspace=ws, **kw)
    torch.cuda.synchronize()
    if dtype != "f32":
        assert ws[12:16].view(torch.int32).item() == 0  # (the work list fitted)
        assert tiles is None or ws[:4].view(torch.int32).item() == tiles
        assert direct is None or (ws[20:24].view(torch.int32).item() > 0) == direct
        if records is not None:
            records.extend(_items(ws, B, T * (Hq // Hkv), D))
        assert cut is None or (ws[4:8].view(torch.int32).item() > ws[:4].view(torch.int32).item()) == cut
    opk, opv = oracle.new_pool(nslots, Hkv, D, dtype)
    oracle.append_kv(opk, opv, backed, pk, pv, dtype)
    ref = oracle.extend_attention(q, k, v, opk, opv, si, off, P, E, eo, D ** -0.5, dtype)
    return np.abs(out_to_f64(out) - ref).max()


# lanes of a key (D / 4), keys of a round (four each), heads of a KV head
@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,D", [(4, 2, 64), (1, 1, 64), (8, 1, 64), (6, 2, 128), (3, 1, 128), (16, 2, 128)])
def test_f32_extend_around_its_key_rounds(pa, gpu_device, Hq, Hkv, D):
    err = _extend(pa, gpu_device, "f32", [0, 1, 3, 4, 5, 7, 8, 15, 16, 17, 31, 33, 63, 65, 97], [1, 1, 2, 1, 3, 9, 1, 2, 1, 5, 1, 4, 1, 17, 1],
                  Hq, Hkv, D, 1)
    assert err <= TOL["f32"], err


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("P,E", [(0, 1), (3, 1), (3, 5), (17, 2), (64, 3), (97, 30)])
def test_f32_extend_with_an_infinite_value(pa, gpu_device, D, P, E):
    """An infinity in a V row that is visible to a row makes that element of the row infinite, not NaN, wherever the row stands
    among the keys; rows that do not see it are untouched."""
    nslots, Hq, Hkv = 128, 4, 2
    gen = torch.Generator(device=gpu_device).manual_seed(P + E)
    mk = lambda n, h: torch.randn(n, h, D, generator=gen, device=gpu_device)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=gpu_device)
    q, k, v, pk, pv = mk(E, Hq), mk(E, Hkv), mk(E, Hkv), mk(nslots, Hkv), mk(nslots, Hkv)
    kw = dict(page_size=1, num_slots=nslots)
    for at in sorted({P + E - 1, P + E // 2, max(P - 1, 0)}):  # the key whose V row holds it
        vv, pvv = v.clone(), pv.clone()
        (pvv[at] if at < P else vv[at - P])[1, 5] = float("inf")
        pool = torch.zeros(pa.kv_pool_bytes(nslots, Hkv, D, torch.float32, 1), dtype=torch.uint8, device=gpu_device)
        pa.append_kv(pool, i32(range(nslots)), pk, pvv, **kw)
        out = pa.extend_attention(q, k, vv, pool, i32(range(P + E)), i32([0, P + E]), i32([P]), i32([E]), i32([0, E]), D ** -0.5,
                                  max_kv_len=P + E, **kw).cpu().double()
        K, V = torch.cat([pk[:P], k]).cpu().double(), torch.cat([pvv[:P], vv]).cpu().double()
        for i in range(E):
            for h in range(Hq):
                n = P + i + 1
                p = torch.softmax(K[:n, h // 2] @ q[i, h].cpu().double() * D ** -0.5, 0)
                torch.testing.assert_close(out[i, h], p @ V[:n, h // 2], atol=TOL["f32"], rtol=0)


# a token's request is found by comparisons of all offsets at once up to 256 requests, by a search beyond; requests without new
# tokens among them, first and last
@pytest.mark.gpu
@pytest.mark.parametrize("B", [64, 65, 255, 256, 257, 400])
def test_f32_extend_finds_the_request_of_a_token(pa, gpu_device, B):
    E = [(r % 3) if r % 50 else 0 for r in range(B)]
    E[-2:] = [2, B % 2]
    assert _extend(pa, gpu_device, "f32", [r % 5 for r in range(B)], E, 2, 1, 64, 1) <= TOL["f32"]


@pytest.mark.gpu
def test_f32_extend_leaves_rows_of_no_request_alone(pa, gpu_device):
    """Offsets that do not begin at 0: the rows before the first request's get no output, its own do."""
    D, gen = 64, torch.Generator(device=gpu_device).manual_seed(1)
    mk = lambda n, h: torch.randn(n, h, D, generator=gen, device=gpu_device)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=gpu_device)
    q, k, v = mk(5, 2), mk(5, 1), mk(5, 1)
    pool = torch.zeros(pa.kv_pool_bytes(8, 1, D, torch.float32, 1), dtype=torch.uint8, device=gpu_device)
    out = torch.full_like(q, 7.0)
    pa.extend_attention(q, k, v, pool, i32([-1] * 2), i32([0, 2]), i32([0]), i32([2]), i32([3, 5]), D ** -0.5, max_kv_len=2,
                        page_size=1, num_slots=8, out=out)
    out = out.cpu()
    assert bool((out[:3] == 7.0).all())
    torch.testing.assert_close(out[3], v[3].expand(2, D).cpu(), atol=TOL["f32"], rtol=0)


# rows around the 32 of a narrow tile and the 128 of a wide one, keys around a block of 32 and a round of the four waves
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "bf16_kv8"])
@pytest.mark.parametrize("D,page", [(128, 16), (64, 1), (64, 64)])
@pytest.mark.parametrize("E,G", [(1, 1), (31, 1), (33, 1), (8, 4), (9, 4), (4, 8), (16, 8), (17, 8)])
def test_extend_around_the_narrow_and_wide_tile(pa, gpu_device, dtype, D, page, E, G):
    P = [0, 1, 31, 32, 33, 63, 64, 127, 128, 129, 300, 1100]
    assert _extend(pa, gpu_device, dtype, P, [E] * len(P), 2 * G, 2, D, page) <= TOL[dtype]


# runs of tiles in assembly for heads of 64: ends of the prefix and of the new tokens around whole tiles, extends past the
# diagonal of several row tiles, key ranges cut into parts
@pytest.mark.usefixtures("both_forms")
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "bf16_kv8"])
@pytest.mark.parametrize("page", [1, 16, 24])
@pytest.mark.parametrize("P,E", [([0], [513]), ([64, 63, 65], [129, 200, 64]), ([640, 127], [70, 300]), ([2100], [40])])
def test_extend_heads_of_64_around_whole_tiles(pa, gpu_device, dtype, page, P, E):
    assert _extend(pa, gpu_device, dtype, P, E, 8, 2, 64, page) <= TOL[dtype]


# common first parts that end around the planner's probes (512, 1,024, 1,536) and between them; own keys from none to tiles
@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("common", [511, 512, 513, 700, 1023, 1024, 1025, 1537])
@pytest.mark.parametrize("own", [1, 3, 65])
def test_extend_common_first_parts_around_the_probes(pa, gpu_device, D, common, own):
    P = [common + own * (r % 3) + r // 3 for r in range(9)]
    assert _extend(pa, gpu_device, "bf16", P, [1 + r % 2 for r in range(9)], 8, 2, D, 16, common=common) <= TOL["bf16"]


# rows of a request up to which a common first part is shared: 48 (heads of 128) or 64, behind fewer than 1,024 common keys 32;
# eight requests share tiles of 128 rows, or have one each
@pytest.mark.gpu
@pytest.mark.parametrize("D,common,E,tiles", [(128, 1100, 12, 3), (128, 1100, 13, 8), (64, 1100, 16, 4), (64, 1100, 17, 8), (128, 700, 8, 2),
                                              (128, 700, 9, 8), (128, 1024, 9, 3), (128, 1023, 9, 8), (128, 1100, 24, 8)])
def test_extend_rows_that_share_a_first_part(pa, gpu_device, D, common, E, tiles):
    P = [common + 70 + r for r in range(8)]
    assert _extend(pa, gpu_device, "bf16", P, [E] * 8, 8, 2, D, 16, common=common, tiles=tiles) <= TOL["bf16"]


# the largest batches of each planner (256: with sharing, 1,024: ordered, beyond: as given) and the smallest that are beyond
@pytest.mark.usefixtures("both_forms")
@pytest.mark.gpu
@pytest.mark.parametrize("B", [1, 2, 63, 64, 255, 256, 257, 1024, 1025])
def test_extend_batch_sizes_around_the_planners(pa, gpu_device, B):
    P = [600 + r % 7 for r in range(B)]
    assert _extend(pa, gpu_device, "bf16", P, [1 + r % 2 for r in range(B)], 4, 1, 64, 16, common=600) <= TOL["bf16"]


@pytest.mark.gpu
def test_hot_path_calls_from_several_threads(pa, gpu_device):
    """Threads with a stream each make the three calls at once, on tensors of their own."""
    errs, lock = [], threading.Lock()

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(3):
                e = _extend(pa, gpu_device, "bf16", [600 + i, 40], [1 + k, 70], 8, 2, 128, 16, seed=10 * i + k)
                with lock:
                    errs.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(errs) == 12 and max(errs) <= TOL["bf16"], errs


@pytest.mark.gpu
def test_hot_path_calls_refuse_none_for_a_number(pa, gpu_device):
    """A TypeError, raised before anything is launched."""
    slots = torch.zeros(1, dtype=torch.int32, device=gpu_device)
    x, pool = torch.zeros(1, 1, 64, device=gpu_device), torch.zeros(4096, device=gpu_device)
    ok = dict(page_size=1, num_slots=1, max_kv_len=1)
    for name in ok:
        bad = dict(ok, **{name: None})
        with pytest.raises(TypeError):
            pa.extend_attention(x, x, x, pool, slots, slots.expand(2).contiguous(), slots, slots, slots.expand(2).contiguous(), 1.0, **bad)
        bad.pop("max_kv_len")
        if name != "max_kv_len":
            with pytest.raises(TypeError):
                pa.append_kv(pool, slots, x, x, **bad)
    with pytest.raises(TypeError):
        pa.extend_attention(x, x, x, pool, slots, slots.expand(2).contiguous(), slots, slots, slots.expand(2).contiguous(), None, **ok)


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["stream object", "raw handle"])
def test_tensors_made_by_a_call_belong_to_its_stream(pa, gpu_device, how):
    """What the calls allocate themselves is used by kernels on the stream they are given, and freed by the host while these still
    wait: it has to come from that stream's share of the allocator, also where another stream is torch's current one."""
    import gc
    side = torch.cuda.Stream()
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=gpu_device)
    tree = pa.Tree()
    tree.insert(np.arange(600, dtype=np.int32), np.arange(600, dtype=np.int32))
    tree.upload()
    gen = torch.Generator(device=gpu_device).manual_seed(2)
    mk = lambda n, h: torch.randn(n, h, 128, generator=gen, dtype=torch.bfloat16, device=gpu_device)
    kw = dict(page_size=1, num_slots=600)
    pool = torch.zeros(pa.kv_pool_bytes(600, 2, 128, torch.bfloat16, 1), dtype=torch.uint8, device=gpu_device)
    pa.append_kv(pool, i32(range(600)), mk(600, 2), mk(600, 2), **kw)
    toks, off = i32(list(range(600)) + [7000] * 64), i32([0, 664])
    q, k, v, e, eo = mk(64, 8), mk(64, 2), mk(64, 2), i32([64]), i32([0, 64])

    def step(stream):
        pl, si = pa.match_prefixes(tree, toks, off, stream=stream)
        return pl, si, pa.extend_attention(q, k, v, pool, si, off, pl, e, eo, 128 ** -0.5, max_kv_len=664, stream=stream, **kw)

    want = [t.clone() for t in step(None)]
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    sizes = lambda: {s["stream"]: sum(x["total_size"] for x in torch.cuda.memory_snapshot() if x["stream"] == s["stream"])
                     for s in torch.cuda.memory_snapshot()}
    before = sizes()
    side.wait_stream(torch.cuda.current_stream())
    print(f"[case] tensors made for a side stream, {how}", flush=True)
    got = step(side if how == "stream object" else side.cuda_stream)
    torch.cuda.current_stream().wait_stream(side)
    after = sizes()
    assert after.get(0, 0) == before.get(0, 0) and after[side.cuda_stream] > before.get(side.cuda_stream, 0)
    for t in got:
        assert any(s["stream"] == side.cuda_stream and s["address"] <= t.data_ptr() < s["address"] + s["total_size"]
                   for s in torch.cuda.memory_snapshot())
    assert torch.cuda.current_stream().cuda_stream == 0
    assert torch.equal(got[0], want[0]) and torch.equal(got[1][:600], want[1][:600]) and torch.equal(got[2], want[2])


def test_hot_path_calls_refuse_what_is_no_device_tensor():
    """Checks that need no GPU: wrong kinds of arguments are refused before anything reaches the device."""
    from paper_2407_00023_amd import binding
    i32 = torch.zeros(2, dtype=torch.int32)
    x = torch.zeros(1, 2, 64)
    tree = binding.Tree()
    with pytest.raises(TypeError):
        binding.match_prefixes(tree, i32, i32)                       # tensors of the host
    with pytest.raises(TypeError):
        binding.match_prefixes(tree, i32)                            # an argument missing
    with pytest.raises(TypeError):
        binding.match_prefixes(tree, i32, i32, nonsense=1)
    with pytest.raises(TypeError):
        binding.append_kv(x, i32[:1], x, x, page_size=1, num_slots=1)
    with pytest.raises(TypeError):
        binding.append_kv(x, i32[:1], x, x, num_slots=1)             # page_size is required
    with pytest.raises(TypeError):
        binding.extend_attention(x, x, x, x, i32, i32, i32, i32, i32, 1.0, page_size=1, num_slots=1, max_kv_len=1)


# launches without a work list: up to 6 requests of up to 16 rows each on average (narrow tiles; up to 64 where they fill the slots
# in 16 parts) or of more than 48 (64 with heads of 64; tiles of 128 rows), tiles cut from 256 (narrow) and 512 or 1,024 keys on, up
# to 16 and 4 parts
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P,E,Hq,Hkv,D,page,direct", [
    ("bf16", [0], [1], 4, 1, 128, 16, True), ("bf16", [511], [1], 8, 2, 128, 16, True), ("bf16", [512], [4], 8, 2, 128, 1, True),
    ("bf16", [255, 4095, 4096, 0, 7, 5000], [1] * 6, 8, 2, 128, 16, True), ("bf16", [300] * 7, [1] * 7, 8, 2, 128, 16, False),
    ("bf16", [900, 0, 3000], [0, 11, 1], 8, 2, 64, 48, True), ("bf16", [700, 20], [1, 23], 32, 8, 64, 16, False),
    ("bf16", [0], [13], 8, 2, 128, 16, True), ("bf16", [1023 - 40, 1024 - 40], [40, 40], 8, 2, 128, 16, True),
    ("bf16", [2100, 5], [33, 64], 8, 1, 128, 16, True), ("bf16", [2400, 600, 0], [300, 97, 1], 16, 8, 64, 1, True),
    ("bf16", [0, 0, 100], [400, 0, 250], 8, 2, 128, 64, True), ("bf16", [1100] * 6, [40] * 6, 8, 2, 128, 24, True),
    ("bf16", [300 + 7 * r for r in range(12)], [1 + r % 3 for r in range(12)], 16, 8, 128, 16, True),
    ("bf16", [40 * r for r in range(40)], [1] * 40, 8, 8, 64, 16, False), ("bf16", [250] * 65, [1] * 65, 4, 4, 64, 16, False),
    ("bf16_kv8", [90 * r for r in range(9)], [1] * 9, 32, 8, 128, 16, True), ("bf16_kv8", [2000] * 20, [1] * 20, 8, 8, 64, 16, False),
    ("bf16_kv8", [700, 1500], [1, 2], 8, 2, 128, 16, True), ("bf16_kv8", [1400, 9], [70, 33], 8, 2, 64, 16, True),
    ("bf16_kv8", [1400, 9], [70, 33], 8, 2, 128, 16, True),
    ("bf16", [30 * r for r in range(20)], [190 + 3 * r for r in range(20)], 32, 32, 128, 16, True),   # four tiles per slot: launched so,
    ("bf16", [200, 0, 90, 64], [400, 390, 1, 130], 64, 64, 64, 16, True), ("bf16", [5, 0], [1600, 1600], 64, 64, 128, 16, False),
    ("bf16", [100, 40], [1536, 1537], 64, 64, 128, 16, False), ("bf16", [9, 70, 0], [1024, 1000, 1048], 64, 64, 64, 16, True)])   # and a little beyond
def test_extend_of_small_batches(pa, gpu_device, dtype, P, E, Hq, Hkv, D, page, direct):
    assert _extend(pa, gpu_device, dtype, P, E, Hq, Hkv, D, page, direct=direct) <= TOL["bf16"]


def _small_batches(pa, dev, sizes, Hq=8, Hkv=2, D=128, page=16, nslots=8192):
    """Batches (P, E) of one pool, each as a function of (workspace, output, stream), with a maker of workspaces and the result
    of a first call on a fresh one."""
    rng = np.random.default_rng(3)
    pool = torch.randn(pa.kv_pool_bytes(nslots, Hkv, D, torch.bfloat16, page) // 2, device=dev).to(torch.bfloat16).view(torch.uint8)
    tt = lambda a: torch.from_numpy(np.asarray(a, np.int32)).to(dev)

    def batch(P, E):
        off, eo = np.concatenate([[0], np.cumsum(np.add(P, E))]), np.concatenate([[0], np.cumsum(E)])
        x = lambda h: torch.randn(int(eo[-1]), h, D, device=dev).to(torch.bfloat16)
        a = [x(Hq), x(Hkv), x(Hkv), pool, tt(rng.permutation(nslots)[:off[-1]]), tt(off), tt(P), tt(E), tt(eo), D ** -0.5]
        kv = int(np.add(P, E).max())
        nbytes = pa.extend_workspace_bytes(len(P), int(eo[-1]), kv, Hq, Hkv, D, torch.bfloat16)
        b = dict(ws=lambda: torch.zeros(nbytes, dtype=torch.uint8, device=dev), out=lambda: torch.zeros_like(a[0]))
        b["run"] = lambda ws, out, stream=None, more_keys=0: pa.extend_attention(
            *a, page_size=page, num_slots=nslots, max_kv_len=kv + more_keys, out=out, workspace=ws, stream=stream)
        b["want"] = b["run"](b["ws"](), b["out"]())
        return b

    made = [batch(*s) for s in sizes]
    torch.cuda.synchronize()
    return made


_IN_PARTS = [([1500, 700], [1, 3]), ([2000], [90]), ([900, 10, 2500], [1, 1, 2]), ([1200, 1100], [40, 30])]


@pytest.mark.gpu
def test_small_batches_on_streams_and_in_graphs(pa, gpu_device):
    """Small batches cut into parts that their workgroups join: eager calls queued on four streams while a graph of 160 captured
    ones is replayed on a fifth, three times in a row.  Every single result equals the first call's bit for bit."""
    batches = _small_batches(pa, gpu_device, _IN_PARTS)
    streams, side, n, eager = [torch.cuda.Stream() for _ in batches], torch.cuda.Stream(), 40, 20
    for b in batches:
        b["eager_ws"], b["graph_ws"] = b["ws"](), b["ws"]()
        b["eager"], b["graph"] = [b["out"]() for _ in range(eager)], [b["out"]() for _ in range(n)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for k in range(n):
            for b in batches:
                b["run"](b["graph_ws"], b["graph"][k])
    for k in range(3):
        print(f"[case] small batches on streams and in graphs, round {k}", flush=True)
        for b in batches:
            for x in b["eager"] + b["graph"]:
                x.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        for b, s in zip(batches, streams):
            with torch.cuda.stream(s):
                for x in b["eager"]:
                    b["run"](b["eager_ws"], x)
        torch.cuda.synchronize()
        for b in batches:
            assert all(torch.equal(x, b["want"]) for x in b["eager"])
            assert all(torch.equal(x, b["want"]) for x in b["graph"])


@pytest.mark.gpu
def test_small_batches_on_many_streams(pa, gpu_device):
    """Calls with workspaces of their own do not depend on one another, on however many streams: 80 of them, batches whose tiles
    have different numbers of parts, six calls queued on each, every result compared."""
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    batches = _small_batches(pa, gpu_device, _IN_PARTS)
    streams = []
    for _ in range(80):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0  # (non-blocking)
        streams.append(s.value)
    per = [(batches[i % 4], batches[i % 4]["ws"](), [batches[i % 4]["out"]() for _ in range(6)]) for i in range(80)]
    torch.cuda.synchronize()
    print("[case] small batches on 80 streams", flush=True)
    for k in range(6):
        for s, (b, ws, outs) in zip(streams, per):
            b["run"](ws, outs[k], s)
    torch.cuda.synchronize()
    for b, _, outs in per:
        assert all(torch.equal(x, b["want"]) for x in outs)
    for s in streams:
        assert hip.hipStreamDestroy(ctypes.c_void_p(s)) == 0


@pytest.mark.gpu
def test_small_batches_whatever_the_workspace_holds(pa, gpu_device):
    """The words that count a tile's finished parts may hold anything before a call: zeros, ones, random bits, the tables that a
    call with a work list left there, what the same captured call left; bit for bit the same result."""
    for b in _small_batches(pa, gpu_device, _IN_PARTS):
        ws, out = b["ws"](), b["out"]()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            b["run"](ws, out)
        large = torch.zeros(1 << 28, dtype=torch.uint8, device=gpu_device)
        fills = {"zeros": lambda: ws.zero_(), "ones": lambda: ws.fill_(255), "ones at the bottom": lambda: ws.view(torch.int64).fill_(1),
                 "random": lambda: ws.random_(0, 256), "as it is": lambda: None}
        for name, fill in fills.items():
            for call in ("eager", "replay", "replay", "eager"):
                print(f"[case] small batches, workspace {name}, {call}", flush=True)
                fill()
                out.zero_()
                graph.replay() if call == "replay" else b["run"](ws, out)
                torch.cuda.synchronize()
                assert torch.equal(out, b["want"])
        for _ in range(2):  # (a call told of 1,000,000 keys more builds a list)
            b["run"](large, out, more_keys=1000000)
            assert (out.float() - b["want"].float()).abs().max() <= TOL["bf16"]
            out.zero_()
            b["run"](large, out)
            assert torch.equal(out, b["want"])


# prefixes cut into 2 to 16 parts of narrow tiles and 2 to 4 of wide ones, with and without a work list; E new tokens of G rows
@pytest.mark.gpu
@pytest.mark.parametrize("kv_more", [0, 1000000])
@pytest.mark.parametrize("P,E,G,D", [(2000, 1, 4, 128), (2000, 1, 4, 64), (700, 2, 8, 128), (1300, 11, 1, 128), (5000, 1, 1, 64), (1600, 90, 2, 128),
                                     (2600, 70, 4, 64)])
def test_extend_in_parts_with_an_infinite_value(pa, gpu_device, P, E, G, D, kv_more):
    """An infinity in a V row of the prefix makes that element of every row infinite, not NaN, whichever part of the keys it lies in
    and however many parts there are; the other elements are untouched.  (kv_more: told of as many keys more, a call builds a list.)"""
    Hkv, nslots = 2, -(-P // 16) * 16
    gen = torch.Generator(device=gpu_device).manual_seed(P + E)
    mk = lambda n, h: torch.randn(n, h, D, generator=gen, device=gpu_device).to(torch.bfloat16)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=gpu_device)
    q, k, v, pk, pv = mk(E, G * Hkv), mk(E, Hkv), mk(E, Hkv), mk(nslots, Hkv), mk(nslots, Hkv)
    kw, slots = dict(page_size=16, num_slots=nslots), torch.arange(nslots, dtype=torch.int32, device=gpu_device)

    def run(pvv):
        pool = torch.zeros(pa.kv_pool_bytes(nslots, Hkv, D, torch.bfloat16, 16), dtype=torch.uint8, device=gpu_device)
        pa.append_kv(pool, slots, pk, pvv, **kw)
        ws = torch.zeros(pa.extend_workspace_bytes(1, E, P + E + kv_more, G * Hkv, Hkv, D, torch.bfloat16), dtype=torch.uint8, device=gpu_device)
        out = pa.extend_attention(q, k, v, pool, i32(list(range(P)) + [-1] * E), i32([0, P + E]), i32([P]), i32([E]), i32([0, E]), D ** -0.5,
                                  max_kv_len=P + E + kv_more, workspace=ws, **kw)
        return out.float().cpu()

    plain = run(pv)
    for at in (3, P // 2, P - 70, P - 1):
        pvv = pv.clone()
        pvv[at, 1, 5] = float("inf")
        out = run(pvv)
        assert (out[:, G:, 5] == float("inf")).all(), at
        out[:, G:, 5] = plain[:, G:, 5]
        assert torch.equal(out, plain), at


# changes of a tree go to the device in pieces of 256 words, runs of more than 16,384 words by copies of their own
@pytest.mark.gpu
def test_upload_of_changes_at_the_edges_of_pieces_and_long_runs(pa, gpu_device):
    """After every insertion and upload the matcher finds the whole new sequence with its slots, the one before it and the first."""
    rng = np.random.default_rng(7)
    tree = pa.Tree()
    tree.insert(*(lambda n: (rng.integers(0, 1000, n).astype(np.int32), np.arange(n, dtype=np.int32)))(60000))
    tree.upload()
    cached, base = [], 100000
    for k, n in enumerate([1, 255, 256, 257, 511, 513, 16383, 16384, 16385, 300, 20000, 2]):
        toks = rng.integers(0, 1000, n).astype(np.int32)
        toks[0] = 2000 + k
        cached.append((toks, np.arange(base, base + n, dtype=np.int32)))
        base += n
        tree.insert(*cached[-1])
        tree.upload()
        print(f"[case] upload of a run of {n} tokens", flush=True)
        ask = [cached[-1], cached[max(0, k - 1)], cached[0]]
        off = np.concatenate([[0], np.cumsum([len(t) + 1 for t, _ in ask])]).astype(np.int32)
        prompt = np.concatenate([np.append(t, np.int32(5000)) for t, _ in ask])
        pl, si = pa.match_prefixes(tree, torch.from_numpy(prompt).to(gpu_device), torch.from_numpy(off).to(gpu_device))
        pl, si = pl.cpu().numpy(), si.cpu().numpy()
        for r, (t, s) in enumerate(ask):
            assert pl[r] == len(t)
            np.testing.assert_array_equal(si[off[r]:off[r] + pl[r]], s)
    full, partial, _ = tree.upload_stats()
    assert partial >= 10


# 16 workgroup slots per KV head and tiles of 35 key tiles: 4 tiles are cut in two, 16 are one round as they are, 17 are cut again
@pytest.mark.gpu
@pytest.mark.parametrize("B", [4, 16, 17])
def test_extend_cuts_tiles_or_not_around_a_round_of_workgroups(pa, gpu_device, B):
    assert _extend(pa, gpu_device, "bf16", [2100 + r % 3 for r in range(B)], [128 - r % 2 for r in range(B)], 32, 32, 128, 16, common=300,
                   kv_more=1000000, cut=B != 16) <= TOL["bf16"]


# lists ordered by length: 16 slots per KV head and just more items than one round, six rounds and just beyond, several threads of the
# planner to a tile and one, cut tiles among them; the last: the planner of more than 256 requests (64 slots, 300 tiles)
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hkv,D,E,longest", [(17, 32, 128, 60, 900), (17, 32, 128, 128, 3000), (60, 32, 64, 40, 700), (96, 32, 64, 40, 700),
                                               (97, 32, 64, 40, 700), (300, 8, 64, 33, 800)])
def test_extend_lists_of_mixed_lengths(pa, gpu_device, B, Hkv, D, E, longest):
    P = [(40, longest // 2, longest, 130, longest // 3)[r % 5] + r % 3 for r in range(B)]
    assert _extend(pa, gpu_device, "bf16", P, [E - r % 2 for r in range(B)], Hkv, Hkv, D, 16, kv_more=1000000) <= TOL["bf16"]


# The order of a list's items.  By length: new prompts (long and short tiles in each), narrow tiles only, narrow ones beside wide
# ones.  As the requests stand: one length; one round of workgroups (heads of 64: 24, three on a compute unit); more than six rounds.
@pytest.mark.gpu
@pytest.mark.parametrize("D,P,E,by_length", [
    (128, [0] * 4, [1500] * 4, True), (64, [0] * 5, [1100] * 5, True), (128, [300 + 977 * r % 2700 for r in range(40)], [4] * 40, True),
    (128, [200 + 331 * r % 1500 for r in range(24)] + [100] * 2, [3] * 24 + [1400, 900], True),
    (128, [1000] * 40, [60] * 40, False), (64, [0] * 2, [1400] * 2, False), (128, [0] * 9, [1500] * 9, False)])
def test_extend_order_of_a_list(pa, gpu_device, D, P, E, by_length):
    records = []
    assert _extend(pa, gpu_device, "bf16", P, E, 32, 32, D, 16, kv_more=1000000, records=records) <= TOL["bf16"]
    tiles = {}  # (request, first row): key tiles, items, narrow
    for r, row0, lo, hi, *rest in records:
        k, n, _ = tiles.get((r, row0), (0, 0, 0))
        tiles[r, row0] = k + -(-(hi - lo) // 64), n + 1, rest[5]
    average = sum((k + 1) // 2 if narrow else k for k, _, narrow in tiles.values()) / len(records)
    if by_length:
        ranks = []
        for r, row0, *_ in records:
            k, n, narrow = tiles[r, row0]
            length = k / n * (0.7 if narrow else 1.0) / average
            if min(abs(length - 1.1), abs(length - 0.75)) > 1e-3:  # (not as good as on a bound)
                ranks.append(0 if length > 1.1 else 1 if length > 0.75 else 2)
        assert ranks == sorted(ranks) and {0, 2} <= set(ranks)
    else:
        seen = [r for i, (r, *_) in enumerate(records) if i == 0 or records[i - 1][0] != r]
        assert len(seen) == len(set(seen)) == len(P)


# wide tiles of which one to three waves (of 32 rows) have no rows, or a single row: runs over the pool and over the new tokens
@pytest.mark.usefixtures("both_forms")
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "bf16_kv8"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("E,G", [(64, 1), (65, 1), (96, 1), (97, 1), (193, 1), (12, 4), (40, 4)])
def test_extend_waves_without_rows(pa, gpu_device, dtype, D, E, G):
    P = [0, 63, 64, 200, 1090]
    assert _extend(pa, gpu_device, dtype, P, [E] * len(P), 2 * G, 2, D, 16) <= TOL[dtype]


# scores that outgrow the running maximum by far more than 2^40 (in probability) from one key on, in the first or the second block of a
# tile: a run over the pool, or over the new tokens, is left there (the fp8 pool: with the next tile's rows still codes), single tiles on the diagonal too
@pytest.mark.usefixtures("both_forms")
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "bf16_kv8"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("at", [64 * 9 + 5, 64 * 9 + 37])
@pytest.mark.parametrize("P,E", [([1300, 1257], [150, 70]), ([320, 300], [700, 450])], ids=["pool", "new tokens"])
def test_extend_scores_that_outgrow_the_running_maximum(pa, gpu_device, dtype, D, at, P, E):
    assert _extend(pa, gpu_device, dtype, P, E, 8, 2, D, 16, louder_from=at) <= TOL[dtype]


# narrow tiles in a list: uncut only where every round of workgroups is at least half full (8, 4 and 2 KV heads: 64, 128 and 256 slots)
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hkv,D,P,cut", [(12, 8, 128, 1000, True), (12, 8, 64, 1000, True), (32, 4, 64, 1000, True), (70, 2, 128, 1000, True),
                                           (70, 8, 64, 520, True), (31, 8, 64, 600, True), (32, 8, 64, 600, False), (48, 8, 64, 600, False),
                                           (64, 8, 64, 600, False), (7, 1, 128, 1000, True)])
def test_extend_cuts_narrow_tiles_or_not(pa, gpu_device, B, Hkv, D, P, cut):
    assert _extend(pa, gpu_device, "bf16", [P + r % 3 for r in range(B)], [1] * B, 4 * Hkv, Hkv, D, 16, kv_more=1000000, cut=cut) <= TOL["bf16"]


# where a list would cut further than the 16 (narrow tiles) or 4 parts of a launch without one, up to which length of a part such
# launches are made, in keys that the call is told of: 34 tiles of 64 keys (fp8 pool: 20), on an almost empty chip 20 (16), wide tiles 32
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,B,E,Hkv,G,D,told,direct", [
    ("bf16", 1, 1, 1, 8, 128, 262144, False), ("bf16", 1, 1, 1, 8, 128, 20480, True), ("bf16", 1, 1, 1, 8, 128, 20481, False),
    ("bf16", 1, 1, 8, 4, 64, 34816, True), ("bf16", 1, 1, 8, 4, 64, 34817, False), ("bf16", 2, 1, 2, 8, 128, 34816, True),
    ("bf16", 2, 1, 2, 8, 128, 34817, False), ("bf16", 4, 2, 2, 8, 64, 65000, False), ("bf16_kv8", 1, 1, 1, 8, 128, 16384, True),
    ("bf16_kv8", 1, 1, 1, 8, 128, 16385, False), ("bf16_kv8", 1, 1, 8, 4, 64, 20480, True), ("bf16_kv8", 1, 1, 8, 4, 64, 20481, False),
    ("bf16", 18, 30, 4, 4, 128, 2048, True), ("bf16", 18, 30, 4, 4, 128, 2049, False), ("bf16", 12, 30, 4, 4, 128, 4096, True),
    ("bf16", 12, 30, 4, 4, 128, 4097, False), ("bf16", 4, 100, 8, 4, 128, 5600, True)])
def test_extend_of_long_requests_takes_a_list(pa, gpu_device, dtype, B, E, Hkv, G, D, told, direct):
    assert _extend(pa, gpu_device, dtype, [40 + r for r in range(B)], [E] * B, G * Hkv, Hkv, D, 16, kv_more=told - (39 + B + E),
                   direct=direct) <= TOL[dtype]
