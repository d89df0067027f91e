"""GPU parity tests (run with -m gpu): the HIP path through the C ABI against the fp64
oracle, element by element, on seeded inputs that span several tiles and ragged tails."""
import numpy as np
import pytest

from oracle import shard as osh
from paper_2503_17924_amd import binding as B
from paper_2503_17924_amd import workloads as wl
from gpu_helpers import Case, check_close

pytestmark = pytest.mark.gpu


def _cu(docs):
    return np.concatenate([[0], np.cumsum(docs)]).astype(np.int32)


def _small(seed, docs, hq, hkv, d, cp=1, rank=0, mode=0):
    w, tens = wl.small_case(seed, docs, hq, hkv, d)
    sh = osh.shard(docs, cp, rank, mode)
    return Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)


FWD_CASES = [
    # docs, hq, hkv, d, cp
    ([300, 45, 1, 700, 130], 4, 2, 128, 1),        # several tiles, ragged tail, 1-token document
    ([64, 64, 128], 2, 2, 64, 1),                  # tile-aligned documents, head_dim 64
    ([1] * 70, 2, 1, 128, 1),                      # only single-token documents
    ([1000], 8, 1, 128, 1),                        # one document, GQA 8:1
    ([3], 1, 1, 64, 1),                            # fewer rows than a tile
    ([5, 900, 2, 3, 333, 64, 1, 77], 4, 4, 64, 2), # per-document sharding with padding
    ([517, 3, 40, 1200], 8, 2, 128, 4),            # documents shorter than 2*CP chunks -> empty chunks
]


@pytest.mark.parametrize("docs,hq,hkv,d,cp", FWD_CASES)
def test_forward_matches_oracle(docs, hq, hkv, d, cp):
    for r in range(cp):
        c = _small(20 + r, docs, hq, hkv, d, cp, r, osh.PER_DOC_PADDED)
        c.check_fwd(f" rank {r}")


def test_forward_per_sequence_sharding():
    docs = [700, 41, 3, 1000, 304]        # T = 2048, divisible by 2*CP
    for r in range(4):
        c = _small(31, docs, 4, 1, 128, 4, r, osh.PER_SEQ)
        c.check_fwd(f" rank {r}")


def test_forward_all_padding_rows():
    w, tens = wl.small_case(5, [40], 2, 1, 64)
    c = Case(tens, np.full(70, -1, dtype=np.int32), _cu([40]), 2, 1, 64, w.scale)
    o, lse = c.run_fwd()
    assert (o == 0).all() and np.isneginf(lse).all()


def test_out_of_range_row_indices_are_padding():
    """q_idx entries outside [0, t_kv) other than -1 are treated like -1 (stated in the header)."""
    import torch
    docs = [200, 57, 1]
    t = sum(docs)
    w, tens = wl.small_case(33, docs, 2, 1, 64)
    clean = np.arange(t, dtype=np.int32)
    bad = np.array([3, 64, 199, 200, 256, 257], dtype=np.int64)
    clean[bad] = -1
    c = Case(tens, clean, _cu(docs), 2, 1, 64, w.scale)
    dirty = clean.copy()
    dirty[bad] = np.array([-5, t, t + 1000, 2**31 - 1, -2**31, -2], dtype=np.int64).astype(np.int32)
    c.attn.q_idx.copy_(torch.from_numpy(dirty))
    c.check_fwd()
    c.check_bwd()


def test_one_token():
    for d in (64, 128):
        c = _small(34, [1], 1, 1, d)
        o, lse = c.run_fwd()
        assert np.array_equal(o[0, 0], c.f64("v")[0, 0])          # a one-token document returns its own V
        c.check_fwd()
        c.check_bwd()


def test_forward_rows_in_arbitrary_order():
    # the mask is per row; nothing requires q_idx to be sorted
    docs = [200, 333, 90]
    w, tens = wl.small_case(6, docs, 2, 2, 128)
    rng = np.random.default_rng(0)
    q_idx = rng.permutation(sum(docs)).astype(np.int32)[:400]
    q_idx[::17] = -1
    Case(tens, q_idx, _cu(docs), 2, 2, 128, w.scale).check_fwd()


@pytest.mark.parametrize("flag", [B.ATTN_SCHEDULE_GANGS, B.ATTN_SCHEDULE_ITEMS])
def test_wavefront_with_rows_of_two_chunks_and_three_documents(flag):
    """32 consecutive rows (one wavefront of the forward and dQ kernels) that hold rows of an early and of a late
    chunk of one long document, rows of a second document and a row of a third, padding in between: the kernels
    cross the keys between the chunks, and the other documents' keys, with whole lanes switched off, in several
    ranges.  Every output element against the oracle, forward and backward."""
    docs = [2000, 700, 300, 77]
    cu = _cu(docs)
    rows = ([int(cu[0]) + i for i in range(0, 9)] + [-1, -1] + [int(cu[0]) + 1900 + i for i in range(7)]
            + [int(cu[1]) + 130 + 3 * i for i in range(8)] + [-1] + [int(cu[2]) + 299] + [int(cu[1]) + 699, int(cu[1]), -1, int(cu[0]) + 1999])
    assert len(rows) == 32
    # a second wavefront of ordinary rows and a third that starts in the last document
    rows += [int(cu[0]) + 640 + i for i in range(32)] + [int(cu[3]) + i for i in range(20)]
    w, tens = wl.small_case(97, docs, 8, 2, 128)
    c = Case(tens, np.asarray(rows, dtype=np.int32), cu, 8, 2, 128, w.scale)
    c.flags = flag
    c.check_fwd(" mixed wavefront")
    c.check_bwd(" mixed wavefront")


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_shapes_match_oracle(seed):
    """A seeded sweep over valid small inputs: document mixes (tiny, mixed, one long plus tiny, medium), head counts
    with groups of 1 to 8 query heads per KV head, both head dimensions, CP 1 to 4 with padded and padding-free maps,
    every schedule flag, and for some cases shuffled rows with extra padding.  Forward and backward, every element."""
    rng = np.random.default_rng(seed)
    for it in range(25):
        n_docs = int(rng.integers(1, 12))
        kind = int(rng.integers(0, 4))
        if kind == 0:
            docs = rng.integers(1, 70, size=n_docs * 6).tolist()
        elif kind == 1:
            docs = rng.integers(1, 1500, size=n_docs).tolist()
        elif kind == 2:
            docs = [int(rng.integers(1500, 4000))] + rng.integers(1, 100, size=n_docs).tolist()
        else:
            docs = rng.integers(100, 700, size=n_docs).tolist()
        if sum(docs) > 6000:
            docs = docs[:max(1, len(docs) // 2)]
        hkv = int(rng.choice([1, 2, 3, 4]))
        hq = hkv * int(rng.choice([1, 2, 3, 4, 5, 7, 8]))
        if hq > 16:
            hq, hkv = 8, 2
        d = int(rng.choice([64, 128]))
        cp = int(rng.choice([1, 1, 2, 3, 4]))
        rank = int(rng.integers(0, cp))
        mode = int(rng.choice([osh.PER_DOC_PADDED, osh.PER_DOC_NOPAD])) if cp > 1 else osh.PER_DOC_PADDED
        flag = int(rng.choice([0, B.ATTN_SCHEDULE_GANGS, B.ATTN_SCHEDULE_ITEMS, B.ATTN_SCHEDULE_ITEMS | B.ATTN_NO_SHORT_PATH]))
        tag = f" seed {seed} case {it}: docs {docs} hq {hq} hkv {hkv} d {d} cp {cp} rank {rank} mode {mode} flag {flag}"
        w, tens = wl.small_case(1000 * seed + it, docs, hq, hkv, d)
        sh = osh.shard(docs, cp, rank, mode)
        q_idx = sh["q_idx"].copy()
        if rng.random() < 0.3 and len(q_idx) > 4:
            q_idx = rng.permutation(q_idx)
            q_idx[rng.integers(0, len(q_idx), size=max(1, len(q_idx) // 10))] = -1
        c = Case(tens, q_idx, sh["cu_seqlens_k"], hq, hkv, d, w.scale)
        c.flags = flag
        c.check_fwd(tag)
        c.check_bwd(tag)


def test_forward_config0_both_ranks():
    w = wl.config(0)
    tens = w.tensors(names=("q", "k", "v"))
    for r in range(2):
        sh = B.wlb_shard(w.doc_len, 2, r, B.SHARD_PER_DOC_PADDED)
        Case(tens, sh["q_idx"], sh["cu_seqlens_k"], w.hq, w.hkv, w.head_dim, w.scale).check_fwd(f" rank {r}")


def test_forward_is_deterministic_and_plan_reuse_changes_nothing():
    c = _small(40, [900, 50, 400], 4, 2, 128)
    o1, l1 = c.run_fwd()
    o2, l2 = c.run_fwd()              # second call reuses the schedule in the workspace
    assert np.array_equal(o1, o2) and np.array_equal(l1, l2)


@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (6, 2, 64), (12, 1, 128), (3, 3, 64), (16, 1, 128), (32, 2, 64)])
@pytest.mark.parametrize("flag", [B.ATTN_SCHEDULE_GANGS, B.ATTN_SCHEDULE_ITEMS])
def test_both_row_schedules_match_oracle(flag, hq, hkv, d):
    """Forward and dQ have two work schedules (fixed gangs with tiles cut at share ends and merged
    from partial results / one workgroup per tile and head); both forced here on an input with
    documents from 1 token to several tiles, pads, and tiles that straddle documents, for head
    groups of 1, 2, 3, 12 and 16 query heads per KV head and both head dimensions."""
    docs = [900, 1, 37, 2600, 130, 64, 700]
    w, tens = wl.small_case(77, docs, hq, hkv, d)
    for cp, r in ((1, 0), (2, 1)):
        sh = osh.shard(docs, cp, r, osh.PER_DOC_PADDED)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)
        c.flags = flag
        c.check_fwd(f" cp {cp} rank {r}")
        c.check_bwd(f" cp {cp} rank {r}")


def check_work_records(attn):
    """The records that the kernels start from, against the schedule's tables: whole tiles; parts that cover their tile's
    key tiles without a gap, with partial results of their own inside the workspace; dK/dV items.  Returns the tables."""
    t = B.plan_tables(attn)
    lay, rec = t["layout"], t["records"]
    hq, hkv = attn.shape[3], attn.shape[4]
    G = hq // hkv
    order, cost = t["fwd_order"], t["fwd_cost"]
    item, part, base = t["row_item"], t["row_part"], t["row_part_base"]
    assert (item[:, 0] == order).all() and (item[:, 2] - item[:, 1] == cost[order]).all()
    assert (item[:, 3] == np.where(t["tile_short"][order] == 1, -2, -1)).all()
    group = t["group"]
    for tile in range(lay.n_fwd_tiles):
        g = group[2 * tile:2 * tile + 2]
        g = g[g[:, 1] > g[:, 0]]
        r = int(np.nonzero(order == tile)[0][0])
        assert item[r, 1] == (g[:, 0].min() // 64 if len(g) else 0)
    count = base[:-1, 1]
    assert (count >= 1).all() and base[-1, 0] == count.sum() == len(part) <= rec.max_parts
    partials, at, longest = [], [], []
    for r in range(lay.n_fwd_tiles):
        mine = part[base[r, 0]:base[r, 0] + count[r]]
        at += range(base[r, 0], base[r, 0] + count[r])
        is_short = t["tile_short"][order[r]]
        assert not is_short or len(mine) == 1
        longest.append((0 if is_short and rec.uses_parts else -(mine[:, 2] - mine[:, 1]).max(), order[r], base[r, 0]))
        if len(mine) == 1:
            assert (mine[0] == item[r]).all()
            continue
        assert (mine[:, 0] == order[r]).all()
        assert mine[0, 1] == item[r, 1] and mine[-1, 2] == item[r, 2] and (mine[1:, 1] == mine[:-1, 2]).all()
        size = mine[:, 2] - mine[:, 1]
        assert size.min() >= 1 and size.max() - size.min() <= 1
        assert (mine[:, 3] >= 0).all() and ((mine[:, 3] & 1) == (np.arange(len(mine)) > 0)).all()
        slots = mine[:, 3] >> 1
        assert (slots == base[r, 2] + np.arange(len(mine))).all()
        partials += slots.tolist()
    assert sorted(at) == list(range(len(part)))
    assert [x[2] for x in sorted(longest)] == sorted(x[2] for x in longest)         # longest part first (short-hull: last), ties by tile
    assert len(set(partials)) == len(partials)
    if partials:
        assert (max(partials) + 1) * hq * rec.row_partial_bytes <= rec.row_partials_bytes
    want, end = [], 0
    for r, kt in enumerate(t["key_order"]):
        first, last = t["key_range"][kt]
        ways = int(t["key_ways"][kt])
        nh = G // ways
        for hk in range(hkv):
            for p in range(ways):
                slot = t["key_slot_base"][r] + hk * ways + p if ways > 1 else -1
                want.append([kt, hk, hk * G + p * nh, nh, slot, first, (last - first) * nh])
    assert (t["dkv_item"][:, :7] == np.asarray(want)).all()
    longest = (t["key_range"][:, 1] - t["key_range"][:, 0]).max()
    assert not t["short_keys_on"] or longest <= rec.short_span
    return t


@pytest.mark.parametrize("docs,hq,hkv,d,cp", [
    ([384, 385, 1], 2, 1, 128, 1),               # 6 key tiles: whole; 7: two parts, one key tile apart
    ([5000], 4, 4, 64, 8),                       # rows of two chunks, tiles of 5 - 79 key tiles in many parts
    ([2600, 3, 700], 6, 2, 128, 2),              # pads, three query heads per KV head
    ([1500, 40, 9], 32, 8, 64, 1),               # more than one workgroup per compute unit: the second half reversed
])
def test_divided_query_tiles_match_oracle(docs, hq, hkv, d, cp):
    """Launches with few items divide heavy query tiles along their keys and merge the parts (forward, dQ); the tables
    of the schedule, and the results against the oracle, at the default schedule choice."""
    w, tens = wl.small_case(78, docs, hq, hkv, d)
    for r in sorted({0, cp - 1}):
        sh = osh.shard(docs, cp, r, osh.PER_DOC_PADDED)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)
        assert not B.wlb_attn_plan_layout(c.attn.desc).uses_gangs
        c.check_fwd(f" cp {cp} rank {r}")
        c.check_bwd(f" cp {cp} rank {r}")
        check_work_records(c.attn)


@pytest.mark.parametrize("docs,hq,hkv,d,cp,mode", [
    ([384, 385, 1, 3000], 2, 1, 128, 1, 0),      # a tile of 6 key tiles whole, one of 7 in two parts
    ([5000, 500], 4, 4, 64, 8, 0),               # rows of two chunks, tiles of up to 79 key tiles in many parts
    ([2600, 3, 700], 6, 2, 128, 2, 0),           # pads, three query heads per KV head
    ([8000], 2, 1, 64, 1, 0),                    # more than 4096 rows: the schedule's three launches
    ([300, 4600, 3, 300], 4, 2, 128, 1, 0),      # the same with more than 128 items
    ([9000, 40, 3000], 1, 1, 64, 2, 1),          # and with rows of two distant places in one tile
])
def test_divided_query_tiles_and_their_records(docs, hq, hkv, d, cp, mode):
    """Query tiles divided along their keys at the default schedule choice, by the one-launch and the three-launch
    schedule: the limit, the records, and the merged results against the oracle."""
    import torch
    if mode == osh.PER_SEQ:
        docs = docs + [2 * cp - sum(docs) % (2 * cp)]
    w, tens = wl.small_case(78, docs, hq, hkv, d)
    for r in sorted({0, cp - 1}):
        sh = osh.shard(docs, cp, r, mode)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)
        c.attn.visible_pairs = int(sh["useful_pairs"])
        c.attn.desc, c.attn.desc_reuse = c.attn.make_desc(0), c.attn.make_desc(B.ATTN_REUSE_PLAN)
        assert B.wlb_attn_plan_records(c.attn.desc).uses_parts
        c.check_fwd(f" cp {cp} rank {r}")
        c.check_bwd(f" cp {cp} rank {r}")
        t = check_work_records(c.attn)
        # a part holds at most 6 key tiles, or 6 / 4 of the mean work of a workgroup slot; more than a compute unit's mean
        # work in one tile; short-hull tiles count as none
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
        lay = t["layout"]
        work = np.where(t["tile_short"] == 1, 0, t["fwd_cost"]).astype(np.int64)
        assert work.max() >= 1.1 * work.sum() * hq / n_cu
        slots = lay.row_gangs * (hq // hkv) // hq * hq
        units = (int(work.sum()) + ROW_ITEM_OVERHEAD * lay.n_fwd_tiles) * hq
        limit = max(6, -(-(units * 6 // 4) // slots))
        parts = t["row_part_base"][:-1, 1]
        assert (parts == np.maximum(1, -(-work[t["fwd_order"]] // limit))).all()
        assert parts.max() > 1


@pytest.mark.parametrize("long,hq,hkv,d", [(2000, 4, 4, 64), (4000, 2, 1, 128)])       # one and three launches of the schedule
def test_short_hull_tiles_of_distant_blocks_stay_whole(long, hq, hkv, d):
    """Blocks of 32 rows from documents all over the sequence side by side in a query tile: each fits the short-hull window,
    the tile's hull is wide.  Beside divided tiles of a long document they stay whole short-hull tiles."""
    docs = [64] * 32 + [long]
    t_kv = sum(docs)
    blocks = np.random.default_rng(6).permutation(64).repeat(32) * 32 + np.tile(np.arange(32), 64)
    q_idx = np.concatenate([blocks, np.arange(2048, t_kv)])
    w, tens = wl.small_case(83, docs, hq, hkv, d)
    c = Case(tens, q_idx, _cu(docs), hq, hkv, d, w.scale)
    c.attn.visible_pairs = sum(n * (n + 1) // 2 for n in docs)
    c.attn.desc, c.attn.desc_reuse = c.attn.make_desc(0), c.attn.make_desc(B.ATTN_REUSE_PLAN)
    c.check_fwd()
    t = check_work_records(c.attn)
    assert t["records"].uses_parts and t["row_part_base"][:-1, 1].max() > 1
    wide = (t["tile_short"] == 1) & (t["fwd_cost"] > 12)
    assert wide.sum() > 8
    assert (t["row_part"][np.isin(t["row_part"][:, 0], np.nonzero(wide)[0]), 3] == -2).all()
    c.check_bwd()


@pytest.mark.parametrize("t_kv,n_q,hq,hkv", [(40000, 200, 1, 1), (20000, 300, 2, 1)])      # three launches of the schedule, one
def test_query_tiles_of_hundreds_of_parts(t_kv, n_q, hq, hkv):
    """The last rows of a long document: two or three query tiles, each in as many parts as fill the GPU."""
    w, tens = wl.small_case(84, [t_kv], hq, hkv, 64)
    c = Case(tens, np.arange(t_kv - n_q, t_kv), _cu([t_kv]), hq, hkv, 64, w.scale)
    c.check_fwd()
    c.check_bwd()
    t = check_work_records(c.attn)
    assert t["row_part_base"][:-1, 1].max() > 50


@pytest.mark.parametrize("docs,hq,hkv,cp,divided", [
    ([3808], 32, 4, 2, False),             # the heaviest tile has the mean work of a compute unit
    ([3328] * 8, 8, 8, 4, False),          # the same with the three-launch schedule
    ([8144], 16, 2, 4, True),
    ([12000], 4, 4, 2, True),
])
def test_query_tiles_stay_whole_where_the_launch_is_balanced(docs, hq, hkv, cp, divided):
    import torch
    sh = osh.shard(docs, cp, 0, osh.PER_DOC_PADDED)
    attn = B.Attention(sh["q_idx"], sh["cu_seqlens_k"], sum(docs), hq, hkv, 128, 0.09, visible_pairs=int(sh["useful_pairs"]))
    assert B.wlb_attn_plan_records(attn.desc).uses_parts
    attn.plan()
    torch.cuda.synchronize()
    t = check_work_records(attn)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert (t["fwd_cost"].max() >= 1.1 * t["fwd_cost"].sum() * hq / n_cu) == divided
    assert (t["row_part_base"][:-1, 1].max() > 1) == divided


@pytest.mark.parametrize("hq,hkv,d,cp,rank,mode", [
    (8, 1, 128, 4, 1, osh.PER_DOC_PADDED), (8, 2, 128, 4, 2, osh.PER_DOC_NOPAD), (32, 2, 128, 8, 7, osh.PER_DOC_PADDED), (12, 1, 64, 4, 0, osh.PER_DOC_PADDED),
    (6, 1, 128, 4, 0, osh.PER_SEQ), (16, 4, 64, 4, 3, osh.PER_DOC_NOPAD), (5, 1, 64, 4, 2, osh.PER_SEQ)])
@pytest.mark.parametrize("docs", [
    # (not fewer tokens: the mean error of 2e-3 of the largest element holds for tensors whose largest element is three times the mean
    # of all; a dK of three rows, each element off by up to three roundings of 2^-9, is at 2.0e-3)
    [35], [1] * 70,                                # short-hull tiles alone, or another launch
    [64, 1, 33, 7, 48] * 9 + [5],
    [90, 3, 700, 40, 1, 17] + [31] * 40])          # a hull of three windows of keys
def test_short_documents_divided_among_ranks(hq, hkv, d, cp, rank, mode, docs):
    """Launches whose units hold the keys of a block of rows for all heads of a KV head (taken with the pair count of short documents)."""
    if mode == osh.PER_SEQ:
        docs = docs + [-sum(docs) % (2 * cp)] if sum(docs) % (2 * cp) else docs
    w, tens = wl.small_case(97, docs, hq, hkv, d)
    sh = osh.shard(docs, cp, rank, mode)
    if len(sh["q_idx"]) == 0:
        pytest.skip("no rows on this rank")
    c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale, visible_pairs=30 * len(sh["q_idx"]))
    if len(docs) > 2 and max(docs) > 1:
        c.attn.plan()
        t = B.plan_tables(c.attn)
        assert t["layout"].row_kernels == B.ROW_SPAN and (mode == osh.PER_SEQ or (t["tile_short"] == 0).any())
    if not (sh["q_idx"] >= 0).any():                   # padding alone
        o, lse = c.run_fwd()
        assert (o == 0).all() and np.isneginf(lse).all() and all((x == 0).all() for x in c.run_bwd())
        return
    c.check_fwd(f" span {hq}/{hkv} d{d} cp{cp}")
    c.check_bwd(f" span {hq}/{hkv} d{d} cp{cp}")


@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 128), (4, 1, 64), (16, 1, 64), (10, 2, 128)])
@pytest.mark.parametrize("n_q", [24, 31, 33, 65, 129])
def test_units_of_few_rows_in_any_order(n_q, hq, hkv, d):
    """Launches of a few units whose rows lie all over the sequence, in no order, padding that holds NaN and Inf among them: a last block of one
    row, blocks that end inside one, fewer and more heads than wavefronts.  The keys of a block fill one window, two, and three."""
    import torch
    t_kv = 16 * n_q // 3
    docs = [50, 3, 40, 1, 22] * 6
    docs = docs[:int(np.searchsorted(np.cumsum(docs), t_kv))]
    docs.append(t_kv - sum(docs))
    rng = np.random.default_rng(n_q)
    q_idx = rng.choice(t_kv, n_q, replace=False).astype(np.int32)
    pad = rng.choice(n_q - 1, n_q // 7, replace=False)         # (the last row is one)
    q_idx[pad] = -1
    w, tens = wl.small_case(99, docs, hq, hkv, d)
    c = Case(tens, q_idx, _cu(docs), hq, hkv, d, w.scale, visible_pairs=20 * n_q)
    for name in ("q", "do"):
        t = c.dev[name].view(dtype=torch.int16)
        t[pad[0::2]] = 0x7FC0
        t[pad[1::2]] = 0x7F80
    c.attn.plan()
    t = B.plan_tables(c.attn)
    assert t["layout"].row_kernels == B.ROW_SPAN and not t["tile_short"][0]
    c.check_fwd()
    c.check_bwd()


@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 128), (8, 2, 128), (16, 2, 64), (10, 2, 128), (24, 4, 64)])
def test_contiguous_short_documents_in_launches_of_units(hq, hkv, d):
    """Contiguous chunks of short documents: query tiles whose blocks are short-hull units, two to a workgroup, in the same launch as units
    of rows of distant places; blocks of padding alone beside blocks with rows, a last tile of one row, padding that holds NaN and Inf."""
    import torch
    docs = [21, 40, 5, 64, 33, 1, 50] * 12
    t_kv = sum(docs)
    near = np.arange(256, dtype=np.int32) + 700
    near[32:64] = near[96:160] = near[250:] = -1
    apart = np.random.default_rng(7).permutation(t_kv)[:128].astype(np.int32)
    q_idx = np.concatenate([near, apart, np.arange(128, dtype=np.int32), [t_kv - 1]])
    w, tens = wl.small_case(98, docs, hq, hkv, d)
    c = Case(tens, q_idx, _cu(docs), hq, hkv, d, w.scale, visible_pairs=20 * len(q_idx))
    pad = np.nonzero(q_idx < 0)[0]
    for name in ("q", "do"):
        t = c.dev[name].view(dtype=torch.int16)
        t[pad[0::2]] = 0x7FC0
        t[pad[1::2]] = 0x7F80
    c.check_fwd()
    c.check_bwd()
    t = B.plan_tables(c.attn)
    assert t["layout"].row_kernels == B.ROW_SPAN and t["tile_short"].tolist() == [1, 1, 0, 1, 1]


@pytest.mark.parametrize("hq,hkv,d,cp,rank,mode,docs", [
    # shares of a gang: tiles cut anywhere, pieces of a few keys, a last tile of 5 rows, padding, two heads and eight to a KV head
    (8, 1, 128, 2, 1, osh.PER_DOC_PADDED, [2600, 1, 37, 900, 130, 64, 705]),
    (4, 2, 128, 1, 0, osh.PER_DOC_PADDED, [1, 128, 129, 63, 1000, 2, 700]),
    (8, 1, 64, 2, 0, osh.PER_DOC_NOPAD, [2600, 1, 37, 900, 130, 64, 705]),
    (6, 1, 64, 1, 0, osh.PER_DOC_PADDED, [300]),
    # items: 1536 and more
    (64, 2, 128, 1, 0, osh.PER_DOC_PADDED, [5, 1300, 64, 31, 1, 33, 90, 1149] + [17, 1, 64, 40] * 4),
    (128, 64, 128, 4, 3, osh.PER_DOC_PADDED, [3, 4000, 1700, 7, 290])])
def test_two_heads_to_a_workgroup(hq, hkv, d, cp, rank, mode, docs):
    """Launches that take two query heads to a workgroup (chosen by the pair count that the caller states, here far more than there are)."""
    w, tens = wl.small_case(91, docs, hq, hkv, d)
    sh = osh.shard(docs, cp, rank, mode)
    c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale, visible_pairs=10 ** 12)
    lay = B.wlb_attn_plan_layout(c.attn.desc)
    assert bool(lay.uses_gangs) == (hq < 64)
    assert lay.row_kernels == B.ROW_FWD_TWO_HEADS + (B.ROW_DQ_TWO_HEADS if d == 128 else 0)
    c.check_fwd(f" pairs {hq}/{hkv} d{d}")
    c.check_bwd(f" pairs {hq}/{hkv} d{d}")
    if lay.uses_gangs:
        assert f"gangs of {hq // hkv // 2} workgroups" in B.plan_report(c.attn)
    # a maximum that rises along the keys, so that what is accumulated is rescaled again and again
    ramp = c.torch.linspace(0.2, 4.0, c.t_kv, device="cuda")[:, None, None]
    q0, k0 = c.dev["q"], c.dev["k"]
    c.dev["k"] = (k0.float().abs() * ramp).bfloat16()
    c.dev["q"] = (q0.float().abs() * 3).bfloat16()
    for name in ("q", "k"):
        c.bits[name] = c.dev[name].view(c.torch.int16).cpu().numpy().view(np.uint16)
    c.check_fwd(f" rising maxima {hq}/{hkv} d{d}")


@pytest.mark.parametrize("hq,hkv,d,shuffled", [(8, 1, 128, False), (8, 1, 128, True), (4, 2, 128, True), (8, 2, 64, True), (64, 2, 128, False), (64, 2, 128, True)])
def test_two_heads_to_a_workgroup_with_garbage_in_padding(hq, hkv, d, shuffled):
    """The same launches (shares of gangs, whose cut tiles are merged, and from 64 heads on items) on rows in no order, and padding rows
    that hold NaN and Inf: they reach nothing else, and beside keys and values that are not finite their O and dQ are 0."""
    import torch
    docs = [1300, 1, 37, 900, 130, 64, 705]
    t_kv = sum(docs)
    w, tens = wl.small_case(92, docs, hq, hkv, d)
    rng = np.random.default_rng(3)
    q_idx = rng.permutation(t_kv).astype(np.int32) if shuffled else np.arange(t_kv, dtype=np.int32)
    q_idx = np.insert(q_idx, np.arange(5, t_kv, 41), -1)
    pad = np.nonzero(q_idx < 0)[0]
    c = Case(tens, q_idx, _cu(docs), hq, hkv, d, w.scale, visible_pairs=10 ** 12)
    lay = B.wlb_attn_plan_layout(c.attn.desc)
    assert bool(lay.uses_gangs) == (hq < 64) and lay.row_kernels == B.ROW_FWD_TWO_HEADS + (B.ROW_DQ_TWO_HEADS if d == 128 else 0)
    for name in ("q", "do"):
        t = c.dev[name].view(dtype=torch.int16)
        t[pad[0::2]] = 0x7FC0          # NaN
        t[pad[1::2]] = 0x7F80          # +Inf
    c.check_fwd()
    c.check_bwd()
    for name in ("k", "v"):
        t = c.dev[name].view(dtype=torch.int16)
        t[0::7, :, 3] = 0x7F80
        t[2::7, :, d - 1] = 0x7FC0
    o, lse = c.run_fwd()
    dq, _, _ = c.run_bwd()
    assert (o[pad] == 0).all() and np.isneginf(lse[:, pad]).all() and (dq[pad] == 0).all()


def test_gang_share_weights_change_the_cuts_not_the_result():
    """wlb_attn_set_gang_weights: very uneven weights (by half of the launch and by XCD) move the points where
    query tiles are cut between gangs; the results still match the oracle, and the defaults come back."""
    docs = [2600, 1, 37, 900, 130, 64, 700]
    w, tens = wl.small_case(79, docs, 8, 1, 128)
    sh = osh.shard(docs, 2, 1, osh.PER_DOC_PADDED)
    c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], 8, 1, 128, w.scale)
    c.flags = B.ATTN_SCHEDULE_GANGS
    o0, _ = c.run_fwd()
    try:
        B.wlb_attn_set_gang_weights(0, [100, 5, 60, 1000, 7, 300, 90, 33, 11, 250, 40, 40, 900, 2, 75, 120])
        B.wlb_attn_set_gang_weights(1, [3, 500, 60, 10, 700, 30, 90, 330, 110, 25, 400, 4, 90, 200, 75, 12])
        c.check_fwd(" uneven weights")
        c.check_bwd(" uneven weights")
        with pytest.raises(B.WlbError):
            B.wlb_attn_set_gang_weights(0, [0] * 16)
        with pytest.raises(B.WlbError):
            B.wlb_attn_set_gang_weights(2, [1] * 16)
    finally:
        B.wlb_attn_set_gang_weights(0, None)
        B.wlb_attn_set_gang_weights(1, None)
    o1, _ = c.run_fwd()
    assert np.array_equal(o0, o1), "default weights restored: same cuts, same bits"


def test_gang_weights_calibrated_from_the_clocks_keep_the_result():
    """binding.calibrate_gang_weights: XCD factors measured from the gangs' recorded clocks on the caller's own
    launches; positive weights in the documented range result, the halves keep their default ratio, and forward
    and backward still match the oracle."""
    docs = [3000, 5, 1200, 64, 333]
    w, tens = wl.small_case(83, docs, 8, 2, 128)
    sh = osh.shard(docs, 1, 0, osh.PER_DOC_PADDED)
    c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], 8, 2, 128, w.scale)
    c.flags = B.ATTN_SCHEDULE_GANGS
    default = [B.wlb_attn_get_gang_weights(k).copy() for k in (0, 1)]
    try:
        def launch():
            c.run_fwd()
            c.run_bwd()
        factors = B.calibrate_gang_weights([c.attn], launch, rounds=2, extra_flags=B.ATTN_SCHEDULE_GANGS)
        assert factors is not None and len(factors["fwd"]) == 8 and len(factors["dq"]) == 8
        for k, name in enumerate(("fwd", "dq")):
            got = B.wlb_attn_get_gang_weights(k).astype(np.float64).reshape(2, 8)
            assert (got >= 1).all() and (got <= 1e6).all()
            f = np.asarray(factors[name])
            assert (f >= 0.8).all() and (f <= 1.25).all()
            want = default[k].astype(np.float64).reshape(2, 8) * f[None, :] * 10.0
            assert np.abs(got - want).max() <= 1.0      # rounding to integers plus the factors' four decimals
        c.check_fwd(" calibrated weights")
        c.check_bwd(" calibrated weights")
        assert B.calibrate_gang_weights([c.attn], launch) is None, "without the flag this problem does not use gangs"
    finally:
        B.wlb_attn_set_gang_weights(0, None)
        B.wlb_attn_set_gang_weights(1, None)
    assert all(np.array_equal(B.wlb_attn_get_gang_weights(k), default[k]) for k in (0, 1))


def test_plan_tables_and_report_describe_the_schedule():
    """binding.plan_tables / plan_report: the host view of the schedule holds the row intervals of the mask's
    definition (document start up to the row itself), orders and running sums that fit together, and the
    text report names the shape and the counts."""
    docs = [700, 3, 1500, 64, 64, 9]
    c = _small(91, docs, 4, 2, 128)
    c.attn.plan()
    t = B.plan_tables(c.attn)
    cu = _cu(docs)
    pos = np.arange(sum(docs))
    start = cu[np.searchsorted(cu, pos, side="right") - 1]
    assert np.array_equal(t["row_lo"], start) and np.array_equal(t["row_hi"], pos + 1)
    lay = t["layout"]
    assert sorted(t["fwd_order"].tolist()) == list(range(lay.n_fwd_tiles))
    assert t["fwd_prefix"][0] == 0 and (np.diff(t["fwd_prefix"]) > 0).all()
    assert int(t["key_item_base"][-1]) == int((t["key_ways"] * 2).sum())
    text = B.plan_report(c.attn, "case")
    assert f"n_q {sum(docs)}" in text and f"{lay.n_fwd_tiles} query tiles" in text and "dK/dV items" in text


def test_gang_schedule_on_one_row():
    """Degenerate work lines: a single query row, and fewer units of work than gangs."""
    for docs in ([1], [5, 1, 2]):
        w, tens = wl.small_case(78, docs, 8, 1, 128)
        sh = osh.shard(docs, 1, 0, osh.PER_DOC_PADDED)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], 8, 1, 128, w.scale)
        c.flags = B.ATTN_SCHEDULE_GANGS
        c.check_fwd(f" docs {docs}")
        c.check_bwd(f" docs {docs}")


SHORT_CASES = [
    # docs, hq, hkv, d, cp: documents of a few dozen tokens, where whole query tiles take the short-hull path
    (list(range(1, 65)) * 2, 16, 2, 128, 1),       # every length 1..64 twice, 8 heads per KV head (two per wavefront)
    ([64] * 9 + [5], 4, 4, 128, 1),                # one head per KV head, last tile ragged
    ([33, 1, 64, 17, 2, 48, 9, 60, 31] * 5, 6, 2, 64, 1),   # three heads per KV head, head_dim 64
    ([40, 7, 64, 23, 12] * 9, 8, 1, 128, 2),       # sharded: pads, and key windows too wide for some tiles
    ([64, 64, 300, 20, 20, 20, 64, 1000, 8, 8], 2, 1, 128, 1),   # short and long tiles in one launch
]


@pytest.mark.parametrize("docs,hq,hkv,d,cp", SHORT_CASES)
def test_short_hull_path_matches_oracle(docs, hq, hkv, d, cp):
    """Tiles whose 32-row blocks each see at most 96 keys run as short-hull units inside the
    one-workgroup-per-item launches (forward, dQ with its own delta).  The schedule must mark them,
    the results must match the oracle, and switching the path off must change nothing beyond rounding."""
    import torch
    w, tens = wl.small_case(90, docs, hq, hkv, d)
    for r in sorted({0, cp - 1}):
        sh = osh.shard(docs, cp, r, osh.PER_DOC_PADDED)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)
        c.flags = B.ATTN_SCHEDULE_ITEMS
        c.check_fwd(f" short rank {r}")
        c.check_bwd(f" short rank {r}")
        lay = B.wlb_attn_plan_layout(c.attn.desc)
        ws = c.attn.workspace.cpu().numpy()
        hull = ws[lay.off_block_hull:lay.off_block_hull + 8 * lay.n_blocks32].view(np.int32).reshape(-1, 2)
        short = ws[lay.off_tile_short:lay.off_tile_short + 4 * lay.n_fwd_tiles].view(np.int32)
        lo, hi = (ws[o:o + 4 * len(c.q_idx)].view(np.int32) for o in (lay.off_row_lo, lay.off_row_hi))
        want_short = []
        for t in range(lay.n_fwd_tiles):
            ok = True
            for b in range(4 * t, min(4 * t + 4, lay.n_blocks32)):
                rows = slice(32 * b, min(32 * b + 32, len(c.q_idx)))
                real = hi[rows] > 0
                if real.any():
                    assert hull[b, 0] == lo[rows][real].min() and hull[b, 1] == hi[rows][real].max()
                    ok &= hull[b, 1] - (hull[b, 0] // 32) * 32 <= 96
                else:
                    assert hull[b, 1] <= hull[b, 0]
            want_short.append(int(ok))
        assert short.tolist() == want_short
        if cp == 1:
            assert sum(want_short) > 0, "this input is meant to exercise the short-hull path"
        o1, l1 = c.run_fwd()
        g1 = c.run_bwd()
        c.flags = B.ATTN_SCHEDULE_ITEMS | B.ATTN_NO_SHORT_PATH
        o2, l2 = c.run_fwd()
        g2 = c.run_bwd()
        real = c.q_idx >= 0
        check_close("O short vs general", o1, o2, rows=real)
        for name, a, b in zip(("dQ", "dK", "dV"), g1, g2):
            check_close(f"{name} short vs general", a, b)


@pytest.mark.parametrize("hq,hkv,d,cp", [(8, 1, 128, 1), (2, 2, 64, 1), (6, 2, 128, 2), (16, 2, 64, 4)])
def test_short_key_tiles_match_oracle(hq, hkv, d, cp):
    """Short documents beside longer ones: spans just below and above the limit of the dK/dV kernel of short key tiles (which
    then leaves them all to the general one), split tiles, pads whose Q and dO are garbage, keys that no row sees, and a
    ragged last tile."""
    docs = [1] * 40 + [128, 190, 256, 700] + [7, 64, 33, 2, 128, 90] * 6 + [5]
    w, tens = wl.small_case(79, docs, hq, hkv, d)
    for r in sorted({0, cp - 1}):
        sh = osh.shard(docs, cp, r, osh.PER_DOC_PADDED)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)
        c.flags = B.ATTN_SCHEDULE_ITEMS
        pads = c.torch.from_numpy(c.q_idx < 0).cuda()
        c.dev["q"][pads] = float("nan")
        c.dev["do"][pads] = float("nan")
        c.check_fwd(f" cp {cp} rank {r}")
        c.check_bwd(f" cp {cp} rank {r}")


def short_keys_estimate(t, hq, hkv, d):
    """Estimated times of dK/dV in the general kernel and in the kernel of short key tiles, in stages of the general one:
    from the schedule's tables, as the schedule's rule is stated."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    G, ways = hq // hkv, t["key_ways"]
    first, last = t["key_range"].T
    span = last - first
    top = span.argmax()
    general = 18 + max(span[top] * (G // ways[top]), 1.45 * span.sum() * hq / n_cu) + 2 * (ways[top] > 1)
    if span[top] > t["records"].short_span:
        return general, np.inf
    hull = t["block_hull"]
    seen = np.zeros((len(span), 4), dtype=np.int64)
    for kt in range(len(span)):
        h = hull[2 * first[kt]:2 * last[kt]]
        for w in range(4):
            seen[kt, w] = ((h[:, 1] > h[:, 0]) & (h[:, 0] < kt * 128 + w * 32 + 32) & (h[:, 1] > kt * 128 + w * 32)).sum()
    run = np.arange(len(span)) // -(-len(span) // 8)
    load = max(seen[run == x].sum() for x in range(8))
    return general, 7 + (1.0 if d == 64 else 1.3) * max(seen.max() * G, 0.25 * load * hq * 8 / n_cu) + 2


@pytest.mark.parametrize("tokens,long,hq,hkv,d,cp,takes", [
    (1024, 0, 4, 1, 64, 1, True),
    (1024, 0, 16, 1, 128, 1, False),       # 48 steps one after another, where the general kernel divides the heads
    (1024, 0, 32, 1, 128, 1, False),
    (4096, 700, 8, 1, 128, 1, False),      # the long document's tiles would need the general launch as well
    (4400, 0, 4, 2, 128, 1, True),         # the three-launch schedule
    (4400, 0, 32, 1, 64, 1, False),
    (9000, 700, 16, 2, 128, 1, False),
    (3000, 190, 6, 2, 128, 2, True),       # pads, whose Q and dO are garbage, and keys that no row sees
    (16800, 0, 4, 4, 64, 3, True),
])
def test_short_key_tiles_are_taken_where_that_is_shorter(tokens, long, hq, hkv, d, cp, takes):
    """dK/dV is left to the kernel of short key tiles only where no tile has a long span and the schedule's estimate of it is
    the shorter one; the results are the oracle's either way."""
    rng = np.random.default_rng(tokens + hq)
    docs = [long] if long else []
    while sum(docs) < tokens:
        docs.append(min(int(rng.integers(1, 65)), tokens - sum(docs)))
    docs = rng.permutation(docs).tolist()
    w, tens = wl.small_case(80, docs, hq, hkv, d)
    sh = osh.shard(docs, cp, 0, osh.PER_DOC_PADDED)
    c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], hq, hkv, d, w.scale)
    pads = c.torch.from_numpy(c.q_idx < 0).cuda()
    c.dev["q"][pads] = float("nan")
    c.dev["do"][pads] = float("nan")
    c.check_fwd()
    t = check_work_records(c.attn)
    assert t["records"].uses_short_keys
    general, short = short_keys_estimate(t, hq, hkv, d)
    assert (short <= general) == takes and abs(short - general) > 0.5       # far enough from the rounding of an estimate
    assert t["short_keys_on"] == takes
    c.check_bwd()


@pytest.mark.parametrize("d", [64, 128])
def test_short_key_tiles_repeat_bit_for_bit(d):
    """Thousands of short key tiles: repeated backward calls give the same bits, and what the general kernels give up to
    rounding (a store whose data registers were written again too early showed in a few rows per call, not in every one)."""
    import torch
    rng = np.random.default_rng(12)
    docs = rng.integers(1, 65, size=990)
    cu = np.concatenate([[0], np.cumsum(docs)]).astype(np.int32)
    t, hq, hkv = int(cu[-1]), 16, 2
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v, do = (torch.randn((t, h, d), device="cuda", generator=gen, dtype=torch.bfloat16) for h in (hq, hkv, hkv, hq))
    attn = B.Attention(np.arange(t, dtype=np.int32), cu, t, hq, hkv, d, d ** -0.5)
    o, lse = attn.forward(q, k, v)
    first = [x.clone() for x in attn.backward(q, k, v, o, lse, do)]
    general = attn.backward(q, k, v, o, lse, do, extra_flags=B.ATTN_NO_SHORT_PATH)
    for a, b in zip(first, general):
        # both round P and dS to bf16 (2^-9) and sum at most 64 of them per result in fp32
        assert (a.float() - b.float()).abs().max() <= 2e-2 * b.float().abs().max()
    for _ in range(6):
        assert all(torch.equal(a, b) for a, b in zip(first, attn.backward(q, k, v, o, lse, do)))


ROW_ITEM_OVERHEAD = 6     # units of fixed cost per query tile in the forward / dQ work line
DKV_SPLIT = 6             # a dK/dV item is at most 1/DKV_SPLIT of a compute unit's mean load
DKV_MIN_ITEM_STAGES = 32  # items this short are not split further


def test_schedule_tables():
    """The schedule in the workspace: row intervals equal the definition, group hulls cover
    their rows, fully visible ranges are visible to every real row, orders are permutations
    sorted heaviest first, and a key tile's group range covers every group that can see it."""
    import torch
    docs = [517, 3, 40, 1200, 64, 9]
    w, tens = wl.small_case(41, docs, 2, 1, 64)
    for cp, r in ((1, 0), (4, 1)):
        sh = osh.shard(docs, cp, r, osh.PER_DOC_PADDED)
        c = Case(tens, sh["q_idx"], sh["cu_seqlens_k"], 2, 1, 64, w.scale)
        c.attn.plan()
        torch.cuda.synchronize()
        lay = B.wlb_attn_plan_layout(c.attn.desc)
        ws = c.attn.workspace.cpu().numpy()

        def arr(off, n):
            return ws[off:off + 4 * n].view(np.int32)

        n_q = len(c.q_idx)
        lo, hi = arr(lay.off_row_lo, n_q), arr(lay.off_row_hi, n_q)
        cu = c.cu_k
        for i, g in enumerate(c.q_idx):
            if g < 0:
                assert lo[i] > hi[i]
            else:
                d = np.searchsorted(cu, g, side="right") - 1
                assert lo[i] == cu[d] and hi[i] == g + 1
        grp = arr(lay.off_group, 4 * lay.n_groups).reshape(-1, 4)
        for g in range(lay.n_groups):
            rows = slice(g * lay.group_rows, min((g + 1) * lay.group_rows, n_q))
            real = c.q_idx[rows] >= 0
            if not real.any():
                assert grp[g, 1] <= grp[g, 0]
                continue
            assert grp[g, 0] == lo[rows][real].min() and grp[g, 1] == hi[rows][real].max()
            assert grp[g, 2] == lo[rows][real].max() and grp[g, 3] == hi[rows][real].min()
        order = arr(lay.off_fwd_order, lay.n_fwd_tiles)
        cost = arr(lay.off_fwd_cost, lay.n_fwd_tiles)
        assert sorted(order.tolist()) == list(range(lay.n_fwd_tiles))
        assert (np.diff(cost[order]) <= 0).all()
        # forward / dQ work line: running sum, in order, of key tiles + the fixed per-tile cost
        prefix = ws[lay.off_fwd_prefix:lay.off_fwd_prefix + 8 * (lay.n_fwd_tiles + 1)].view(np.int64)
        assert prefix[0] == 0 and (np.diff(prefix) == cost[order] + ROW_ITEM_OVERHEAD).all()
        n_cu = torch.cuda.get_device_properties(0).multi_processor_count
        assert lay.row_gangs == 8 * max(1, (2 * n_cu // 8) // (c.hq // c.hkv))
        korder = arr(lay.off_key_order, lay.n_key_tiles)
        krange = arr(lay.off_key_range, 2 * lay.n_key_tiles).reshape(-1, 2)
        assert sorted(korder.tolist()) == list(range(lay.n_key_tiles))
        for kt in range(lay.n_key_tiles):
            k0, k1 = kt * lay.bwd_key_tile, min((kt + 1) * lay.bwd_key_tile, c.t_kv)
            sees = [g for g in range(lay.n_groups) if grp[g, 1] > grp[g, 0] and grp[g, 0] < k1 and grp[g, 1] > k0]
            if sees:
                assert krange[kt, 0] == sees[0] and krange[kt, 1] == sees[-1] + 1
            else:
                assert krange[kt, 0] == krange[kt, 1]
        # dK/dV items: a tile is cut by heads into a power-of-two number of items, tiles are ordered by
        # item cost (groups in range x heads per item), heaviest first, and the item / partial-slot
        # bases are the running sums in that order
        ways = arr(lay.off_key_ways, lay.n_key_tiles)
        item_base = arr(lay.off_key_item_base, lay.n_key_tiles + 1)
        slot_base = arr(lay.off_key_slot_base, lay.n_key_tiles + 1)
        g_heads = c.hq // c.hkv
        assert all(w in (1, 2, 4, 8) and g_heads % w == 0 for w in ways.tolist())
        span = krange[:, 1] - krange[:, 0]
        icost = span * (g_heads // ways)
        assert (np.diff(icost[korder]) <= 0).all()
        assert item_base[0] == 0 and slot_base[0] == 0
        assert (np.diff(item_base) == ways[korder] * c.hkv).all()
        assert (np.diff(slot_base) == np.where(ways[korder] > 1, ways[korder] * c.hkv, 0)).all()
        assert item_base[-1] <= lay.dkv_max_items and slot_base[-1] <= lay.dkv_max_partials
        # no item is heavier than the threshold unless it is already a single head
        total = int(span.sum()) * c.hq
        assert (icost[ways < g_heads] <= max(DKV_MIN_ITEM_STAGES, -(-total // (DKV_SPLIT * n_cu)))).all()
        check_work_records(c.attn)


@pytest.mark.parametrize("docs,hq,hkv", [
    ([1700, 2, 900, 64, 1600], 4, 2),                                                       # just above 4096 rows
    (np.random.default_rng(4).integers(1, 33, size=2500).tolist() + [700], 8, 1),           # more documents than LDS holds
    ([700] * 13 + [77], 36, 18),                                                            # records of a tile shared by a wavefront
])
@pytest.mark.parametrize("shuffled", [False, True])
def test_schedule_tables_of_larger_calls(docs, hq, hkv, shuffled):
    """The tables of the three-launch schedule against their definitions, with the document starts searched in LDS and
    in global memory, rows in order and shuffled with padding in between."""
    import torch
    cu = _cu(docs)
    t_kv = int(cu[-1])
    q_idx = np.arange(t_kv, dtype=np.int32)
    if shuffled:
        q_idx = np.random.default_rng(3).permutation(q_idx)
        q_idx[::11] = -1
    assert len(q_idx) > 4096
    attn = B.Attention(q_idx, cu, t_kv, hq, hkv, 64, 0.125)
    attn.plan()
    torch.cuda.synchronize()
    t = check_work_records(attn)
    lay = t["layout"]
    lo, hi = t["row_lo"], t["row_hi"]
    real = q_idx >= 0
    start = cu[np.searchsorted(cu, np.maximum(q_idx, 0), side="right") - 1]
    assert (lo[real] == start[real]).all() and (hi[real] == q_idx[real] + 1).all() and (lo[~real] > hi[~real]).all()

    def hulls(n, rows):
        pad = np.full(n * rows - len(q_idx), -1)
        q = np.concatenate([q_idx, pad]).reshape(n, rows)
        l = np.concatenate([start, pad]).reshape(n, rows)
        return [(l[i][q[i] >= 0], q[i][q[i] >= 0] + 1) for i in range(n)]

    for want, got in zip(hulls(lay.n_groups, lay.group_rows), t["group"]):
        if len(want[0]):
            assert got.tolist() == [want[0].min(), want[1].max(), want[0].max(), want[1].min()]
        else:
            assert got[1] <= got[0]
    fits = []
    for want, got in zip(hulls(lay.n_blocks32, 32), t["block_hull"]):
        if len(want[0]):
            assert got.tolist() == [want[0].min(), want[1].max()]
        else:
            assert got[1] <= got[0]
        fits.append(not len(want[0]) or want[1].max() - want[0].min() // 32 * 32 <= 96)
    fits = np.asarray(fits + [True] * (4 * lay.n_fwd_tiles - len(fits))).reshape(-1, 4).all(axis=1)
    assert (t["tile_short"] == fits).all()
    tile = hulls(lay.n_fwd_tiles, lay.fwd_tile_rows)
    cost = np.asarray([-(-h.max() // 64) - l.min() // 64 if len(l) else 0 for l, h in tile])
    assert (t["fwd_cost"] == cost).all()
    assert (t["fwd_order"] == np.lexsort((np.arange(len(cost)), -cost))).all()
    prefix = t["fwd_prefix"]
    assert prefix[0] == 0 and (np.diff(prefix) == cost[t["fwd_order"]] + ROW_ITEM_OVERHEAD).all()
    g = t["group"]
    for kt in range(lay.n_key_tiles):
        k0, k1 = kt * lay.bwd_key_tile, min((kt + 1) * lay.bwd_key_tile, t_kv)
        sees = np.nonzero((g[:, 1] > g[:, 0]) & (g[:, 0] < k1) & (g[:, 1] > k0))[0]
        first, last = t["key_range"][kt]
        assert (first, last) == (sees[0], sees[-1] + 1) if len(sees) else first == last
    G, ways = hq // hkv, t["key_ways"]
    span = t["key_range"][:, 1] - t["key_range"][:, 0]
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    limit = max(DKV_MIN_ITEM_STAGES, -(-int(span.sum()) * hq // (DKV_SPLIT * n_cu)))
    for kt in range(lay.n_key_tiles):
        w = 1
        while (G // w) % 2 == 0 and span[kt] * (G // w) > limit:
            w *= 2
        assert ways[kt] == w
    icost = span * (G // ways)
    assert (t["key_order"] == np.lexsort((np.arange(len(icost)), -icost))).all()
    in_order = ways[t["key_order"]]
    assert (np.diff(t["key_item_base"]) == in_order * hkv).all() and t["key_item_base"][0] == 0
    assert (np.diff(t["key_slot_base"]) == np.where(in_order > 1, in_order * hkv, 0)).all() and t["key_slot_base"][0] == 0
    assert t["key_item_base"][-1] <= lay.dkv_max_items and t["key_slot_base"][-1] <= lay.dkv_max_partials


def test_schedule_orders_with_thousands_of_tiles():
    """600K tokens: more tiles than one pass of the counting rank holds.  Both orders must be the
    stable sort by cost, heaviest first (ties by index), and the running sums must follow them."""
    import torch
    rng = np.random.default_rng(5)
    docs = [200000, 70001] + rng.integers(1, 3000, size=220).tolist()
    cu = np.concatenate([[0], np.cumsum(docs)]).astype(np.int32)
    t = int(cu[-1])
    attn = B.Attention(np.arange(t, dtype=np.int32), cu, t, 2, 1, 64, 0.125)
    attn.plan()
    torch.cuda.synchronize()
    lay = B.wlb_attn_plan_layout(attn.desc)
    assert lay.n_fwd_tiles > 4096 and lay.n_key_tiles > 4096
    ws = attn.workspace.cpu().numpy()
    arr = lambda off, n: ws[off:off + 4 * n].view(np.int32)
    cost = arr(lay.off_fwd_cost, lay.n_fwd_tiles)
    # a query tile's cost: 64-key tiles from its first row's document start to its last row
    tile_rows = t // lay.n_fwd_tiles + (t % lay.n_fwd_tiles > 0)
    assert tile_rows == 128
    first = np.arange(lay.n_fwd_tiles) * 128
    last = np.minimum(first + 128, t) - 1
    lo = cu[np.searchsorted(cu, first, side="right") - 1]
    assert (cost == (last + 1 + 63) // 64 - lo // 64).all()
    order = arr(lay.off_fwd_order, lay.n_fwd_tiles)
    assert (order == np.lexsort((np.arange(lay.n_fwd_tiles), -cost))).all()
    prefix = ws[lay.off_fwd_prefix:lay.off_fwd_prefix + 8 * (lay.n_fwd_tiles + 1)].view(np.int64)
    assert prefix[0] == 0 and (np.diff(prefix) == cost[order].astype(np.int64) + ROW_ITEM_OVERHEAD).all()
    krange = arr(lay.off_key_range, 2 * lay.n_key_tiles).reshape(-1, 2)
    ways = arr(lay.off_key_ways, lay.n_key_tiles)
    icost = (krange[:, 1] - krange[:, 0]) * (2 // ways)
    korder = arr(lay.off_key_order, lay.n_key_tiles)
    assert (korder == np.lexsort((np.arange(lay.n_key_tiles), -icost))).all()
    item_base = arr(lay.off_key_item_base, lay.n_key_tiles + 1)
    assert item_base[0] == 0 and (np.diff(item_base) == ways[korder]).all()


BWD_CASES = [
    ([300, 45, 1, 700, 130], 4, 2, 128, 1),
    ([64, 64, 128], 2, 2, 64, 1),
    ([1] * 70, 2, 1, 128, 1),
    ([1000], 8, 1, 128, 1),
    ([3], 1, 1, 64, 1),
    ([5, 900, 2, 3, 333, 64, 1, 77], 4, 4, 64, 2),
    ([517, 3, 40, 1200], 8, 2, 128, 4),
]


@pytest.mark.parametrize("docs,rows,hq,hkv,coarse", [
    ([1024] * 16, range(16384), 32, 8, True),                          # documents of one length, three launches
    ([18432], range(10240, 18432), 8, 2, False),                       # too many long items
    ([16384], range(8192, 16384), 10, 5, True),
    ([18432], range(14336, 18432), 8, 2, True),                        # the single launch
    ([900, 3000, 77] * 4 + [384], range(1, 16276, 4), 16, 4, True),
    ([16384], range(12288, 16384), 16, 2, False),                      # too many long items
    ([1024] * 15 + [1000], range(0, 16360, 3), 6, 1, False),           # fewer key tiles and KV heads than compute units
    ([1024] * 16, range(16384), 6, 2, False),                          # three heads are never split
])
def test_dkv_items_are_coarse_where_they_balance(docs, rows, hq, hkv, coarse):
    """The limit of a dK/dV item in both schedules against its rule."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    cu = _cu(docs)
    attn = B.Attention(np.asarray(rows, dtype=np.int32), cu, int(cu[-1]), hq, hkv, 64, 0.125)
    attn.plan()
    torch.cuda.synchronize()
    t = check_work_records(attn)
    G, span = hq // hkv, t["key_range"][:, 1] - t["key_range"][:, 0]
    total = int(span.sum()) * hq

    def ways_of(limit):
        ways = np.ones(len(span), dtype=np.int64)
        while (more := ((G // ways) % 2 == 0) & (span * (G // ways) > limit)).any():
            ways[more] *= 2
        return ways

    want = ways_of(max(64, -(-total // (2 * n_cu))))
    even = all((want * hkv)[span * (G // want) * 16 * q * n_cu > 17 * total + 256 * n_cu].sum() <= (q - 1) * n_cu for q in range(1, 9))
    takes = G % 2 == 0 and len(span) * hkv >= n_cu and even
    assert takes == coarse or n_cu != 256
    if not takes:
        want = ways_of(max(DKV_MIN_ITEM_STAGES, -(-total // (DKV_SPLIT * n_cu))))
    assert (t["key_ways"] == want).all()
    assert t["key_slot_base"][-1] <= t["layout"].dkv_max_partials


@pytest.mark.parametrize("docs,hq,hkv,d,cp", BWD_CASES)
def test_backward_matches_oracle(docs, hq, hkv, d, cp):
    for r in range(cp):
        c = _small(50 + r, docs, hq, hkv, d, cp, r, osh.PER_DOC_PADDED)
        c.check_fwd(f" rank {r}")
        c.check_bwd(f" rank {r}")


def test_backward_per_sequence_sharding_and_rank_sum():
    """Per-rank dK/dV partials add up to the unsharded gradient (what the reduce-scatter of
    all-gather context parallelism would deliver)."""
    docs = [700, 41, 3, 1000, 304]
    cp = 4
    full = _small(60, docs, 4, 1, 128)
    full.run_fwd()
    _, rdk, rdv = full.oracle_bwd()
    dk_sum, dv_sum = np.zeros_like(rdk), np.zeros_like(rdv)
    for r in range(cp):
        c = _small(60, docs, 4, 1, 128, cp, r, osh.PER_SEQ)
        c.check_fwd(f" rank {r}")
        c.check_bwd(f" rank {r}")
        _, dk, dv = c.run_bwd()
        dk_sum += dk
        dv_sum += dv
    check_close("sum of dK partials", dk_sum, rdk)
    check_close("sum of dV partials", dv_sum, rdv)


def test_backward_rows_in_arbitrary_order_with_garbage_in_padding():
    docs = [200, 333, 90]
    w, tens = wl.small_case(61, docs, 4, 2, 128)
    rng = np.random.default_rng(1)
    q_idx = rng.permutation(sum(docs)).astype(np.int32)[:400]
    q_idx[::13] = -1
    c = Case(tens, q_idx, _cu(docs), 4, 2, 128, w.scale)
    # padding rows may hold anything, including NaN and Inf bit patterns
    pad = np.nonzero(q_idx < 0)[0]
    for name in ("q", "do"):
        t = c.dev[name].view(dtype=__import__("torch").int16)
        t[pad[0::2]] = 0x7FC0          # NaN
        t[pad[1::2]] = 0x7F80          # +Inf
    c.check_fwd()
    c.check_bwd()


@pytest.mark.parametrize("hq,hkv,d", [(1, 1, 128), (3, 1, 128), (4, 4, 64), (8, 1, 64), (8, 2, 128)])
@pytest.mark.parametrize("docs", [[1], [33], [64, 64], [63, 1, 65, 127], [129, 31, 96, 700], [300, 5, 2100]], ids=str)
def test_general_key_tiles_at_their_edges(docs, hq, hkv, d):
    """The general dK/dV kernel where documents begin and end at, before and after a wavefront's 64 keys and 32 rows: a last tile
    that ends in either half of its keys, items of one stage to dozens, stages that only some of the wavefronts see (between
    stages that they do), a wavefront without a visible pair, and padding rows that hold NaN and Inf among them."""
    import torch
    w, tens = wl.small_case(63, docs, hq, hkv, d)
    q_idx = np.arange(sum(docs), dtype=np.int32)
    q_idx = np.insert(q_idx, np.arange(0, len(q_idx), 37), -1)
    if len(docs) == 3:
        q_idx = np.concatenate([q_idx[1000:], np.full(70, -1, dtype=np.int32), q_idx[:700]])      # late rows first, a group of padding
    c = Case(tens, q_idx, _cu(docs), hq, hkv, d, w.scale)
    c.flags = B.ATTN_NO_SHORT_PATH
    pad = np.nonzero(q_idx < 0)[0]
    for name in ("q", "do"):
        t = c.dev[name].view(dtype=torch.int16)
        t[pad[0::2]] = 0x7FC0          # NaN
        t[pad[1::2]] = 0x7F80          # +Inf
    c.check_fwd()
    c.check_bwd()


@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 128), (4, 4, 64), (8, 2, 128)])
@pytest.mark.parametrize("docs,bad,cp", [([32, 300], 100, 1), ([64, 300], 200, 1), ([96, 40, 300], 250, 1), ([200, 300, 64], 400, 1),
                                         ([16, 700, 33], 300, 1), ([32, 600, 40, 90], 200, 2)], ids=str)
@pytest.mark.parametrize("where", ["q", "do", "lse"])
def test_non_finite_rows_stay_with_the_keys_that_see_them(docs, bad, cp, where, hq, hkv, d):
    """Inf or NaN in a row of Q or dO: dK and dV of other documents stay as they are, at least in the aligned blocks of 32 keys that none
    of the same 64 rows sees (0 x Inf inside such a block is NaN).  In a row's LSE: those of every key that the row does not see."""
    import torch
    w, tens = wl.small_case(64, docs, hq, hkv, d)
    cu = _cu(docs)
    q_idx = np.arange(int(cu[-1]), dtype=np.int32) if cp == 1 else B.wlb_shard(docs, cp, 1, B.SHARD_PER_DOC_NOPAD)["q_idx"]
    c = Case(tens, q_idx, cu, hq, hkv, d, w.scale)
    c.flags = B.ATTN_NO_SHORT_PATH
    c.run_fwd()
    _, dk0, dv0 = c.run_bwd()

    doc_of = np.searchsorted(cu, q_idx, side="right") - 1
    seen = np.arange(int(cu[doc_of[bad]]), int(q_idx[bad]) + 1)
    apart = np.ones(len(dk0), dtype=bool)
    if where == "lse":
        apart[seen] = False
        c.lse[0::2, bad] = float("nan")
        c.lse[1::2, bad] = float("-inf")
    else:
        t = c.dev[where].view(dtype=torch.int16)
        t[bad, :, 3] = 0x7F80              # +Inf
        t[bad, :, d - 1] = 0x7FC0          # NaN
        c.run_fwd()
        group = np.arange(bad // 64 * 64, min(bad // 64 * 64 + 64, len(q_idx)))
        lo, hi = int(cu[doc_of[group]].min()), int(q_idx[group].max()) + 1
        apart[lo // 32 * 32:-(-hi // 32) * 32] = False
    assert apart.any()
    _, dk1, dv1 = c.run_bwd()
    for name, was, now, keys in [("dK", dk0, dk1, apart), ("dV", dv0, dv1, apart)]:
        assert np.isfinite(now[keys]).all(), f"{name}: {np.nonzero(~np.isfinite(now).all(axis=(1, 2)) & keys)[0]}"
        assert (np.abs(now[keys] - was[keys]) <= 2e-2 * np.abs(was).max()).all(), name
    if where == "do":
        assert not np.isfinite(dv1[seen][:, :, [3, d - 1]]).any()
    if where == "q":
        assert not np.isfinite(dk1[seen][:, :, [3, d - 1]]).any()
    if where == "lse":
        assert not np.isfinite(dv1[seen]).any()


def test_backward_is_deterministic():
    c = _small(62, [900, 50, 400], 4, 2, 128)
    c.run_fwd()
    a = c.run_bwd()
    b = c.run_bwd()
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_padding_free_sharding_forward_backward():
    """Padding-free per-document maps go through the same kernels: the mask is per row."""
    docs = [517, 3, 41, 1203, 66, 9, 217]          # T = 2056 = 8 * 257: every rank gets 514 slots, none padding
    cp = 4
    sizes = set()
    for r in range(cp):
        c = _small(70, docs, 8, 2, 128, cp, r, osh.PER_DOC_NOPAD)
        assert (c.q_idx >= 0).all()
        sizes.add(len(c.q_idx))
        c.check_fwd(f" rank {r}")
        c.check_bwd(f" rank {r}")
    assert sizes == {sum(docs) // cp}


@pytest.mark.parametrize("flag", [0, B.ATTN_SCHEDULE_GANGS])
def test_graph_replay_matches_eager_calls(flag):
    """The library only launches kernels on the caller's stream, so schedule + forward + backward
    can be captured into a HIP graph.  Every replay must reproduce the eager results bit for bit,
    with eager calls and other inputs in between (the workspace is shared and rewritten)."""
    import torch
    c = _small(81, [700, 3, 260, 1, 90], 4, 2, 128)
    other = _small(82, [700, 3, 260, 1, 90], 4, 2, 128)
    a = c.attn
    n_q = len(c.q_idx)
    q, k, v, do = (c.dev[n].clone() for n in ("q", "k", "v", "do"))
    o = torch.empty_like(q)
    lse = torch.empty((c.hq, n_q), dtype=torch.float32, device=q.device)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)

    def step():
        a.plan()
        a.forward(q, k, v, o, lse, extra_flags=flag)
        a.backward(q, k, v, o, lse, do, dq, dk, dv, extra_flags=flag)

    def results():
        torch.cuda.synchronize()
        return [t.clone() for t in (o, lse, dq, dk, dv)]

    step()
    eager = results()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for replay in range(4):
        for t in (o, lse, dq, dk, dv):
            t.fill_(float("nan"))
        if replay == 2:
            # other inputs through the same graph, then back
            for dst, name in ((q, "q"), (k, "k"), (v, "v"), (do, "do")):
                dst.copy_(other.dev[name])
            graph.replay()
            step()
            for dst, name in ((q, "q"), (k, "k"), (v, "v"), (do, "do")):
                dst.copy_(c.dev[name])
        graph.replay()
        got = results()
        for name, x, y in zip(("O", "LSE", "dQ", "dK", "dV"), got, eager):
            assert torch.equal(x, y), f"{name} differs on replay {replay}"
        step()                                        # eager work between the replays
        for name, x, y in zip(("O", "LSE", "dQ", "dK", "dV"), results(), eager):
            assert torch.equal(x, y), f"{name} differs in the eager call after replay {replay}"


@pytest.mark.parametrize("hq,hkv,d,cp,mode,docs,pairs", [
    # units of short documents on a rank, a padding row in most blocks of 32 rows
    (8, 1, 128, 4, osh.PER_DOC_PADDED, [61, 33, 7, 48, 21] * 9, 50),
    (8, 2, 64, 4, osh.PER_DOC_PADDED, [61, 133, 7, 48, 21] * 9, 50),
    # short-hull units
    (8, 1, 128, 1, osh.PER_DOC_PADDED, [61, 33, 7, 48, 21] * 4, 0),
    (3, 1, 64, 1, osh.PER_DOC_PADDED, [61, 33, 7, 48, 21] * 4, 0),
])
def test_padding_rows_are_zero_whatever_lies_beside_them(hq, hkv, d, cp, mode, docs, pairs):
    """Padding rows that hold NaN and Inf in Q and dO leave everything else as it is; beside keys and values that are not finite, O and dQ of
    padding are 0 and LSE -inf all the same."""
    import torch
    w, tens = wl.small_case(65, docs, hq, hkv, d)
    sh = osh.shard(docs, cp, 0, mode)
    q_idx = sh["q_idx"] if cp > 1 else np.insert(sh["q_idx"], np.arange(0, sum(docs), 11), -1)
    pad = np.nonzero(q_idx < 0)[0]
    assert len(pad)
    c = Case(tens, q_idx, sh["cu_seqlens_k"], hq, hkv, d, w.scale, visible_pairs=pairs * len(q_idx))
    assert B.wlb_attn_plan_layout(c.attn.desc).row_kernels == (B.ROW_SPAN if pairs else 0)
    for name in ("q", "do"):
        t = c.dev[name].view(dtype=torch.int16)
        t[pad[0::2]] = 0x7FC0          # NaN
        t[pad[1::2]] = 0x7F80          # +Inf
    c.check_fwd()
    c.check_bwd()
    for name in ("k", "v"):
        t = c.dev[name].view(dtype=torch.int16)
        t[0::7, :, 3] = 0x7F80
        t[2::7, :, d - 1] = 0x7FC0
    o, lse = c.run_fwd()
    dq, _, _ = c.run_bwd()
    assert (o[pad] == 0).all() and np.isneginf(lse[:, pad]).all()
    assert (dq[pad] == 0).all()
