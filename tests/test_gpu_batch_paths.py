"""The coalesce's paths by batch size, at the edges of their tiles, against the oracle: every kernel
variant of the small batches (512, 1024 and 2048 tokens) with whole, partial and looped column
slices, vector and scalar rows, and both gradient types; the bucket sort's bucket and tile sizes; the
radix sort's digit widths and pass counts; the lookup requests, the split and device-side token counts
over the same paths; and the other calls at the edges of their rules on sizes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2110_09132_amd as emb
import tolerance
from gpu_helpers import check_coalesce, host, to_dev
from test_gpu_by_owner import check_by_owner, check_split, grads_for, ids_for, owners
from test_gpu_lookup_request import check_request

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 511, 512, 513, 1024, 1025, 2047, 2048])
@pytest.mark.parametrize("D,bf16", [(4, False), (36, False), (33, False), (260, True), (31, True)])
def test_small_batches(T, D, bf16):
    V, P = 700, 3
    ids = ids_for("zipf", T + D, T, V)
    ids[T // 2::97] = V + 1  # some tokens take no part
    check_by_owner(ids, grads_for(T * D, T, D, 0.01, bf16=bf16), V, owners("mod", V, P), P, bf16=bf16)


@pytest.mark.parametrize("T,D", [(2048, 4100), (1024, 2053), (300, 8196)])
def test_small_batches_of_wide_rows(T, D):
    # more column slices than one per XCD; a last slice that is not whole; a hot row
    V, P = 5000, 8
    ids = ids_for("zipf", T + D, T, V, 1.3)
    check_by_owner(ids, grads_for(T + D, T, D, 0.01), V, owners("range", V, P), P)


@pytest.mark.parametrize("T,D", [(512, 1), (511, 3), (300, 15), (512, 17), (512, 16), (512, 20), (1024, 1), (1023, 7),
                                 (1024, 9), (1024, 8), (1024, 12), (2048, 1), (2047, 3), (2048, 5), (2048, 4), (1100, 8)])
@pytest.mark.parametrize("bf16", [False, True])
def test_small_batches_of_narrow_rows(T, D, bf16):
    # both sides of half a slice's vectors, for each kernel's slice; ids of 1 to 18 tokens, so that every
    # remainder of the sums' blocks of eight occurs, and ids of one token
    V, P = 3000, 2
    rng = np.random.default_rng(T + D)
    ids = np.repeat(np.arange(T, dtype=np.int32), np.resize(np.r_[np.arange(1, 19), 1, 1, 1], T))[:T]
    ids = rng.permutation(V)[:T][ids % V].astype(np.int32) if T < V else ids
    rng.shuffle(ids)
    check_by_owner(ids, grads_for(T * D, T, D, 0.01, bf16=bf16), V, owners("mod", V, P), P, bf16=bf16)


# ------------------------------------------------------------------ bucket sort
def sample_tokens(n, T):
    """The tokens the bucket sort samples (sample_token in bucket_sort.hip)."""
    i = np.arange(n, dtype=np.uint64)
    lo, hi = (i * np.uint64(T)) // np.uint64(n), ((i + np.uint64(1)) * np.uint64(T)) // np.uint64(n)
    m = np.uint64(0xFFFFFFFF)
    h = (i * np.uint64(0x9E3779B1) + np.uint64(0x7F4A7C15)) & m
    h ^= h >> np.uint64(15)
    h = (h * np.uint64(0x85EBCA77)) & m
    h ^= h >> np.uint64(13)
    return (lo + ((h * np.maximum(hi - lo, np.uint64(1))) >> np.uint64(32))).astype(np.int64)


# distinct ids of the tokens outside the one-key bucket: spread evenly, bunched at the low end (more
# than 64 in an interval: radix passes), a handful (one radix pass), and over the whole 32-bit key
LAWS = {"even": (1 << 20, 1 << 20), "bunched": (1 << 20, 300), "few": (1 << 20, 9), "wide": ((1 << 31) - 1, 1 << 31)}


@pytest.mark.parametrize("law", sorted(LAWS))
@pytest.mark.parametrize("T,n,m", [(30000, 512, m) for m in (1, 511, 513, 1025, 2049, 4096, 4097, 20000)] +
                         [(T, n, m) for T, n in ((140000, 1024), (262144, 1024), (655360, 2048))
                          for m in (600, 4096, 4097, 20000)])
def test_bucket_of_any_size(T, n, m, law):
    # every sampled token (n of the batch) holds id 5, so the ids above it fall into one bucket of m
    # tokens: each variant of the bucket's sort, and the one for buckets that do not fit in LDS, in each
    # of the sort's three configurations
    V, top = LAWS[law]
    D = 4 if T < 100000 else 1
    rng = np.random.default_rng(m)
    ids = np.full(T, 5, np.int32)
    free = np.setdiff1d(np.arange(T), sample_tokens(n, T))
    at = rng.choice(free, m, replace=False)
    ids[at] = rng.integers(6, min(top, V), m)
    if law == "bunched":
        ids[at[0]] = V - 1  # the range is wide all the same
    G = grads_for(m, T, D, 0.01)
    if law == "wide":
        check_coalesce(ids, G, V)
    else:
        check_by_owner(ids, G, V, owners("range", V, 4), 4)


@pytest.mark.parametrize("T", [2049, 3071, 3073, 131072, 131073, 133121, 262144, 262145, 266241, 655360, 655361])
@pytest.mark.parametrize("s", [0.0, 1.0, 1.5])
def test_batch_sizes(T, s):
    # edges of the sort's tiles and of the three bucket counts, the largest bucket-sorted batch and
    # the smallest radix-sorted one; even ids, and hot ids with buckets of their own
    V, P, D = 1 << 18, 5, 4
    ids = ids_for("uniform" if s == 0.0 else "zipf", T, T, V, s)
    ids[3::1001] = -1
    own = owners("mod", V, P)
    own[7::500] = P  # not an owner
    check_by_owner(ids, grads_for(T, T, D, 0.01), V, own, P)


# ------------------------------------------------------------------- radix sort
# Keys of at most nine bits above 131072 tokens, and every batch above 655360.  (V, P): the key bits
# are those of V alone (P = 0: the plain call) or of V and P; the passes in comments.
RADIX = [(1, 0), (256, 0), (128, 2),                                     # one pass of 8-bit digits
         (512, 0), (300, 0), (128, 3),                                   # one of 9-bit digits
         (1024, 0), (65536, 0), (1 << 12, 16),                           # two of 8-bit digits
         (65537, 0), (1 << 18, 0), (1 << 14, 9),                         # two of 9-bit digits
         (1 << 24, 0), (1 << 19, 1), (1 << 20, 16),                      # three of 8-bit digits
         (1 << 25, 0), (1 << 27, 0), (1 << 20, 33),                      # three of 9-bit digits
         ((1 << 28) - 3, 0), ((1 << 31) - 1, 0), ((1 << 22) - 1, 1024)]  # four of 8-bit digits


@pytest.mark.parametrize("V,P", RADIX)
@pytest.mark.parametrize("T", [655361, 700000])
def test_radix_passes(V, P, T):
    law = "zipf" if V < 1 << 22 and T % 2 else "uniform"
    ids = ids_for(law, V + T, T, V)
    ids[5::1003] = -1
    G = grads_for(T, T, 2, 0.01)
    if P == 0:
        check_coalesce(ids, G, V)
    else:
        check_by_owner(ids, G, V, owners("mod", V, P), P)


@pytest.mark.parametrize("V", [1, 256, 512, 513])
@pytest.mark.parametrize("T", [131072, 131073, 200000, 442368, 442369])
def test_one_pass_keys(V, T):
    # the edges of the range in which keys of one pass take the radix sort
    ids = ids_for("uniform", V + T, T, V)
    check_coalesce(ids, grads_for(T, T, 2, 0.01), V)


@pytest.mark.parametrize("V,P", [(100, 2), (1 << 14, 4), (1 << 20, 7), (1 << 23, 16), ((1 << 22) - 1, 1024)])
@pytest.mark.parametrize("T", [150000, 655361])
def test_lookup_request_radix(V, P, T):
    # requests of radix-sorted tokens (above 131072 those of one pass): offsets first, counts from them
    ids = ids_for("zipf" if P == 7 else "uniform", V + T, T, V)
    ids[[0, T // 2, T - 1]] = [-3, V, V + 77]
    own = owners("rand", V, P, seed=T)
    own[::13] = P
    check_request(ids, V, own, P)


def test_lookup_request_radix_without_tokens():
    V, P, T = 1000, 5, 655361
    check_request(np.full(T, V, np.int32), V, owners("mod", V, P), P)


@pytest.mark.parametrize("V,P,T_next", [(60, 2, 700), (50000, 3, 20000), (1 << 20, 16, 700000), ((1 << 24) + 9, 8, 5000),
                                        ((1 << 21) - 1, 1024, 1)])
@pytest.mark.parametrize("T", [140000, 655361])
def test_split_radix(V, P, T, T_next):
    ids, nxt = ids_for("uniform", V + T, T, V), ids_for("uniform", V + T + 1, T_next, V)
    nxt[3::11] = -1
    check_split(ids, nxt, grads_for(T, T, 2, 0.01), V, owners("mod", V, P), P)


@pytest.mark.parametrize("T", [1, 63, 700, 1025, 140000, 270000])
def test_lookup_request_sizes(T):
    V, P = 40000, 7
    ids = ids_for("zipf", T, T, V)
    own = owners("range", V, P)
    check_request(ids, V, own, P)


@pytest.mark.parametrize("used", [[0], [1023], [511], [0, 1023], [1, 2, 700], [5, 1022]])
@pytest.mark.parametrize("T", [1, 3, 200, 70000])
def test_lookup_request_owners_without_requests(used, T):
    # runs of owners that nothing is asked of, at either end and between: only a run's ends change the
    # counts
    V, P = 1 << 14, 1024
    rng = np.random.default_rng(T)
    ids = (rng.choice(used, T) + P * rng.integers(0, V // P, T)).astype(np.int32)
    check_request(ids, V, owners("mod", V, P), P)


@pytest.mark.parametrize("T,V,P,count", [(140000, 5000, 3, c) for c in (0, 1, 3000, 139999)] +
                         # the radix sort: one pass of 9-bit digits, two of 8, four of 8
                         [(140000, 100, 3, 77777), (655361, 5000, 3, 0), (655361, 5000, 3, 400000),
                          (655361, (1 << 22) - 1, 1024, 655360)])
def test_device_count(T, V, P, count):
    # a device-side token count: the samples of the bucket sort come from the tokens that exist
    D = 4
    ids = ids_for("zipf", 3, T, V)
    G = grads_for(3, T, D, 0.01)
    own = owners("mod", V, P)
    out = emb.receive_merge(to_dev(ids), to_dev(G), to_dev(np.array([count], np.int32)), V, to_dev(own), P)
    torch.cuda.synchronize()
    merged_ids, seg, rows, counts, offs, nu = (host(x) for x in out)
    U = int(nu[0])
    orc = oracle.coalesce(ids[:count], G[:count], V)
    pk = oracle.pack_by_owner(orc["uniq_ids"], orc["uniq_grad"], own, P)
    assert U == orc["U"] and np.array_equal(merged_ids[:U], pk["send_ids"])
    assert np.array_equal(counts, pk["send_counts"]) and np.array_equal(offs, pk["send_offsets"])
    idx = np.searchsorted(orc["uniq_ids"], merged_ids[:U])
    tolerance.assert_grad_close(rows[:U], orc["sum_f64"][idx], orc["absum"][idx])


# ------------------------------------------------------------------------- pack
@pytest.mark.parametrize("T,D,P", [(700, 3, 2), (1024, 4, 1), (1025, 2052, 7), (3000, 260, 3), (5000, 9000, 2),
                                   (4096, 16, 1024), (9000, 8, 256), (9000, 8, 257), (40000, 12, 203), (40000, 12, 204)])
def test_pack_places(T, D, P):
    # rows per workgroup from one to all of its threads, both sides of the histogram limit, more
    # vectors than one round of loads, rows without an owner
    V = 60000
    ids = ids_for("uniform", T + P, T, V)
    own = owners("rand", V, P, seed=T)
    own[::11] = -1
    out = emb.grad_coalesce(to_dev(ids), to_dev(grads_for(T, T, D, 0.01)), V)
    torch.cuda.synchronize()
    U = int(out[3].item())
    uid, ug = host(out[0][:U]), host(out[2][:U])
    want = oracle.pack_by_owner(uid, ug, own, P)
    st = emb.new_status()
    send_ids, rows, counts, offs = emb.pack_by_owner(out[0], out[2], out[3], to_dev(own), P, dev_status=st)
    torch.cuda.synchronize()
    n = int(want["send_offsets"][P])
    assert np.array_equal(host(counts), want["send_counts"]) and np.array_equal(host(offs), want["send_offsets"])
    assert np.array_equal(host(send_ids[:n]), want["send_ids"])
    assert np.array_equal(host(rows[:n]).view(np.uint32), want["send_rows"].view(np.uint32))
    assert int(st.item()) == emb.EMB_DEV_OWNER_OUT_OF_RANGE


# ------------------------------------------------------------------------ split
@pytest.mark.parametrize("T,T_next,V", [
    (300, 1, 1000), (1000, 2048, 900000), (2048, 2048, 1 << 25), (2000, 2049, 5000), (1500, 3000, (1 << 24) + 5),  # small batches
    (2049, 1, 1 << 18), (5000, 8192, 1 << 18), (5000, 8193, 1 << 18), (5000, 700, (1 << 18) + 1), (3000, 8191, 33),
    (131072, 9000, 40000), (131073, 9000, 40000)])
@pytest.mark.parametrize("law", ["zipf", "uniform"])
def test_split_next_sets(T, T_next, V, law):
    # the next batch's ids as a set in LDS (a hash set for small batches, a bit per row for the bucket
    # sort) and past its limits in memory; some next ids are not rows
    ids, nxt = ids_for(law, T, T, V), ids_for(law, T_next + 1, T_next, V)
    nxt[5::17] = -1
    nxt[6::17] = V
    check_split(ids, nxt, grads_for(T, T, 4, 0.01), V, owners("mod", V, 3), 3)


# --------------------------------------------------------------- column packs
@pytest.mark.parametrize("cap,R,D,P", [(5, 0, 64, 4), (5, 5, 64, 4), (9, 8, 2048, 8), (700, 641, 16, 1), (33, 31, 300, 7),
                                       (3, 2, 12000, 3),
                                       # both sides of the rule on the tile's size: owners, units, row width
                                       (700, 699, 96, 12), (700, 699, 104, 13), (4096, 4095, 512, 16),
                                       (4097, 4096, 512, 16), (30721, 30720, 512, 16), (30000, 29999, 512, 16),
                                       (2048, 2047, 512, 32), (2049, 2048, 512, 32), (50, 49, 528, 33),
                                       (37, 36, 1024, 8), (37, 36, 1028, 1), (37, 36, 1532, 1), (37, 36, 1536, 8),
                                       (37, 36, 1540, 1), (37, 36, 1600, 8)])
def test_column_pack_counts_and_tiles(cap, R, D, P):
    # the counts come with the pack; whole and partial tiles, rows wider than a tile, no rows at all
    rows = grads_for(cap + D, cap, D)
    blocks, counts = emb.pack_by_column(to_dev(rows), P, num_rows=to_dev(np.array([R], np.int32)),
                                        out=(torch.zeros(cap * D, device="cuda"),
                                             torch.full((P,), -7, dtype=torch.int32, device="cuda")))
    torch.cuda.synchronize()
    assert host(counts).tolist() == [R] * P
    off = emb.column_offsets(D, P)
    for p in range(P):
        got = host(emb.column_block(blocks, cap, D, P, p))
        assert np.array_equal(got[:R], rows[:R, off[p]:off[p + 1]]) and not got[R:].any()


# -------------------------------------------------------------------- reduction
@pytest.mark.parametrize("T,D", [(2100, 4), (2100, 6), (2100, 130), (2500, 516), (9000, 258), (9601, 128), (19100, 64),
                                 (19300, 64), (40000, 62), (40000, 64), (40000, 66)])
@pytest.mark.parametrize("bf16", [False, True])
def test_reduction_vector_widths(T, D, bf16):
    # one, two and four floats per lane (few workgroups take narrower vectors), rows that only two
    # floats divide, ids crossing chunks and workgroups, column blocks with idle lanes
    V, P = 900, 4
    ids = ids_for("zipf", T + D, T, V, 1.2)
    check_by_owner(ids, grads_for(T + D, T, D, 0.01, bf16=bf16), V, owners("mod", V, P), P, bf16=bf16)


# ----------------------------------------------------------------------- lookup
@pytest.mark.parametrize("T,D", [(1, 300), (8, 1024), (9, 259), (63, 2052), (1000, 516), (2047, 260), (8184, 257),
                                 (8192, 257), (8193, 257), (32768, 4), (500, 12),
                                 # rows of whole lines and others, narrow and wide, about half the limit's waves
                                 (700, 32), (700, 33), (4096, 288), (4097, 288), (4096, 260), (4097, 260),
                                 (4097, 65), (8184, 64), (8193, 64)])
def test_lookup_spread(T, D):
    # few waves: one per workgroup, the column steps of wide rows over several; both sides of the limits
    V = 700
    W = grads_for(D, V, D)
    ids = ids_for("uniform", T, T, V)
    ids[T // 2] = V
    st = emb.new_status()
    out = emb.gather(to_dev(W), to_dev(ids), out=torch.full((T, D), 7.0, device="cuda"), dev_status=st)
    torch.cuda.synchronize()
    want = np.where((ids < V)[:, None], W[np.minimum(ids, V - 1)], np.float32(0))
    assert np.array_equal(host(out).view(np.uint32), want.view(np.uint32)) and int(st.item()) == emb.EMB_DEV_ID_OUT_OF_RANGE


# --------------------------------------------------------------------- exchange
@pytest.mark.parametrize("P,cap,D", [(P, cap, D) for P in (1, 3, 31, 32, 33, 64)
                                     for cap, D in ((1, 4), (40, 0), (333, 5), (500, 132))] +
                         # workgroups without rows leave early from 8192 workgroups on; the most block
                         # sizes that the workgroups read themselves, and one workgroup per sender more
                         [(8, 32736, 33), (8, 32737, 33), (32, 8192, 33), (32, 8193, 33)])
def test_exchange_destinations(P, cap, D):
    # destinations worked out by every workgroup (up to 32 workers) or by a launch of their own; empty
    # blocks, senders with nothing to send, ids alone
    rng = np.random.default_rng(P * 1000 + cap)
    offs = np.zeros((P, P + 1), np.int32)
    for w in range(P):
        n = 0 if w % 5 == 3 else int(rng.integers(0, cap + 1))
        offs[w, 1:] = np.sort(np.r_[rng.integers(0, n + 1, P - 1), n])
    ids = rng.integers(0, 1 << 30, (P, cap)).astype(np.int32)
    rows = rng.standard_normal((P, cap, max(D, 1))).astype(np.float32)
    r_ids, r_rows, r_offs, total = emb.exchange_simulated(to_dev(ids), to_dev(rows) if D else None, to_dev(offs))
    torch.cuda.synchronize()
    want = [(w, slice(offs[w, p], offs[w, p + 1])) for p in range(P) for w in range(P)]
    n = int(offs[:, P].sum())
    starts = np.cumsum([0] + [offs[w, p + 1] - offs[w, p] for p in range(P) for w in range(P)])
    got = host(r_offs)
    assert int(total.item()) == n and np.array_equal(got[:, :P].ravel(), starts[:-1])
    assert np.array_equal(got[:, P], starts[P::P])
    assert np.array_equal(host(r_ids)[:n], np.concatenate([ids[w, s] for w, s in want]))
    if D:
        assert np.array_equal(host(r_rows)[:n], np.concatenate([rows[w, s] for w, s in want]))
