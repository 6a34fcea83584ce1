"""GPU kernels at the sizes where their splits change: edges of registers, waves and tables."""
import numpy as np
import pytest

import oracle
import synth
from parity import check_bank_order

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sindi():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_08395_amd as s
    s._lib.load()
    return s


def _np(t):
    return t.detach().cpu().numpy()


def _rows(rng, lens, vocab, ties=False):
    """Signed rows of exactly these lengths; with ties every |value| is one of four, zero too."""
    indptr = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=indptr[1:])
    ids = np.concatenate([np.sort(rng.choice(vocab, n, replace=False)) for n in lens] or [[]])
    val = (rng.choice([0.0, 0.5, 1.0, 2.0], indptr[-1]) if ties else rng.lognormal(0, 0.8, indptr[-1]))
    val = val * rng.choice([-1.0, 1.0], indptr[-1])
    return synth.Csr(indptr, ids.astype(np.int32), val.astype(np.float32), vocab)


# ------------------------------------------------------------------ query preparation
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("beta", [0.8, 0.3, 1.0])
def test_query_prep_row_lengths(sindi, beta, ties):
    """beta-mass rows on both sides of every register split: the same coarse results, bit for
    bit, as the rows the oracle pruned (the coarse weights are then the same numbers)."""
    rng = np.random.default_rng(5)
    vocab = 3_000
    corpus = synth.random_csr(rng, 3_000, vocab, 60, signed=True)
    lens = [0, 1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 700]
    q = _rows(rng, lens, vocab, ties)
    idx = sindi.Index(corpus, alpha=1.0, window=1_000, value_dtype="f32")
    got = idx.search_coarse(sindi.DeviceCsr.from_host(q), 40, beta=beta)
    cut = oracle.apply_mask(q, oracle.mass_prune(q, beta))
    ref = idx.search_coarse(sindi.DeviceCsr.from_host(cut), 40)
    assert np.array_equal(_np(got[0]), _np(ref[0]))
    assert np.array_equal(_np(got[1]).view(np.uint32), _np(ref[1]).view(np.uint32))


# ------------------------------------------------------------------ rerank
def test_rerank_table_sizes(sindi):
    """Query rows around every table size (full and spilling tables among them) against document
    rows around every 64-entry round: FP32 inner products within the rounding of their sums."""
    rng = np.random.default_rng(6)
    vocab, nd = 5_000, 210
    corpus = _rows(rng, [0, 1, 2, 63, 64, 65, 127, 128, 129, 130, 192, 193, 300] * 16 + [0, 77], vocab)
    q = _rows(rng, [0, 1, 7, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 512, 513, 1500, 4096], vocab)
    idx = sindi.Index(corpus, alpha=0.5, window=100, value_dtype="f32")
    for rows in (np.arange(q.n_rows), np.array([9]), np.array([18])):  # many and few workgroups
        sub = q.take_rows(rows)
        ids, sc = (_np(t) for t in idx.search(sindi.DeviceCsr.from_host(sub), nd, gamma=nd))
        assert all(sorted(r) == list(range(nd)) for r in ids.tolist())
        qi = np.repeat(np.arange(sub.n_rows), nd)
        ref = oracle.pair_scores(corpus, sub, qi, ids.reshape(-1))
        mag = lambda m: synth.Csr(m.indptr, m.indices, np.abs(m.values), m.n_cols)
        # at most 5 additions on a lane and 6 across the wave, each within 2^-24 of the partial sums
        tol = 11 * 2.0 ** -24 * oracle.pair_scores(mag(corpus), mag(sub), qi, ids.reshape(-1))
        assert (np.abs(sc.reshape(-1) - ref) <= tol + 1e-30).all()


# ------------------------------------------------------------------ pair scores
@pytest.mark.parametrize("n_cand", [1, 3, 16, 17, 130])
@pytest.mark.parametrize("lens", [[0, 1, 8, 9, 64, 65, 129], [512, 513], [4096], [12] * 700])
def test_pair_scores_and_gradients_at_split_edges(sindi, n_cand, lens):
    """Scores and gradients against the FP64 oracle, each within the rounding of its additions:
    one to many workgroups per query, every table size, rows around every 64-entry round, ids
    outside the corpus and candidates shared by several queries."""
    rng = np.random.default_rng(7)
    vocab, u = 5_000, 2.0 ** -24
    corpus = _rows(rng, [0, 1, 63, 64, 65, 127, 128, 129, 192, 300] * 9, vocab)
    q = _rows(rng, lens, vocab)
    nq, nd = q.n_rows, corpus.n_rows
    cand = rng.integers(-1, nd, (nq, n_cand))
    g = rng.standard_normal((nq, n_cand)).astype(np.float32)
    idx = sindi.Index(corpus, alpha=0.5, window=100)
    dq, tc = sindi.DeviceCsr.from_host(q), torch.from_numpy(cand).cuda()
    xv = torch.from_numpy(corpus.values).cuda()
    s = _np(idx.score(dq, tc, doc_values=xv))
    mag = lambda m: synth.Csr(m.indptr, m.indices, np.abs(m.values), m.n_cols)
    qi = np.repeat(np.arange(nq), n_cand)
    ok = cand.reshape(-1) >= 0
    ref = np.where(ok, oracle.pair_scores(corpus, q, qi, np.maximum(cand, 0).reshape(-1)), 0.0)
    size = oracle.pair_scores(mag(corpus), mag(q), qi, np.maximum(cand, 0).reshape(-1))
    assert (np.abs(s.reshape(-1) - ref) <= 11 * u * size + 1e-30).all()
    gq, gx = torch.zeros_like(dq.values), torch.zeros_like(xv)
    idx.score_backward(dq, tc, torch.from_numpy(g).cuda(), gq, gx, doc_values=xv)
    rq, rx = oracle.score_grad(corpus, q, cand, g.astype(np.float64))
    sq, sx = oracle.score_grad(mag(corpus), mag(q), cand, np.abs(g).astype(np.float64))
    m = np.bincount(cand.reshape(-1)[ok], minlength=1).max() if ok.any() else 0
    assert (np.abs(_np(gq) - rq) <= (n_cand + 3) * u * sq + 1e-30).all()
    assert (np.abs(_np(gx) - rx) <= (m + 2) * u * sx + 1e-30).all()


# ------------------------------------------------------------------ selection
def _int_setup(nd, nq, signed, seed=8):
    """Small integer values: every product and sum is exact, and most scores tie."""
    rng = np.random.default_rng(seed)
    vocab = 60
    corpus = synth.random_csr(rng, nd, vocab, 6)
    q = synth.random_csr(rng, nq, vocab, 5, min_nnz=1)
    draw = [-2.0, -1.0, 1.0, 2.0] if signed else [1.0, 2.0]
    corpus = synth.Csr(corpus.indptr, corpus.indices, rng.choice(draw, corpus.nnz).astype(np.float32), vocab)
    q = synth.Csr(q.indptr, q.indices, np.ones(q.nnz, np.float32), vocab)
    dense = np.zeros((nd, vocab))
    dense[np.repeat(np.arange(nd), np.diff(corpus.indptr)), corpus.indices] = corpus.values
    qd = np.zeros((nq, vocab))
    qd[np.repeat(np.arange(nq), np.diff(q.indptr)), q.indices] = q.values
    return corpus, q, qd @ dense.T


def _ranked(scores, k):
    """The first k of every row, score descending, equal scores by ascending id."""
    ids = np.argsort(-scores, axis=1, kind="stable")[:, :k]
    return ids, np.take_along_axis(scores, ids, 1)


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("nd, cand_cap", [(1, 0), (255, 0), (2047, 0), (2049, 0), (8193, 0), (9001, 2500)])
@pytest.mark.parametrize("nq", [3, 520])
def test_selection_with_ties(sindi, nd, cand_cap, nq, signed):
    """Top-k of scores that mostly tie, over every workgroup size, register and memory path,
    with every document a candidate and with a candidate threshold: exactly the ranking order."""
    corpus, q, scores = _int_setup(nd, nq, signed)
    idx = sindi.Index(corpus, alpha=1.0, window=4_000, tile=1_000)
    dq = sindi.DeviceCsr.from_host(q)
    for k, gamma in ((1, 0), (50, 500), (256, 300), (257, 600), (1, 2049), (600, 2100)):
        ref = _ranked(scores, k)
        n = ref[0].shape[1]
        for got in (idx.search_coarse(dq, k, cand_cap=cand_cap),
                    idx.search(dq, k, gamma=gamma, cand_cap=cand_cap)):
            ids, sc = _np(got[0]), _np(got[1])
            assert np.array_equal(ids[:, :n], ref[0]) and np.array_equal(sc[:, :n], ref[1])
            assert (ids[:, n:] == -1).all() and np.isneginf(sc[:, n:]).all()


# ------------------------------------------------------------------ calls of few entries
@pytest.mark.parametrize("lens", [[35], [512], [513], [60, 68], [60, 69], [0], [0, 3]])
def test_few_entries_malformed_device_queries_write_nothing(sindi, lens):
    """Device queries on both sides of the sizes that are searched without waiting for their
    check: each malformed form is refused with the outputs untouched, and the next call on the
    same index is right."""
    rng = np.random.default_rng(9)
    vocab = 2_000
    corpus = synth.random_csr(rng, 4_000, vocab, 40)
    idx = sindi.Index(corpus, alpha=0.6, window=1_500)
    q = _rows(rng, lens, vocab)
    good = sindi.DeviceCsr.from_host(q)
    host = idx.search(q, 7, gamma=90)  # checked on the host
    nnz = q.nnz

    def broken():
        p, i, v = (t.clone() for t in (good.indptr, good.indices, good.values))
        p[0] = 1
        yield sindi.DeviceCsr(p, i, v, vocab)
        p = good.indptr.clone()
        p[-1] = nnz + 5
        yield sindi.DeviceCsr(p, i, v, vocab)
        p = good.indptr.clone()
        p[-1] = -3
        yield sindi.DeviceCsr(p, i, v, vocab)
        if nnz > 1:
            for bad in (vocab, -1, int(i[0])):
                j = i.clone()
                j[1] = bad
                yield sindi.DeviceCsr(good.indptr, j, v, vocab)
            w = v.clone()
            w[nnz - 1] = float("nan")
            yield sindi.DeviceCsr(good.indptr, i, w, vocab)

    out = (torch.full((q.n_rows, 7), -7, dtype=torch.int64, device="cuda"),
           torch.full((q.n_rows, 7), 7.0, device="cuda"))
    for bad in broken():
        for call in (lambda: idx.search(bad, 7, gamma=90, out=out),
                     lambda: idx.search_coarse(bad, 7, out=out)):
            with pytest.raises(sindi.SindiError, match="malformed"):
                call()
            assert (out[0] == -7).all() and (out[1] == 7.0).all()
    got = idx.search(good, 7, gamma=90)
    assert torch.equal(got[0], host[0]) and torch.equal(got[1], host[1])
    with pytest.raises(sindi.SindiError, match="malformed"):
        idx.score(next(broken()), torch.zeros((q.n_rows, 3), dtype=torch.int64, device="cuda"))


# ------------------------------------------------------------------ scoring items
@pytest.mark.parametrize("run", [1, 8, 64])
@pytest.mark.parametrize("schedule", [1, 2])
def test_items_of_many_queries(sindi, run, schedule):
    """Items of up to 64 queries over one tile, with few and with hundreds of candidates per query
    and tile (the workgroup's candidate buffer filling, flushed inside an item and passed), tiles
    of 1 to 16,384 documents: exactly the ranking order."""
    corpus, q, scores = _int_setup(17_400, 600, False, seed=10)
    ref = _ranked(scores, 40)
    for tile, window, cap in ((16_384, 16_384, 2_500), (1_000, 3_001, 400)):
        idx = sindi.Index(corpus, alpha=1.0, window=window, tile=tile, value_dtype="f16")
        reps = max(1, -(-4096 * run // (600 * idx.info()["n_tiles"])))  # items enough for the run
        many = synth.Csr(np.concatenate([[0], np.cumsum(np.tile(np.diff(q.indptr), reps))]),
                         np.tile(q.indices, reps), np.tile(q.values, reps), q.n_cols)
        got = idx.search_coarse(sindi.DeviceCsr.from_host(many), 40, cand_cap=cap, tile_run=run,
                                schedule=schedule)
        assert np.array_equal(_np(got[0]), np.tile(ref[0], (reps, 1)))
        assert np.array_equal(_np(got[1]), np.tile(ref[1], (reps, 1)))


@pytest.mark.parametrize("n_tiles", [7, 8, 9, 15, 26])
def test_items_over_queues(sindi, n_tiles):
    """Eight work queues of equal and unequal length (tiles off every multiple of eight), from which
    the workgroups that run dry take: every item is scored once, exactly as by a workgroup each."""
    corpus, q, scores = _int_setup(100 * n_tiles - 37, 600, False, seed=12)
    ref = _ranked(scores, 30)
    idx = sindi.Index(corpus, alpha=1.0, window=100, tile=100, value_dtype="f16")
    assert idx.info()["n_tiles"] == n_tiles
    for run in (1, 0):  # 4,200 to 15,600 items of one query, and the call's own choice
        got = idx.search_coarse(sindi.DeviceCsr.from_host(q), 30, tile_run=run, sample_tiles=n_tiles)
        assert np.array_equal(_np(got[0]), ref[0])
        assert np.array_equal(_np(got[1]), ref[1])


# ------------------------------------------------------------------ device build
@pytest.mark.parametrize("nd, vocab, tile", [(255, 9, 300), (513, 4_001, 600), (5_000, 33_000, 5_000),
                                             (9_001, 70_001, 700), (40_000, 300, 1_000)])
def test_device_build_parts(sindi, nd, vocab, tile):
    """Tiles cut into one to sixteen parts, one to three fill passes, vocabularies off every vector
    and round width: the same arrays as the host build."""
    rng = np.random.default_rng(11)
    corpus = synth.random_csr(rng, nd, vocab, min(40, vocab), signed=True)
    a, b = (sindi.Index(corpus, alpha=0.7, window=max(tile, nd // 2), tile=tile, value_dtype="bf16",
                        gpu_build=g).export(raw=True) for g in (False, True))
    for name in a:
        assert np.array_equal(a[name], b[name]), name


@pytest.mark.parametrize("vocab, tile", [(1_027, 5_000), (262_149, 5_000), (262_143, 250), (524_289, 250),
                                         (524_293, 125)])
def test_bank_order_of_every_run(sindi, vocab, tile):
    """Waves of one to eight neighbouring lists (terms times tiles on both sides of the rule's
    steps, vocabularies off every run and wave): every chunk in LDS-bank order."""
    nd = 1_001
    rng = np.random.default_rng(23)
    lists = rng.choice(vocab, 150, replace=False)  # long ones, the first and the last terms among them
    lists[:3] = 0, vocab - 2, vocab - 1
    lists = np.unique(np.concatenate([lists, lists[3:] // 8 * 8 + 7])).astype(np.int32)
    lists = lists[lists < vocab]
    rows = [lists[rng.random(lists.size) < 0.3] for _ in range(nd)]
    indptr = np.concatenate([[0], np.cumsum([r.size for r in rows])])
    corpus = synth.Csr(indptr, np.concatenate(rows), rng.lognormal(0, 0.8, indptr[-1]).astype(np.float32), vocab)
    idx = sindi.Index(corpus, alpha=1.0, window=nd, tile=tile, value_dtype="f16", gpu_build=True)
    check_bank_order(idx.export(raw=True), idx.export())


def test_rebuilt_indexes_reuse_and_return_memory(sindi):
    """Indexes built beside the one they replace take its memory over (old contents must not
    show), and the last one to go gives the library's memory back to the driver."""
    def corpus(nd, seed):
        return synth.generate(nd, 3_000, nnz=("poisson", 60.0), seed=seed)
    q = synth.generate(20, 3_000, nnz=("poisson", 15.0), seed=3, stream=1)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    want = []
    for seed in range(3):
        idx = sindi.Index(corpus(30_000 - 500 * seed, seed), alpha=0.5, window=10_000, value_dtype="f16")
        want.append(tuple(_np(t) for t in idx.search(q, 10, gamma=60)))
        idx.close()
    live = None
    for k in range(9):
        new = sindi.Index(corpus(30_000 - 500 * (k % 3), k % 3), alpha=0.5, window=10_000,
                          value_dtype="f16", gpu_build=k % 2 == 0)
        got = tuple(_np(t) for t in new.search(q, 10, gamma=60))
        assert np.array_equal(got[0], want[k % 3][0]) and np.array_equal(got[1], want[k % 3][1])
        if live:
            live.close()
        live = new
    live.close()
    torch.cuda.synchronize()
    assert free0 - torch.cuda.mem_get_info()[0] < 64 << 20  # torch's own small results


# ------------------------------------------------------------------ empty index
def test_search_and_server_over_an_empty_index(sindi):
    """No documents: every result is padding.  The pass then ends with the report launch, whose
    words the server keeps a buffer for of its own."""
    corpus = synth.Csr(np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0, np.float32), 50)
    idx = sindi.Index(corpus, alpha=0.5, window=1_000)
    q = _rows(np.random.default_rng(13), [0, 3, 7], 50)
    for queries in (q, sindi.DeviceCsr.from_host(q)):
        for ids, sc in (idx.search(queries, 5), idx.search_coarse(queries, 5)):
            assert (_np(ids) == -1).all() and np.isneginf(_np(sc)).all()
    with sindi.Server(idx, max_inflight=2, max_batch=2, k_max=5) as srv:
        got = srv.replay(q, np.full(3, 5, np.int32), np.zeros(3))
    assert (np.asarray(got[0]) == -1).all() and np.isneginf(np.asarray(got[1])).all()


# ------------------------------------------------------------------ thresholds out of reach
@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("tile, short", [(500, 300), (400, 1), (600, 511)])
def test_fewer_sampled_maxima_than_the_rank(sindi, tile, short, batch):
    """Tiles of fewer documents than sampling threads and a pool that asks for more maxima than
    there are: no threshold is found, and the retries give exactly the ranking order."""
    nd = 6 * tile + short
    need = nd // 2 - 3
    # every tile is sampled: the rank exceeds the maxima that documents have
    assert 6 * min(tile, 512) + min(short, 512) < min(2 * need + 8, 7 * 512)
    corpus, q, scores = _int_setup(nd, 40, False, seed=14)
    idx = sindi.Index(corpus, alpha=1.0, window=tile, tile=tile)
    assert idx.info()["n_tiles"] == 7
    ref = _ranked(scores, 30)
    for schedule in (1, 2):
        got = idx.search(sindi.DeviceCsr.from_host(q), 30, gamma=need, cand_cap=200, batch=batch,
                         schedule=schedule)
        assert np.array_equal(_np(got[0]), ref[0]) and np.array_equal(_np(got[1]), ref[1])


# ------------------------------------------------------------------ candidates past the buffer
@pytest.mark.parametrize("gamma", [90, 300, 1_100, 2_900])
@pytest.mark.parametrize("order", ["mixed", "sorted"])
@pytest.mark.parametrize("tile", [16_381, 2_300, 257])
def test_candidates_past_the_workgroups_buffer(sindi, tile, order, gamma):
    """From a few to thousands of candidates per query and tile, spread over the corpus or gathered
    in its first tiles, so that steps place theirs lane by lane, together, across the buffer's end
    and past it, whole steps and the one across the tile's end: exactly the ranking order."""
    rng = np.random.default_rng(15)
    nd, nq, vocab = 16_381, 70, 40
    dense = rng.choice([0.0, 1.0, 2.0, 3.0], (nd, vocab), p=[0.6, 0.2, 0.1, 0.1])
    if order == "sorted":
        dense = dense[np.argsort(-dense[:, :12].sum(1), kind="stable")]
    lens = (dense != 0).sum(1)
    corpus = synth.Csr(np.concatenate([[0], np.cumsum(lens)]), np.nonzero(dense)[1].astype(np.int32),
                       dense[dense != 0].astype(np.float32), vocab)
    qd = np.zeros((nq, vocab))
    qd[:, :12] = rng.choice([1.0, 2.0, 5.0], (nq, 12))
    q = synth.Csr(np.arange(nq + 1, dtype=np.int64) * 12, np.tile(np.arange(12, dtype=np.int32), nq),
                  qd[:, :12].reshape(-1).astype(np.float32), vocab)
    ref = _ranked(qd @ dense.T, gamma)
    idx = sindi.Index(corpus, alpha=1.0, window=16_384, tile=tile, value_dtype="f16")
    for run in (1, 64):
        ids, sc = (_np(t) for t in idx.search_coarse(sindi.DeviceCsr.from_host(q), gamma, cand_cap=9_000,
                                                     sample_tiles=64, tile_run=run))
        assert np.array_equal(ids, ref[0]) and np.array_equal(sc, ref[1])


# ------------------------------------------------------------------ limits of the calls
def test_largest_candidate_buffer(sindi):
    """The candidate buffer's limit (its bitmap and the pool's keys in LDS): the largest size is
    taken, one entry more is refused."""
    nd, vocab = 1_300_000, 64
    rng = np.random.default_rng(16)
    ids = np.sort(rng.integers(0, vocab // 2, (nd, 2)) * 2 + [0, 1], axis=1).astype(np.int32)
    corpus = synth.Csr(np.arange(nd + 1, dtype=np.int64) * 2, ids.reshape(-1),
                       rng.lognormal(0, 0.8, 2 * nd).astype(np.float32), vocab)
    idx = sindi.Index(corpus, alpha=1.0, window=100_000, value_dtype="f32", gpu_build=True)
    q = sindi.DeviceCsr.from_host(_rows(rng, [3, 1, 2], vocab))
    ref = idx.search(q, 20, gamma=500)
    got = idx.search(q, 20, gamma=500, cand_cap=1_269_004)
    assert torch.equal(ref[0], got[0]) and torch.equal(ref[1], got[1])
    with pytest.raises(sindi.SindiError):
        idx.search(q, 20, gamma=500, cand_cap=1_269_005)


def test_largest_index_of_a_search_without_allocations(sindi):
    """The static array's limit, one query of the pass that keeps every document: the largest index
    is searched, with one document more the call is refused and leaves its outputs."""
    import ctypes
    lib = sindi._lib.load()
    q = sindi.DeviceCsr.from_host(synth.Csr(np.array([0, 1], np.int64), np.zeros(1, np.int32),
                                            np.ones(1, np.float32), 1))
    qs, p = q.struct(), sindi._lib.SindiSearchParams(1.0, 5, 0, 0, 0, 0)
    for nd, fits in ((33_553_984, True), (33_553_985, False)):
        indptr = np.zeros(nd + 1, np.int64)
        indptr[nd - 2:] = [1, 2, 2]
        corpus = synth.Csr(indptr, np.zeros(2, np.int32), np.array([1, 2], np.float32), 1)
        idx = sindi.Index(corpus, alpha=1.0, window=100_000, value_dtype="f32", gpu_build=True)
        ids = torch.full((1, 5), -7, dtype=torch.int64, device="cuda")
        sc = torch.full((1, 5), 7.0, device="cuda")
        rc = lib.sindi_search_noalloc(idx._h, ctypes.byref(qs), 5, ctypes.byref(p),
                                      ctypes.c_void_p(ids.data_ptr()), ctypes.c_void_p(sc.data_ptr()),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        idx.close()
        if fits:
            assert rc == 0
            assert ids.tolist() == [[nd - 2, nd - 3, 0, 1, 2]] and sc.tolist() == [[2.0, 1.0, 0.0, 0.0, 0.0]]
        else:
            assert rc == sindi._lib.SINDI_E_INVALID
            assert (ids == -7).all() and (sc == 7.0).all()


# ------------------------------------------------------------------ implicit zeros
@pytest.mark.parametrize("nd, cand_cap", [(12_000, 5_000), (12_000, 2_060), (3_000, 2_700)])
@pytest.mark.parametrize("signed", [False, True])
def test_pools_of_positives_zeros_and_negatives(sindi, nd, cand_cap, signed):
    """Pools of one to thousands of positive sums, of documents without a common term, and of
    negative sums where those run out, from registers and from memory: exactly the ranking order."""
    rng = np.random.default_rng(17)
    vocab, nq = 50, 24
    dense = np.where(rng.random((nd, vocab)) < np.linspace(0.0005, 0.8, vocab) ** 2, rng.choice([1.0, 2.0], (nd, vocab)), 0.0)
    if signed:
        dense *= rng.choice([-1.0, 1.0], (nd, vocab), p=[0.8, 0.2])
    corpus = synth.Csr(np.concatenate([[0], np.cumsum((dense != 0).sum(1))]), np.nonzero(dense)[1].astype(np.int32),
                       dense[dense != 0].astype(np.float32), vocab)
    terms = rng.integers(0, vocab, nq).astype(np.int32)
    q = synth.Csr(np.arange(nq + 1, dtype=np.int64), terms, np.ones(nq, np.float32), vocab)
    idx = sindi.Index(corpus, alpha=1.0, window=1_000, tile=500)
    for k in (10, 2_000):
        ref = _ranked(dense.T[terms], k)
        got = idx.search_coarse(sindi.DeviceCsr.from_host(q), k, cand_cap=cand_cap)
        assert np.array_equal(_np(got[0]), ref[0]) and np.array_equal(_np(got[1]), ref[1])


# ------------------------------------------------------------------ memory kept between builds
def test_memory_kept_between_builds_is_bounded_and_released(sindi):
    """What the library keeps idle: no more than the live indexes hold, nothing once it is told to
    release it or the last index is gone."""
    nd, vocab, n = 400_000, 2_000, 40
    g = torch.Generator("cuda").manual_seed(18)
    ids = (torch.rand((nd, vocab // n), device="cuda", generator=g) * n).int()
    ids += torch.arange(vocab // n, device="cuda", dtype=torch.int32) * n
    values = torch.rand(ids.numel(), device="cuda", generator=g) + 0.1
    corpus = sindi.DeviceCsr(torch.arange(nd + 1, device="cuda") * ids.shape[1], ids.reshape(-1), values, vocab)
    del ids

    def build():
        return sindi.Index(corpus, alpha=0.6, window=100_000, value_dtype="f16", gpu_build=True)

    def held():  # by the library: torch allocates nothing in between
        torch.cuda.synchronize()
        return free0 - torch.cuda.mem_get_info()[0]

    build().close()  # code objects and the like are loaded
    sindi.release_memory()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    slack = 4 << 20  # below any of the large arrays
    a = build()
    size = a.info()["device_bytes"]
    assert size > 16 * slack
    sindi.release_memory()  # the build's scratch
    alone = held()
    assert size - slack < alone < size * 17 // 16 + slack
    for _ in range(3):
        b = build()
        a.close()
        a = b
        assert held() <= 2 * alone + slack
    assert held() >= alone + slack  # something is kept for the next build
    sindi.release_memory()
    assert abs(held() - alone) < slack
    b = build()
    a.close()
    assert held() <= 2 * alone + slack
    b.close()
    assert held() < slack


# ------------------------------------------------------------------ large grids
@pytest.mark.parametrize("nd, nq, tile", [(100_000, 1_400, 16), (140_001, 3, 2)])
def test_items_beyond_one_grid_dimension(sindi, nd, nq, tile):
    """One workgroup per item, more items than threads of one grid dimension can count and more
    tiles than its second holds: every item is scored, as from the queues."""
    corpus = synth.generate(nd, 300, nnz=("poisson", 6.0), seed=19)
    q = sindi.DeviceCsr.from_host(synth.generate(nq, 300, nnz=("poisson", 4.0), seed=20, stream=1))
    idx = sindi.Index(corpus, alpha=1.0, window=nd, tile=tile)
    ref = idx.search(q, 10, gamma=100)
    got = idx.search(q, 10, gamma=100, schedule=1, tile_run=1)
    assert torch.equal(ref[0], got[0]) and torch.equal(ref[1], got[1])


@pytest.mark.parametrize("tile, batch", [(3_836, 8), (8_700, 4)])
@pytest.mark.parametrize("lens", [[25, 9, 12, 9], [20]])
def test_merged_batches_of_few_entries_beside_full_tiles(sindi, tile, batch, lens):
    """Merged batches whose score rows leave the lists room for short queries only: calls of few
    entries in all are taken where each of their rows fits, as calls of many are."""
    rng = np.random.default_rng(21)
    corpus = synth.generate(3 * tile, 500, nnz=("poisson", 5.0), seed=22)
    idx = sindi.Index(corpus, alpha=1.0, window=tile, tile=tile)
    q = sindi.DeviceCsr.from_host(_rows(rng, lens, 500))
    ref, got = idx.search(q, 10, gamma=100), idx.search(q, 10, gamma=100, batch=batch)
    assert torch.equal(ref[0], got[0]) and torch.equal(ref[1], got[1])
