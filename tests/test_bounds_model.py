"""CPU bounds model of the kernels' indexing.

For every supported shape (b in {16, 64}, dh in {32, 64, 128}, fp32/bf16),
this mirrors the largest element offset each kernel touches in each buffer
(from its loop bounds and lane mappings) and checks it lies inside the buffer
the ABI sizes for it.  It runs before any kernel change goes to a GPU: an
access past a tensor's end is caught here, not as a memory fault."""
import ctypes
import functools
import itertools
import os
import subprocess
import tempfile

import pytest

SPLIT_CAP = 64
SPLIT_STRIDE = SPLIT_CAP + 1
SPLIT_CAP_PREFILL = 32
MIN_PAGES_DECODE = 8
MIN_PAGES_PREFILL = 4


def pages_per_split(n_read, min_pages, cap=SPLIT_CAP):
    return max(min_pages, -(-n_read // cap))


def test_xcd_order_is_a_bijection():
    for T in list(range(1, 70)) + [384, 3142, 50257]:
        items = [plan().lp_xcd_order(i, T) for i in range(plan().lp_xcd_grid(T))]
        assert sorted(p for p in items if p >= 0) == list(range(T))
        per = plan().lp_xcd_grid(T) // 8    # each XCD's items are one contiguous range
        for x in range(8):
            mine = [p for i, p in enumerate(items) if i % 8 == x and p >= 0]
            assert mine == list(range(x * per, min(T, (x + 1) * per)))


def page_head_offset(page, h, H, b, dh):
    return (page * H + h) * 2 * b * dh


SHAPES = [(b, dh, es) for b in (16, 64) for dh in (32, 64, 128) for es in (4, 2)]


@pytest.mark.parametrize("b,dh,es", SHAPES)
def test_reader_valu_indexing(b, dh, es):
    E = 16 // es
    LPR = dh // E
    RPL = 64 // LPR
    KLOADS = b // RPL
    LPV = b // E
    DPL = 64 // LPV
    VLOADS = dh // DPL
    assert RPL * LPR == 64 and KLOADS * RPL == b and DPL * LPV == 64 and VLOADS * DPL == dh
    for H, n_pages, n_slots, nq in [(1, 1, 1, 1), (16, 4096, 64, 1), (4, 9, 16, b), (64, 3, 128, 1)]:
        pool = n_pages * H * 2 * b * dh
        base = page_head_offset(n_pages - 1, H - 1, H, b, dh)
        k_max = base + ((KLOADS - 1) * RPL + RPL - 1) * dh + (LPR - 1) * E + E - 1
        v_max = base + b * dh + ((VLOADS - 1) * DPL + DPL - 1) * b + (LPV - 1) * E + E - 1
        assert k_max < pool and v_max < pool
        # query / output rows: ((qs*H + h)*dh + c*E) + E - 1
        rows = n_slots * nq
        assert ((rows - 1) * H + H - 1) * dh + (LPR - 1) * E + E - 1 < rows * H * dh
        # in-block keys: ((slot*b + r)*H + h)*dh, r < b; decode cache write at pos < b
        assert (((n_slots - 1) * b + b - 1) * H + H - 1) * dh + (LPR - 1) * E + E - 1 < n_slots * b * H * dh
        # null row [2][H][dh]
        assert ((1 * H + H - 1) * dh + (LPR - 1) * E + E - 1) < 2 * H * dh
        # split partials: split index <= memory splits <= cap, rows (query rows x heads) fit the workspace
        for n_read in (0, 1, 63, 64, 65, 4096, 65536):
            pps = pages_per_split(n_read, 4 if dh <= 32 else MIN_PAGES_DECODE)
            nms = -(-n_read // pps)
            nsplit = nms + 1   # the null row and in-block keys have their own split
            assert nsplit <= SPLIT_STRIDE
            assert ((rows * H - 1) * SPLIT_STRIDE + nsplit - 1) * (dh + 4) + dh + 1 < rows * H * SPLIT_STRIDE * (dh + 4)
            # wave w of split k reads live entries k*pps + w + 4i < min(n_read, (k+1)*pps)
            for k in {0, max(0, nms - 1)}:
                p0, p1 = k * pps, min(n_read, k * pps + pps)
                assert all(pi < n_read for pi in range(p0, p1))


@pytest.mark.parametrize("dh", [32, 64, 128])
def test_mfma_indexing(dh):
    BT = 64
    # in-block transpose: (row pair, chunk) jobs cover 64 rows x dh, each writes dims c8*8..+7 at rows 2p, 2p+1
    NP = 32 * (dh // 8)
    CPR = dh // 8
    jobs = [((j // CPR), (j % CPR)) for j in range(NP)]       # (row pair, chunk): chunks of a pair adjacent
    assert len(set(jobs)) == NP and max(p for p, _ in jobs) == 31 and max(c for _, c in jobs) * 8 + 7 < dh
    # prefill partials: at most 32 splits (split 0 also reads the in-block tile) inside the 65-wide stride
    for n_read in (0, 1, 4, 5, 512, 4096, 65536):
        for H in (1, 12, 16, 24, 32, 64, 600):
            cap = min(SPLIT_CAP_PREFILL, max(1, 512 // H))       # prefill_split_cap(H)
            pps = pages_per_split(n_read, MIN_PAGES_PREFILL, cap)
            assert max(-(-n_read // pps), 1) <= cap <= SPLIT_CAP_PREFILL <= SPLIT_STRIDE
    # output/ws lane writes: d0 = dt*16 + g*4, 4 values
    assert (dh // 16 - 1) * 16 + 3 * 4 + 3 < dh


def test_prefill_workspace_fits_slot_chunk():
    # prefill launches at most min(16, n_seq * max_blocks) slots of b query
    # rows each (one sequence may fill several slots); decode at most
    # min(128, n_seq) slots of one row (a sequence appears once)
    for n_seq, mb, b, H, dh in itertools.product((1, 8, 16, 64), (1, 3, 40), (16, 64), (1, 16), (32, 128)):
        dec_rows = n_seq * H
        slots = min(n_seq * mb, 16)
        pre_rows = slots * b * H
        ws = max(dec_rows, pre_rows) * SPLIT_STRIDE * (dh + 4)
        assert (slots * b * H) * SPLIT_STRIDE * (dh + 4) <= ws
        assert (min(128, n_seq) * 1 * H) * SPLIT_STRIDE * (dh + 4) <= ws


@pytest.mark.parametrize("b,dh,es", SHAPES)
def test_rope_table_indexing(b, dh, es):
    """Rotary table reads: row phase * dh, columns 2*k0 + 4m .. +3 per 16-byte read.
    The host admits a call only when every phase it uses is below n_phases."""
    E = 16 // es
    LPR = dh // E
    for c in range(LPR):                      # VALU reader: lane chunk c, pairs c*E/2 ..
        k0 = c * (E // 2)
        assert k0 % 2 == 0 and 2 * k0 + 4 * (E // 4 - 1) + 3 < dh
    for kk in range(dh // 32):                # MFMA query fragments
        for g in range(4):
            k0 = kk * 16 + g * 4
            assert 2 * k0 + 4 + 3 < dh
    for c8 in range(dh // 8):                 # MFMA key tile rows
        assert 2 * (c8 * 4) + 4 + 3 < dh
    for J, W in [(0, 0), (1, 15), (40, 15), (4096, 0), (4096, 15)]:
        turn = min(J, W) if W > 0 else J
        n_phases = max(b - 1, turn) + 1       # smallest table the host admits
        clip = W if W > 0 else 2 ** 31 - 1
        for j in {0, max(0, J - 1), max(0, J - W)} if J > 0 else set():
            if j < J:
                dlt = min(J - j, clip)
                assert 1 <= dlt < n_phases
        assert min(J, clip) < n_phases and b - 1 < n_phases
        assert (n_phases - 1) * dh + dh - 1 < n_phases * dh


@pytest.mark.parametrize("dh", [32, 64, 128])
def test_rope_prefill_lds_rows(dh):
    """Rotary prefill split: turns of its pages (ascending block index) fall
    monotonically, so every page's turn lies in [d_lo, d_hi]; the LDS copy of
    rows d_lo..d_hi (taken when it has fewer than 24 rows) fits its array and
    reads inside the table; the page ring and the rows fit two workgroups
    per CU (160 KiB of LDS)."""
    ROWS = 24
    rng = __import__("random").Random(dh)
    for _ in range(200):
        J = rng.randint(1, 5000)
        W = rng.choice([0, 1, 3, 15, 31, 100])
        clip = W if W > 0 else 2 ** 31 - 1
        blocks = sorted(rng.sample(range(J), min(J, rng.randint(1, 40))))
        n_phases = max(63, min(J, W) if W > 0 else J) + 1
        d = [min(J - j, clip) for j in blocks]
        assert d == sorted(d, reverse=True)
        d_hi, d_lo = d[0], d[-1]
        assert all(d_lo <= x <= d_hi for x in d) and d_hi < n_phases
        if d_hi - d_lo < ROWS:
            n4 = (d_hi - d_lo + 1) * dh // 4
            assert n4 * 4 <= ROWS * dh
            assert d_lo * dh + n4 * 4 <= n_phases * dh
            assert all((x - d_lo) * dh + dh <= ROWS * dh for x in d)
    # LDS per workgroup: the page ring (its first stage takes the in-block tile) + rows; two workgroups per CU
    tile, _, _, ns, _ = _ints(plan().ap_ring, 5, dh)
    assert 2 * (ns * tile + ROWS * dh * 4) <= 160 * 1024


def _pps_rows(n):
    return max(8, -(-n // 32))


@pytest.mark.parametrize("b,D", [(b, D) for b in (16, 64) for D in (512, 768, 1024, 2048)])
def test_rows_reader_indexing(b, D):
    """Row-plane reader: chunk loads stay inside a page, LDS reads inside the
    chunk and query tiles, and a launch's split partials inside the workspace."""
    N = 16 * D // 8 // 256
    assert N * 256 * 8 == 16 * D
    assert (255 + (N - 1) * 256) * 8 + 7 < 16 * D               # one 16-row chunk
    assert (b // 16 - 1) * 16 * D + 16 * D <= b * D              # last chunk of a page
    # chunk DMA: per row ceil(D / 512) instructions of 64 lanes x 8 elements;
    # a lane loads only inside its row, and the row's elements are all loaded
    RI = -(-D // 512)
    loaded = set()
    for hk in range(RI):
        for lane in range(64):
            if hk * 512 + 512 <= D or hk * 512 + lane * 8 < D:
                e0 = hk * 512 + lane * 8
                assert e0 + 7 < D
                loaded.update(range(e0, e0 + 8))
    assert loaded == set(range(D))
    # head tiles: absorbed queries of (slot, tile) and the tile's 16 heads stay in the
    # kMaxSlots x 64-head region; launch index -> (unit, tile group) and the group's
    # TG tiles (TG = 2 when the tiles pair up) cover every (unit, tile) once
    for H in (1, 16, 17, 24, 32, 48, 64):
        ht = -(-H // 16)
        assert ((127 * ht + ht - 1) * 16 + 15) < 128 * 64
        tg = 2 if ht % 2 == 0 else 1
        groups = ht // tg
        for units in (1, 7, 8, 9, 100):
            grid = -(-units // 8) * 8 * groups
            seen = []
            for n in range(grid):
                unit, tgi = (n // (8 * groups)) * 8 + n % 8, (n // 8) % groups
                if unit < units:
                    seen += [(unit, tgi * tg + grp) for grp in range(tg)]
            assert sorted(seen) == [(u, t) for u in range(units) for t in range(ht)]
    DW = D // 4
    for wave in range(4):
        for kk in range(DW // 32):
            for g4 in range(4):
                assert wave * DW + kk * 32 + g4 * 8 + 7 < D
        for n in range(DW // 16):
            assert wave * DW + n * 16 + 15 < D
    # splits per read stay within the per-sequence bound the workspace is sized for,
    # and one read's partials (a split per head tile, up to 4 tiles) fit the
    # launch cap however few sequences the store holds
    for max_blocks in (1, 7, 8, 9, 64, 255, 256, 257, 300, 4096):
        per_seq = min(32, -(-max_blocks // 8))
        for n_seq in (1, 2, 130):
            cap = max(1, min(1024, n_seq * per_seq * 4))
            assert per_seq * 4 <= cap
        for n_read in range(0, max_blocks + 1):
            sp = -(-n_read // _pps_rows(n_read)) if n_read else 0
            assert sp <= per_seq
    # k_merge_rows keeps split weights in a 64-entry array
    assert 32 <= 64


@functools.lru_cache(None)
def plan():
    """The library's own plans, compiled from their headers."""
    here = os.path.dirname(os.path.abspath(__file__))
    out = os.path.join(tempfile.mkdtemp(), "plan.so")
    csrc = os.path.join(here, "..", "paper_2609_32395_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", csrc,
                    os.path.join(here, "native", "plan_c.cpp"), "-o", out], check=True)
    return ctypes.CDLL(out)


def _ints(fn, n, *args):
    o = (ctypes.c_int * n)()
    fn(*args, o)
    return list(o)


def gemm_tile(M, N, K):
    """wide 0, tall 1, pair 2, small 3, brief 4"""
    return plan().lp_gemm_tile(M, N, K)


def lin_chunk(K):
    return 256 * ((K + 256 * 16 - 1) // (256 * 16))


def _some(n):
    """First, last and a few indices between of n."""
    return sorted({0, 1, n // 3, n // 2, n - 2, n - 1} & set(range(n)))


def _walk(T, rt):
    """(row tile, column group) of every launch index of a few-row map: each pair once."""
    seen = [plan().lp_xcd_order(i, T) for i in range(plan().lp_xcd_grid(T))]
    seen = [(p % rt, p // rt) for p in seen if p >= 0]
    assert len(seen) == len(set(seen)) == T
    return seen


class _Map:
    """Largest element index that a linear map's kernel touches in each operand."""

    def __init__(self, M, N, K, ldx, ldy, n2, ns, split):
        self.__dict__.update(M=M, N=N, K=K, ldx=ldx, ldy=ldy, n2=n2, ns=ns, split=split)
        self.hi = {"x": -1, "w": -1, "w2": -1, "y": -1}
        self.done = set()                     # (row, column) of the outputs stored, where asked for

    def x(self, m, k):
        assert 0 <= m < self.M and 0 <= k and k + 7 < self.K
        self.hi["x"] = max(self.hi["x"], m * self.ldx + k + 7)

    def w(self, n, k):
        assert 0 <= n < self.N and 0 <= k and k + 7 < self.K
        key, row = ("w", n) if n < self.n2 else ("w2", n - self.n2)
        self.hi[key] = max(self.hi[key], row * self.K + k + 7)

    def out4(self, m, n):                     # lin_store4: columns n .. n + 3 of row m
        assert n % 4 == 0 and (self.ldy % 4 == 0 or not self.split)
        for e in range(4):
            if m < self.M and n + e < self.N:
                self.done.add((m, n + e))
                if self.split:
                    g, c = divmod(n + e, self.ns)
                    assert g < 3 and c < self.ns
                    self.hi["y"] = max(self.hi["y"], m * self.ns + c)
                else:
                    self.hi["y"] = max(self.hi["y"], m * self.ldy + n + e)


def _few_load(row, k, nt, load):
    """few_load: 8 instructions of two 512-byte rows; the chunks that a short
    last piece does not have are re-reads of its first."""
    for i, lane in itertools.product(range(8), (0, 1, 31, 32, 63)):
        s = lane & 31
        load(row(2 * i + (lane >> 5)), k + (s if s < 4 * nt else 0) * 8)


def _few_finish(o, RT, G, threads, NC, m0, n0, part, lds):
    for q in range(64 * RT * G):              # few_finish, all strides of the workgroup
        row, c0 = q // (4 * G), (q % (4 * G)) * 4
        assert part + (((NC - 1) * 16 * RT + row) * 16 * G + c0) * 4 + 16 <= lds
        if m0 + row < o.M:
            o.out4(m0 + row, n0 + c0)


def _few_range(o):
    """k_linear_few."""
    M, N, K = o.M, o.N, o.K
    RT, G, nw, loop, lds = _ints(plan().lp_few_plan, 5, plan().lp_few_kind(M, N, K), K)
    KS, CS = K // 32, lin_chunk(K) // 32
    NC = -(-KS // CS)
    assert 1 <= nw <= 16 and lds <= 160 * 1024 and (loop or NC <= nw)
    part = nw * 8192
    assert part + NC * RT * G * 1024 <= lds
    # every wave's pieces: chunks w, w + nw, .. in ascending steps, at most 8 at a time
    pieces = []
    for w in range(nw):
        c, st = w, w * CS
        while c < NC:
            nt = min(8, min(KS, (c + 1) * CS) - st)
            assert nt >= 1 and (loop or st == c * CS)
            pieces.append((w, c, st, nt))
            st += 8
            if st >= min(KS, (c + 1) * CS):
                if not loop:
                    break
                c += nw
                st = c * CS
    steps = sorted(s for _, _, st, nt in pieces for s in range(st, st + nt))
    assert steps == list(range(KS))           # each step of K once
    assert all(s // CS == c for _, c, st, nt in pieces for s in range(st, st + nt))
    rt, cg = -(-M // (16 * RT)), -(-N // (16 * G))
    tiles = _walk(rt * cg, rt)
    for r_t, g in {tiles[i] for i in _some(len(tiles))} | {(rt - 1, cg - 1), (0, cg - 1), (rt - 1, 0)}:
        m0, n0 = r_t * 16 * RT, g * 16 * G
        for w, c, st, nt in pieces:
            for i in range(RT):
                _few_load(lambda r: min(m0 + i * 16 + r, M - 1), st * 32, nt, o.x)
            for j in range(G):
                _few_load(lambda r: min(n0 + j * 16 + r, N - 1), st * 32, nt, o.w)
            for i, j, lane in itertools.product(range(RT), range(G), (0, 15, 16, 63)):
                at = part + (((c * RT + i) * 16 + (lane & 15)) * 16 * G + j * 16 + 4 * (lane >> 4)) * 4
                assert at % 16 == 0 and at + 16 <= lds
        _few_finish(o, RT, G, 64 * nw, NC, m0, n0, part, lds)
        assert all((m, n) in o.done for m in range(m0, min(m0 + 16 * RT, M)) for n in range(n0, min(n0 + 16 * G, N)))


def _wide_range(o):
    """k_linear_wide: x rows once into LDS, two column tiles per wave."""
    M, N, K = o.M, o.N, o.K
    RT, XP, n_tiles = -(-M // 16), K + 8, -(-N // 16)
    assert plan().lp_wide_lds(RT, K) == RT * 16 * XP * 2 <= 160 * 1024
    for q in range(RT * 16 * (K // 8)):
        r, c8 = q // (K // 8), q % (K // 8)
        assert r * XP + c8 * 8 + 8 <= RT * 16 * XP
        if r < M:
            o.x(r, c8 * 8)
    tiles = set()
    for blk, wave in itertools.product(range(-(-n_tiles // 16)), range(8)):
        t0 = (blk * 8 + wave) * 2
        if t0 >= n_tiles:
            continue
        for t in {t0, t0 + 1 if t0 + 1 < n_tiles else t0}:
            tiles.add(t)
            if t in (0, n_tiles - 1):
                for lane in (0, 15, 16, 63):
                    n = min(t * 16 + (lane & 15), N - 1)
                    for c, u in itertools.product((0, K // 256 - 1), (0, 7)):
                        o.w(n, (lane >> 4) * 8 + c * 256 + u * 32)
                    for i in range(RT):
                        if i * 16 + (lane & 15) < M:
                            o.out4(i * 16 + (lane & 15), t * 16 + 4 * (lane >> 4))
    assert tiles == set(range(n_tiles))


def _gemm_range(o):
    """k_gemm on the tile the host picks."""
    M, N, K = o.M, o.N, o.K
    tile = gemm_tile(M, N, K)
    BM, BN, BK, NS, NW, WM, WN, IA, IB, RPI, CPR, STAGE, PER = _ints(plan().lp_gemm_cfg, 13, tile)
    assert NS * STAGE * 2 <= 160 * 1024 // PER and K % BK == 0
    tm_, tn_ = -(-M // BM), -(-N // BN)
    T = tm_ * tn_
    grid = plan().lp_gemm_grid(PER, T)
    seen = []
    for wg in range(grid):                    # a workgroup that fills its CU takes tile after tile
        i = wg
        while True:
            p = plan().lp_gemm_place(i, tm_, tn_)
            if p < 0:
                break
            seen.append(p)
            if PER != 1:
                break
            i += grid
    assert sorted(seen) == list(range(T))     # every tile once
    assert grid % 8 == 0                      # so a workgroup's tiles are its XCD's
    for p in {seen[i] for i in _some(T)} | {T - 1, tn_ - 1}:
        m0, n0 = p // tn_ * BM, p % tn_ * BN
        for wave, lane in itertools.product(range(NW), (0, 7, 8, 63)):
            for op, n, lim in ((o.x, IA, (m0, M)), (o.w, IB, (n0, N))):
                for i in range(n):
                    r = (wave * n + i) * RPI + lane // CPR
                    c = (lane % CPR) ^ plan().lp_gemm_swz(tile, r)
                    for kt in {0, K // BK - 1}:
                        op(min(lim[0] + r, lim[1] - 1), c * 8 + kt * BK)
        o.done = set()
        for wave, lane in itertools.product(range(NW), range(64)):
            wm, wn = wave % (BM // WM), wave // (BM // WM)
            for i, j in itertools.product(range(WM // 16), range(WN // 16)):
                m = m0 + wm * WM + i * 16 + (lane & 15)
                if m < M:
                    o.out4(m, n0 + wn * WN + j * 16 + 4 * (lane >> 4))
        assert len(o.done) == (min(m0 + BM, M) - m0) * (min(n0 + BN, N) - n0)


def _linear_ranges(M, N, K, ldx, ldy, n2, ns, split, f32):
    """Operand ranges of the kernel that the host picks for a map without LayerNorm."""
    o = _Map(M, N, K, ldx, ldy, n2, ns, split)
    if f32 and plan().lp_wide_fits(M, N, K):
        _wide_range(o)
    elif M <= 128:
        _few_range(o)
    else:
        _gemm_range(o)
    return o.hi


@pytest.mark.parametrize("d,vocab,rows", [(128, 256, 448), (768, 1000, 130), (2048, 77, 64), (256, 300, 100),
                                         (768, 50257, 64), (1024, 4000, 4096), (832, 300, 256), (2048, 300, 256),
                                         (2048, 50257, 520), (2048, 50257, 136), (2048, 50257, 1), (832, 1000, 200),
                                         (1024, 9001, 17), (1088, 12001, 48), (1984, 12001, 128), (64, 8192, 33),
                                         (1216, 9000, 1300), (2048, 50257, 32)])
def test_model_kernel_indexing(d, vocab, rows):
    """Every linear-map launch the model makes stays inside its operands (x
    [rows, K] in a [max_tokens, ldx] buffer, W [N or n2, K] and [N - n2, K],
    y [rows, ldy]); LayerNorm and embedding lanes stay inside a d-wide row."""
    calls = [  # M, N, K, ldx, ldy, n2, ns, split, rows of W (first, second), fp32
        (rows, 3 * d, d, d, d, 3 * d, d, True, 3 * d, 0, False),        # qkv, split into q, k, v
        (rows, d, d, d, d, d, 0, False, d, 0, False),                   # attention out (+ residual)
        (rows, 4 * d, d, d, 4 * d, 4 * d, 0, False, 4 * d, 0, False),   # ffn up
        (rows, d, 4 * d, 4 * d, d, d, 0, False, d, 0, False),           # ffn down (+ residual)
        (rows, 2 * d, d, d, d, d, d, True, d, d, False),                # memory K | V maps
        (1, 2 * d, d, d, 2 * d, d, 0, False, d, d, False),              # null row through K | V
        (rows, vocab, d, d, vocab, vocab, 0, False, vocab, 0, True),    # output head (fp32)
    ]
    for M, N, K, ldx, ldy, n2, ns, split, wrows, w2rows, f32 in calls:
        assert K % 64 == 0 and K <= ldx
        hi = _linear_ranges(M, N, K, ldx, ldy, n2, ns, split, f32)
        assert hi["x"] < M * ldx
        assert hi["w"] < wrows * K
        assert hi["w2"] < max(w2rows, 0) * K or hi["w2"] == -1
        assert hi["y"] < (M * ns if split else M * ldy)
    # embedding: lane chunks c = i*512 + 8*lane (i < 4) guarded by c < d, 8 values each
    assert d % 8 == 0 and d <= 2048
    for i, lane in itertools.product(range(4), range(64)):
        c = i * 512 + lane * 8
        if c < d:
            assert c + 7 < d
    assert 3 * 512 + 63 * 8 + 8 >= 2048         # the four chunks cover d = 2048


def test_few_row_launches_fit():
    """Every few-row launch, whatever its size: LDS within a CU's 160 KB,
    threads within the kernels' launch bounds, and a wave per chunk unless the
    waves loop."""
    kinds, ln_kinds = set(), set()
    for M, N, K in itertools.product((1, 16, 17, 48, 64, 100, 128), (4, 64, 516, 1024, 3072, 4096, 8200, 20000, 50257),
                                     list(range(64, 2049, 64)) + [2112, 3008, 4096, 4160, 6144, 8192, 16384]):
        k = plan().lp_few_kind(M, N, K)
        RT, G, nw, loop, lds = _ints(plan().lp_few_plan, 5, k, K)
        NC = -(-K // lin_chunk(K))
        assert lds == nw * 8192 + NC * RT * G * 1024 <= 160 * 1024 and (loop or nw == NC)
        assert loop or lin_chunk(K) == 256        # one piece of 8 steps holds a whole chunk
        assert nw <= (16 if k in (3, 4) else 8)   # the kernels' launch bounds
        kinds.add(k)
        if K > 2048:
            continue
        k = plan().lp_few_ln_kind(M, N, K)
        RT, G, wpc, u, threads, lds = _ints(plan().lp_few_ln_plan, 6, k, K)
        assert threads == 64 * NC * max(1, wpc) <= 512 and lds <= 160 * 1024 and lin_chunk(K) == 256 and NC <= 8
        assert wpc in (0, 1, 2) and (wpc == 0 or (RT == 1 and G % wpc == 0))
        ln_kinds.add(k)
    assert kinds == set(range(7)) and ln_kinds == set(range(8))   # every tile is reached


# us of a map, measured on an MI355X with the weights out of the caches.
# Without LayerNorm (K <= 2048) on 1x1, 2x2 and 2x4 tiles:
FEW_MEASURED = {
    (64, 1024, 1024): (4.1, 6.0, 8.8), (64, 2048, 2048): (6.7, 7.8, 11.4), (64, 50256, 2048): (98.7, 86.0, 79.8),
    (32, 8192, 64): (3.6, 4.7, 6.8), (32, 8192, 256): (4.4, 5.6, 7.6), (128, 2048, 256): (3.7, 4.8, 7.1),
    (128, 8192, 512): (9.5, 8.2, 9.3), (128, 50256, 1024): (84.1, 50.2, 58.1), (48, 12000, 1088): (14.6, 17.2, 19.7),
    (16, 12000, 1984): (13.5, 17.4, 15.8), (64, 3072, 1536): (7.7, 7.3, 10.2), (128, 8192, 320): (9.4, 7.8, 9.0),
    (128, 4096, 1088): (11.9, 11.2, 10.1), (96, 3072, 1088): (8.4, 10.9, 9.7), (96, 6144, 2048): (20.8, 21.0, 23.2)}
# with it, by kind:
FEW_LN_MEASURED = {
    (64, 512, 64): {0: 4.7, 1: 5.4, 2: 6.8, 3: 4.4, 4: 5.2, 5: 4.0, 6: 4.2, 7: 7.2},
    (128, 4096, 64): {0: 6.9, 1: 6.5, 2: 7.5, 3: 5.8, 4: 6.7, 5: 7.2, 6: 5.4, 7: 7.3},
    (64, 3072, 256): {0: 5.1, 1: 5.6, 2: 6.7, 3: 4.9, 4: 5.1, 5: 5.4, 6: 5.4, 7: 8.7},
    (32, 4096, 512): {0: 6.3, 1: 6.0, 2: 7.2, 3: 5.0, 4: 5.8, 5: 7.1, 6: 5.8, 7: 9.3},
    (128, 8192, 512): {0: 17.1, 1: 14.5, 2: 11.2, 3: 12.0, 4: 10.8, 5: 20.9, 6: 17.2, 7: 12.8},
    (64, 1024, 1024): {0: 5.6, 1: 6.3, 2: 7.9, 3: 5.7, 4: 7.3, 5: 6.5, 6: 7.3, 7: 11.6},
    (64, 2048, 768): {0: 6.7, 1: 6.2, 2: 7.9, 3: 5.6, 4: 7.0, 5: 7.9, 6: 6.4, 7: 10.6},
    (64, 4096, 1024): {0: 10.2, 1: 8.5, 2: 8.3, 3: 8.1, 4: 7.7, 5: 12.6, 6: 10.2, 7: 11.6},
    (128, 3072, 768): {0: 11.8, 1: 10.6, 2: 10.7, 3: 9.9, 4: 11.7, 5: 14.3, 6: 11.3, 7: 10.6},
    (128, 4096, 1024): {0: 16.4, 1: 13.4, 2: 11.0, 3: 12.6, 4: 13.0, 5: 20.7, 6: 15.4, 7: 11.8},
    (1, 50256, 768): {0: 22.7, 1: 21.3, 2: 21.6, 3: 22.2, 4: 25.5, 5: 23.8, 6: 19.4, 7: 24.3},
    (16, 2048, 2048): {0: 7.1, 1: 8.7, 2: 11.7, 5: 9.4, 6: 10.9, 7: 16.2},
    (64, 2048, 1088): {0: 11.3, 1: 8.5, 2: 10.4, 5: 13.3, 6: 8.9, 7: 13.8},
    (16, 12000, 1536): {0: 17.4, 1: 17.6, 2: 14.2, 5: 24.1, 6: 19.4, 7: 17.6},
    (64, 3072, 2048): {0: 17.0, 1: 15.8, 2: 11.8, 5: 23.4, 6: 19.5, 7: 17.5},
    (64, 8192, 2048): {0: 40.9, 1: 33.2, 2: 25.2, 5: 59.1, 6: 37.7, 7: 21.0},
    (17, 12000, 1088): {0: 28.2, 1: 22.1, 2: 20.3, 5: 35.1, 6: 22.7, 7: 15.0}}


@pytest.mark.parametrize("shape", FEW_MEASURED, ids=str)
def test_few_row_rule_picks_a_fast_tile(shape):
    us = FEW_MEASURED[shape]
    kind = plan().lp_few_kind(*shape)
    assert us[kind] <= 1.1 * min(us), (kind, us)


@pytest.mark.parametrize("shape", FEW_LN_MEASURED, ids=str)
def test_few_row_layernorm_rule_picks_a_fast_tile(shape):
    us = FEW_LN_MEASURED[shape]
    kind = plan().lp_few_ln_kind(*shape)
    assert us[kind] <= 1.1 * min(us.values()), (kind, us)


# us of a map on the wide, tall, pair, small and brief tiles, measured on an
# MI355X: short and long reductions, one round of tiles and many, rows and
# columns that fill the tiles and not.
GEMM_MEASURED = {
    (320, 8192, 320): (10.5, 7.5, 7.9, 7.5, 6.5), (640, 2048, 512): (13.5, 9.3, 10.7, 6.8, 7.5),
    (4096, 768, 320): (10.5, 7.8, 8.1, 7.6, 6.6), (2048, 3072, 256): (11.5, 12.8, 10.9, 11.8, 10.8),
    (1024, 3072, 768): (16.2, 11.3, 12.8, 12.6, 10.7), (1300, 3072, 768): (17.8, 21.2, 18.6, 15.9, 13.8),
    (4096, 3072, 768): (31.2, 29.2, 28.3, 37.3, 34.0), (8192, 2304, 768): (47.1, 45.0, 43.1, 54.0, 49.8),
    (320, 12001, 1024): (26.8, 31.4, 29.5, 22.0, 22.5), (200, 12001, 1024): (25.3, 17.9, 20.1, 18.3, 18.5),
    (1024, 1024, 4096): (48.6, 32.0, 44.4, 19.9, 30.8), (8192, 1024, 4096): (63.0, 77.3, 70.5, 101.1, 96.0),
    (1280, 4096, 2048): (29.7, 36.8, 33.6, 35.8, 37.8), (640, 8192, 4096): (58.2, 73.2, 66.0, 78.4, 98.2),
    (2048, 2048, 2048): (28.9, 21.6, 26.3, 27.6, 26.4), (8192, 8192, 2048): (283.2, 339.5, 309.5, 436.9, 415.9),
    (1536, 8192, 1024): (35.8, 36.2, 33.6, 45.1, 43.3), (6144, 512, 768): (15.6, 11.1, 12.6, 12.2, 10.3)}


@pytest.mark.parametrize("shape", GEMM_MEASURED, ids=str)
def test_gemm_tile_rule_picks_a_fast_tile(shape):
    """The tile that the price table gives is within 5% of the fastest one
    measured (two runs of one tile differ by up to 3%)."""
    us = GEMM_MEASURED[shape]
    assert us[gemm_tile(*shape)] <= 1.05 * min(us), (gemm_tile(*shape), us)


@pytest.mark.parametrize("tile", range(5), ids=["wide", "tall", "pair", "small", "brief"])
def test_gemm_stage_layout(tile):
    """k_gemm's stage in LDS: the DMA instructions of the waves write every
    16-byte slot of it once, from inside the tile's rows, and each operand
    read (one lane address per operand, the second 32-wide step's slots those
    of the first with bit 2 flipped, tiles of 16 rows at fixed offsets) finds
    the chunk of its row and step."""
    BM, BN, BK, NS, NW, WM, WN, IA, IB, RPI, CPR, STAGE, PER = _ints(plan().lp_gemm_cfg, 13, tile)
    WAVES_M = BM // WM
    assert BK == 64 and NS * STAGE * 2 * PER <= 160 * 1024 and IA * RPI * NW == BM and IB * RPI * NW == BN
    swz = lambda r: plan().lp_gemm_swz(tile, r)
    slots = {}                                     # element offset of a 16-byte slot -> (operand, row, chunk)
    for wave, lane in itertools.product(range(NW), range(64)):
        for op, n, base in (("x", IA, 0), ("w", IB, BM * BK)):
            for i in range(n):
                r = (wave * n + i) * RPI + lane // CPR
                dst = base + (wave * n + i) * 512 + lane * 8
                assert dst not in slots and dst + 8 <= STAGE and r < (BM if op == "x" else BN)
                slots[dst] = (op, r, (lane % CPR) ^ swz(r))
    assert len(slots) == STAGE // 8
    for wave, lane, ks in itertools.product(range(NW), range(64), range(2)):
        wm, wn = wave % WAVES_M, wave // WAVES_M
        l16, g = lane & 15, lane >> 4
        sl = ((g ^ swz(l16)) << 3) ^ (ks << 5)
        for i in range(WM // 16):
            assert slots[(wm * WM + l16) * BK + sl + i * 16 * BK] == ("x", wm * WM + i * 16 + l16, ks * 4 + g)
        for j in range(WN // 16):
            assert slots[BM * BK + (wn * WN + l16) * BK + sl + j * 16 * BK] == ("w", wn * WN + j * 16 + l16, ks * 4 + g)


def test_few_row_tile_layout():
    """The few-row maps' 16-row piece in a wave's LDS tile: the 8 loads'
    writes fill 8 KB once, operand reads of step t find chunk 4 t + l / 16 of
    row l % 16, and the 16 rows of one read lie in 16 different 16-byte
    columns of the banks."""
    put, get = plan().lp_few_put, plan().lp_few_get
    at = {}
    for i, lane in itertools.product(range(8), range(64)):
        r, s = 2 * i + (lane >> 5), lane & 31
        assert 0 <= put(r, s) and put(r, s) + 16 <= 8192 and put(r, s) not in at
        at[put(r, s)] = (r, s)
    for t, lane in itertools.product(range(8), range(64)):
        assert at[get(lane, t)] == (lane & 15, 4 * t + (lane >> 4))
    for t, g in itertools.product(range(8), range(4)):
        assert len({(get(g * 16 + r, t) >> 4) & 15 for r in range(16)}) == 16


@pytest.mark.parametrize("R", [4, 8])
def test_layernorm_tree_is_one_order(R):
    """The statistics' tree over a chunk's 32 pieces adds in one order in its
    three forms: a piece per lane, R rows at once, and pieces 4 t + g in the
    registers of MFMA-operand lanes.  A sum is written as a nested pair whose
    members are unordered (an addition commutes bit for bit)."""
    add = lambda x, y: frozenset((x, y)) if x != y else (x, y)
    lanes = range(32)
    partner = {16: lambda s: s ^ 16, 8: lambda s: s ^ 8, 7: lambda s: s ^ 7, 3: lambda s: s ^ 3, 1: lambda s: s ^ 1}
    x = {s: ("p", s) for s in lanes}
    for k in (16, 8, 7, 3, 1):
        x = {s: add(x[s], x[partner[k](s)]) for s in lanes}
    assert len(set(x.values())) == 1
    want = x[0]
    # R rows: level 16 leaves lane s rows of its bit 4, level 8 of bit 3, level 7 (R = 8) of bit 2
    row = lambda r, s: ("p", s) if r is None else (r, s)
    t = [{s: row(r, s) for s in lanes} for r in range(R)]
    u = [{s: add(t[i + (R // 2 if s & 16 else 0)][s], t[i + (R // 2 if s & 16 else 0)][s ^ 16]) for s in lanes}
         for i in range(R // 2)]
    v = [{s: add(u[i + (R // 4 if s & 8 else 0)][s], u[i + (R // 4 if s & 8 else 0)][s ^ 8]) for s in lanes}
         for i in range(R // 4)]
    y = {s: add(v[1 if R == 8 and s & 4 else 0][s], v[1 if R == 8 and s & 4 else 0][s ^ 7]) for s in lanes}
    for k in (3, 1):
        y = {s: add(y[s], y[partner[k](s)]) for s in lanes}
    name = lambda tree, r: (frozenset if isinstance(tree, frozenset) else tuple)(
        name(c, r) for c in tree) if isinstance(tree, frozenset) or isinstance(tree[0], (tuple, frozenset)) else (r, tree[1])
    for s in lanes:
        assert y[s] == name(want, (s >> 2) // (8 // R))
    # operand lanes: group g holds pieces 4 t + g
    o = {}
    for g in range(4):
        p = [("p", 4 * t_ + g) for t_ in range(8)]
        o[g] = (add(add(p[0], p[4]), add(p[2], p[6])), add(add(p[1], p[5]), add(p[3], p[7])))
    v1 = {g: add(o[g][0], o[g ^ 3][1]) for g in range(4)}
    z = {g: add(v1[g], v1[g ^ 3]) for g in range(4)}
    assert {add(z[g], z[g ^ 1]) for g in range(4)} == {want}


def _ln_rows_pieces(d, rows):
    """k_ln_rows: the 8-value pieces of a row by (chunk, piece), from the lanes
    that load them (a wave per row, a half-wave per chunk of 256, up to four
    chunks per half-wave); every load and store inside the row."""
    NC = (d + 255) // 256
    assert NC <= 8
    seen = {}
    for blk, tid in itertools.product(range(-(-rows // 4)), range(256)):
        lane, row = tid & 63, blk * 4 + (tid >> 6)
        if row >= rows:
            continue
        half = lane >> 5
        k0 = half * 256 + (lane & 31) * 8
        for i in range(4):
            if k0 + 512 * i < d:
                assert k0 + 512 * i + 7 < d
                # register i of half-wave h holds chunk 2 i + h, which the total takes from lane 32 h
                seen.setdefault(row, {})[(2 * i + half, lane & 31)] = k0 + 512 * i
    assert sorted(seen) == list(range(rows)) and all(v == seen[0] for v in seen.values())
    assert all(c < NC for c, _ in seen[0])     # totals are taken of chunks below NC only
    return seen[0]


def _few_ln_pieces(M, N, K, kind):
    """k_linear_few_ln: the same pieces as its waves load them, with every load
    inside the operands and every LDS access inside its region."""
    RT, G, WPC, _, threads, lds = _ints(plan().lp_few_ln_plan, 6, kind, K)
    KS = K // 32
    NC = (KS + 7) // 8
    GW, RI = G // WPC, 8 // WPC
    tiles, st0 = NC * WPC * 8192, NC * WPC * 8192
    st1 = st0 + 512
    part = st1 + 512
    assert part + NC * G * 1024 <= lds and threads == 64 * NC * WPC
    zeroed = {e for e in range(NC * 16, 128)}  # statistics past the last chunk
    o = _Map(M, N, K, K, N, N, 0, False)
    rt, cg = -(-M // 16), -(-N // (16 * G))
    walk = _walk(rt * cg, rt)
    pieces, pub = {}, {}
    for r_t, g in {walk[i] for i in _some(len(walk))} | {(rt - 1, cg - 1)}:
        m0, n0 = r_t * 16, g * 16 * G
        for w in range(NC * WPC):
            c, h = w // WPC, w % WPC
            nt, k0 = min(8, KS - 8 * c), c * 256
            assert nt >= 1
            rows_put = set()
            for lane in range(64):
                half, s = lane >> 5, lane & 31
                in_ = s < 4 * nt
                q = s if in_ else 0
                assert k0 + q * 8 + 7 < K             # gain and bias
                for i in range(RI):
                    r = h * 2 * RI + 2 * i + half
                    assert r < 16
                    o.x(min(m0 + r, M - 1), k0 + q * 8)
                    if in_ and m0 + r < M:
                        pieces.setdefault((c, s), set()).add(k0 + q * 8)
                    at = c * WPC * 8192 + plan().lp_few_put(r, s)
                    assert at + 16 <= tiles and at not in rows_put
                    rows_put.add(at)
                tr = h * 2 * RI + 2 * ((s >> 2) // (8 // RI)) + half
                if s & 3 == 0:                        # publishes row tr: the tree's row for these lanes
                    assert tr < 16 and c * 16 + tr < 128
                    pub.setdefault((c, tr), set()).add(h)
            for j in range(GW):
                _few_load(lambda r: min(n0 + (h * GW + j) * 16 + r, N - 1), k0, nt, o.w)
                for lane in (0, 15, 16, 63):
                    at = part + ((c * 16 + (lane & 15)) * 16 * G + (h * GW + j) * 16 + 4 * (lane >> 4)) * 4
                    assert at % 16 == 0 and at + 16 <= part + NC * G * 1024
            assert w * 8192 + 8192 <= tiles           # the wave's own tile
        _few_finish(o, 1, G, threads, NC, m0, n0, part, lds)
    assert set(pub) == {(c, r) for c in range(NC) for r in range(16)} and all(len(v) == 1 for v in pub.values())
    assert {c * 16 + r for c, r in pub} | zeroed == set(range(128))
    assert o.hi["x"] < M * K and o.hi["w"] < N * K and o.hi["y"] < M * N
    return {k: next(iter(v)) for k, v in pieces.items() if len(v) == 1}


def _skinny_ln_pieces(M, N, K, kind):
    """k_linear_skinny_ln: the pieces as wave c, lane group g = lane / 16 hold
    them (piece 4 t + g of step t), loads and LDS regions inside their bounds."""
    RT, G, _, U, threads, lds = _ints(plan().lp_few_ln_plan, 6, kind, K)
    KS = K // 32
    NC = (KS + 7) // 8
    assert threads == 64 * NC <= 512 and U <= 8
    st0 = 4 * K
    st1 = st0 + NC * 16 * RT * 4
    assert st0 % 16 == 0 and st1 + NC * 16 * RT * 4 <= lds and NC * 256 * RT * G * 4 <= lds
    for tid in range(threads):                # gain and bias staging
        if tid * 8 < K:
            assert 2 * (K + tid * 8 + 7) < st0
    assert 8 * threads >= K
    o = _Map(M, N, K, K, N, N, 0, False)
    rt, cg = -(-M // (16 * RT)), -(-N // (16 * G))
    walk = _walk(rt * cg, rt)
    pieces = {}
    for r_t, g in {walk[i] for i in _some(len(walk))} | {(rt - 1, cg - 1)}:
        m0, n0 = r_t * 16 * RT, g * 16 * G
        for c, lane in itertools.product(range(NC), (0, 15, 16, 32, 48, 63)):
            s0, ns, kofs = 8 * c, min(8, KS - 8 * c), (lane >> 4) * 8
            assert ns >= 1
            for t in range(8):
                k = (s0 + min(t, ns - 1)) * 32 + kofs
                for i in range(RT):
                    o.x(min(m0 + i * 16 + (lane & 15), M - 1), k)
                for j in range(G):
                    o.w(min(n0 + j * 16 + (lane & 15), N - 1), k)
                if t < ns:
                    pieces[(c, 4 * t + (lane >> 4))] = k
            for i in range(RT):
                assert c * 16 * RT + i * 16 + (lane & 15) < NC * 16 * RT
        _few_finish(o, RT, G, threads, NC, m0, n0, 0, lds)
    assert o.hi["x"] < M * K and o.hi["w"] < N * K and o.hi["y"] < M * N
    return pieces


@pytest.mark.parametrize("M,N,K", [(64, 3072, 1024), (64, 6144, 2048), (64, 8192, 2048), (64, 1024, 1024),
                                   (128, 3072, 768), (1, 4096, 1024), (33, 4160, 832), (64, 2048, 128),
                                   (64, 2496, 832), (64, 3328, 832), (64, 832, 832), (16, 6144, 2048),
                                   (16, 8192, 2048), (1, 36, 64), (128, 4096, 64), (15, 100, 320), (128, 8192, 512),
                                   (128, 4096, 1024), (17, 2048, 1088), (70, 6148, 1984), (9, 20000, 1984), (7, 30000, 768)])
def test_layernorm_fused_indexing_and_order(M, N, K):
    """The LayerNorm fused into a few-row map and the stand-alone kernel cut
    every row into the same (chunk, piece) values, covering it once (the tree
    that adds the pieces is one order in all of them:
    test_layernorm_tree_is_one_order); loads, LDS regions and stores of the
    kernel that the host picks stay inside their buffers."""
    want = _ln_rows_pieces(K, 5)
    assert sorted(k + e for k in want.values() for e in range(8)) == list(range(K))
    assert all(k == c * 256 + p * 8 for (c, p), k in want.items())
    kind = plan().lp_few_ln_kind(M, N, K)
    wpc = _ints(plan().lp_few_ln_plan, 6, kind, K)[2]
    got = _few_ln_pieces(M, N, K, kind) if wpc else _skinny_ln_pieces(M, N, K, kind)
    assert got == want


def test_layernorm_rstd_is_correctly_rounded():
    """The LayerNorm's statistics use no approximate reciprocal or square-root
    instruction: rstd is a correctly rounded square root and division."""
    src = open(os.path.join(os.path.dirname(__file__), "..", "paper_2609_32395_amd", "csrc", "linear.h")).read()
    body = src[src.index("void ln_unpack("):src.index("inline void launch_ln(")]
    assert "1.f / sqrtf(" in body and "rsqf" not in body and "rcpf" not in body


def test_gelu_erf_formula_in_source():
    """The erf of the GELU epilogue (Abramowitz & Stegun 7.1.26), evaluated
    with the constants read from linear.h, stays within the published bound
    1.5e-7 of math.erf in float64, and within 1e-6 in float32 arithmetic (a
    few float32 ulps of 1 on top; bf16 activations carry 2^-9)."""
    import math
    import re
    import numpy as np
    src = open(os.path.join(os.path.dirname(__file__), "..", "paper_2609_32395_amd", "csrc", "linear.h")).read()
    body = src[src.index("float erf_as("):src.index("float gelu_erf(")]
    p = float(re.search(r"1\.f \+ ([0-9.]+)f \* ax", body).group(1))
    a5, a4, a3, a2, a1 = (float(x) for x in re.search(
        r"\(\(\(\(([0-9.]+)f \* t - ([0-9.]+)f\) \* t \+ ([0-9.]+)f\) \* t - ([0-9.]+)f\) \* t \+ ([0-9.]+)f\)",
        body).groups())
    a4, a2 = -a4, -a2
    x = np.linspace(-6, 6, 200001)
    for dt, bound in ((np.float64, 1.5e-7), (np.float32, 1e-6)):
        xs = x.astype(dt)
        ax = np.abs(xs)
        t = (1 / (1 + dt(p) * ax)).astype(dt)
        poly = ((((dt(a5) * t + dt(a4)) * t + dt(a3)) * t + dt(a2)) * t + dt(a1)) * t
        y = np.copysign(1 - poly * np.exp2(-ax * ax * dt(1.4426950408889634)), xs)
        ref = np.array([math.erf(float(v)) for v in xs[::50]])
        assert np.max(np.abs(y[::50] - ref)) <= bound, dt


def _tile_reads_find(dh, src):
    """The score and value operand reads of a 64-key tile whose 16-byte slots
    (LDS byte -> byte of the (page, head) tile) are `src`: a score row is the key
    that the causal mask takes it for, and a lane's 8 value slots are the keys of
    its weights of score tiles 2c and 2c + 1."""
    _, KB, KRB, _, _ = _ints(plan().ap_ring, 5, dh)
    key_of = lambda kt, i, lane: plan().ap_score_key(kt, i) + 8 * (lane >> 4)
    for lane in range(64):
        g, l16 = lane >> 4, lane & 15
        for kt, kk in itertools.product(range(4), range(dh // 32)):   # score operand: row kt*16 + l16, chunk kk*4 + g
            row, c = kt * 16 + l16, kk * 4 + g
            key, chunk = divmod(src[plan().ap_key_at(dh, row, c)], KRB)
            assert chunk == c * 16 and key < 64
            # row 4 g' + i of score tile kt comes out in lane group g', value i
            assert key == key_of(kt, l16 % 4, (l16 // 4) * 16)
        for dt, c in itertools.product(range(dh // 16), range(2)):
            d, first = divmod(src[plan().ap_operand_at(dh, lane, dt, c)] - KB, 128)
            assert d == dt * 16 + l16
            assert [first // 2 + j for j in range(8)] == [key_of(2 * c + j // 4, j % 4, lane) for j in range(8)]


@pytest.mark.parametrize("dh", [32, 64, 128])
def test_attention_tile_key_order(dh):
    """The DMA's key rows are the keys that the in-block writer puts there: LDS
    row tile_row(k) holds key k, and the rows are a permutation."""
    KRB = 2 * dh
    assert sorted(plan().ap_tile_row(k) for k in range(64)) == list(range(64))
    for k, c in itertools.product(range(64), range(dh // 8)):
        assert plan().ap_source(dh, plan().ap_key_at(dh, plan().ap_tile_row(k), c)) == k * KRB + c * 16


@pytest.mark.parametrize("dh,ns", [(32, 4), (64, 4), (128, 2)])
def test_prefill_page_ring_indexing(dh, ns):
    """Non-rotary prefill's DMA page ring: every lane's source byte lies in
    its (page, head) tile, every LDS byte of a stage is written exactly once,
    and each operand read finds the chunk the DMA put there."""
    TILE, KB, KRB, NS, IPW = _ints(plan().ap_ring, 5, dh)
    assert (TILE, KB, KRB, NS) == (256 * dh, 128 * dh, 2 * dh, ns) and 4 * IPW * 1024 == TILE
    placed = {}                                   # LDS byte offset in the stage -> source byte offset
    for wave, i, lane in itertools.product(range(4), range(IPW), range(64)):
        byte = (wave * IPW + i) * 1024 + lane * 16
        assert byte not in placed
        placed[byte] = plan().ap_source(dh, byte)
    assert sorted(placed) == list(range(0, TILE, 16)) and sorted(placed.values()) == list(range(0, TILE, 16))
    assert NS * TILE <= 64 * 1024 and 3 * IPW < 64
    _tile_reads_find(dh, placed)
    # (the swizzles' bank behaviour is a measured property of the hardware: a
    # one-wave probe of these reads shows no conflicts; the model of 64
    # 4-byte banks that first chose them does not describe gfx950's LDS)


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("threads", [256, 512])
def test_in_block_tile_writes(dh, threads):
    """A block's own keys and values in LDS (the encoder, the final split): key
    chunks and 32-bit value pairs fill the tile once each, and the operand reads
    find there what they would find in a page."""
    TILE, KB, KRB, _, _ = _ints(plan().ap_ring, 5, dh)
    CPR = dh // 8
    NK, NJ = 64 * CPR, 64 * CPR + 32 * CPR
    half = {}                                     # 2-byte LDS place -> byte of the tile in memory
    for tid in range(threads):
        for j in range(tid, NJ, threads):
            if j < NK:
                row, c8 = j // CPR, j % CPR
                at = plan().ap_key_at(dh, plan().ap_tile_row(row), c8)
                put = [(at + 2 * e, row * KRB + c8 * 16 + 2 * e) for e in range(8)]
                assert at % 16 == 0 and at + 16 <= KB
            else:
                key, c8 = 2 * ((j - NK) // CPR), (j - NK) % CPR
                put = []
                for d in range(c8 * 8, c8 * 8 + 8):
                    at = plan().ap_value_at(dh, d, key)
                    assert at % 4 == 0 and KB <= at and at + 4 <= TILE
                    put += [(at + 2 * e, KB + d * 128 + (key + e) * 2) for e in range(2)]
            for at, what in put:
                assert at not in half
                half[at] = what
    assert len(half) == TILE // 2
    slots = {at: half[at] for at in range(0, TILE, 16)}
    assert all(half[at + 2 * e] == slots[at] + 2 * e for at in slots for e in range(8))
    _tile_reads_find(dh, slots)


@pytest.mark.parametrize("all_", [512, 518, 600, 1200, 4095, 4096])
def test_encoder_tile_ranges(all_):
    """xcd_range: a permutation of the tiles in which each XCD (workgroup index
    mod 8) has one contiguous range."""
    got = [plan().ap_xcd_range(n, all_) for n in range(all_)]
    assert sorted(got) == list(range(all_))
    for x in range(8):
        mine = got[x::8]
        assert mine == list(range(mine[0], mine[0] + len(mine)))


@pytest.mark.parametrize("b,dh,es", SHAPES)
def test_export_indexing_and_transpose(b, dh, es):
    """k_export: 16-byte chunks of the key plane and of the output rows stay in
    their buffers; the value plane's LDS slots (chunk rc of row d at
    rc ^ ((d / E) mod (b / E))) are a permutation of each row, and the gather
    of output chunk (r, cc) reads exactly value (d = cc*E + j, r) for j < E."""
    E = 16 // es
    CR, CB = dh // E, b // E
    for H, n_pages, n_live in [(1, 1, 1), (16, 4096, 4096), (4, 9, 5)]:
        pool = n_pages * H * 2 * b * dh
        base = page_head_offset(n_pages - 1, H - 1, H, b, dh)
        assert base + b * dh + (dh - 1) * b + (CB - 1) * E + E - 1 < pool          # value plane chunk reads
        assert base + (b - 1) * dh + (CR - 1) * E + E - 1 < pool                    # key plane chunk reads
        out = n_live * b * H * dh
        assert ((n_live - 1) * b * H + H - 1) * dh + (b - 1) * H * dh + (CR - 1) * E + E - 1 < out
    tile = {}
    for d in range(dh):
        for rc in range(CB):
            slot = rc ^ ((d // E) % CB)
            assert 0 <= slot < CB
            for e in range(E):
                pos = d * b + slot * E + e
                assert pos < dh * b and pos not in tile
                tile[pos] = (d, rc * E + e)
    assert len(tile) == dh * b
    for r in range(b):
        for cc in range(CR):
            off = ((r // E) ^ (cc % CB)) * E + r % E
            assert [tile[(cc * E + j) * b + off] for j in range(E)] == [(cc * E + j, r) for j in range(E)]


@pytest.mark.parametrize("dh,qw", [(32, 1), (32, 2), (64, 1), (64, 2)])
def test_prefill_par_lds_and_thread_ranges(dh, qw):
    """The few-pair prefill (4 wave groups of qw waves, as launched up to 64
    pairs and beyond): each group's DMA ring, the in-block tile, the null row and
    the split-state slots stay inside the workgroup's LDS; each stage holds a
    page whose operand reads find the chunk the DMA put there; the launch
    indices cover every (pair, part) once, the parts of a pair on one XCD; every
    query row is owned by one wave."""
    BT = 64
    TILE, KBYTES, KRB, _, _ = _ints(plan().ap_ring, 5, dh)
    G, NSP, IPW, THREADS, ROWS, RING, OFF_IN, OFF_NULL, BYTES, STATE = _ints(plan().ap_par, 10, dh, qw)
    assert G == 4 and THREADS == 64 * G * qw and ROWS == 16 * qw and IPW * qw * 1024 == TILE and 3 * IPW < 64
    assert RING == G * NSP * TILE and OFF_IN >= RING and OFF_NULL >= OFF_IN + TILE and OFF_NULL + 4 * dh <= BYTES
    assert BYTES <= 160 * 1024 and (G + 1) * qw * STATE <= RING and STATE >= (dh // 16) * 1024 + 64 * 8
    placed = {}
    for g, w, stage, i, lane in itertools.product(range(G), range(qw), range(NSP), range(IPW), range(64)):
        byte = (w * IPW + i) * 1024 + lane * 16       # of the stage
        lds = (g * NSP + stage) * TILE + byte
        assert 0 <= lds and lds + 16 <= RING and lds not in placed
        placed[lds] = plan().ap_source(dh, byte)
    assert len(placed) * 16 == RING
    for g, stage in itertools.product(range(G), range(NSP)):
        base = (g * NSP + stage) * TILE
        page = {at - base: v for at, v in placed.items() if base <= at < base + TILE}
        assert sorted(page.values()) == list(range(0, TILE, 16))
        if g in (0, G - 1) and stage == NSP - 1:
            _tile_reads_find(dh, page)
    CPR = dh // 8
    assert 2 * CPR <= THREADS and OFF_NULL + 2 * CPR * 16 <= BYTES                    # null row
    # split states: slots 0..3 the memory splits, slot 4 the final split; the
    # folding wave (g, w) reads dimension tile g < dh/16 of each
    assert dh // 16 <= G
    for j, w in itertools.product(range(G + 1), range(qw)):
        base = (j * qw + w) * STATE
        assert base + (dh // 16 - 1) * 1024 + 63 * 16 + 16 <= RING
        assert base + (dh // 16) * 1024 + 63 * 8 + 8 <= (j * qw + w + 1) * STATE
    npart = 4 // qw
    for n_pairs in (1, 7, 8, 9, 96, 128, 511):
        grid = plan().ap_par_grid(n_pairs, qw)
        got = {}
        for n in range(grid):
            pair, part = plan().ap_par_pair(n, qw), plan().ap_par_part(n, qw)
            if pair >= n_pairs:
                continue
            assert (pair, part) not in got
            got[(pair, part)] = n % 8                   # the XCD the index lands on
        assert len(got) == n_pairs * npart
        assert all(got[(p, 0)] == got[(p, k)] for p in range(n_pairs) for k in range(npart))
    rows = sorted(part * ROWS + w * 16 + r for part in range(npart) for w in range(qw) for r in range(16))
    assert rows == list(range(BT))
    assert [plan().ap_par_row_waves(n) for n in (1, 64, 65, 128)] == [1, 1, 2, 2]


def _meta_items(live, edits, mb, chunk=1024, max_edits=128, max_items=128):
    """The host side of a metadata update (push_edits): per group of edits,
    (sequence, chunk, base, last) items from the host's live sets before the
    edits; returns the launches as (edits, items)."""
    import bisect
    launches = []
    n_chunks = (mb + chunk - 1) // chunk
    for i0 in range(0, len(edits), max_edits):
        i1 = min(len(edits), i0 + max_edits)
        group = edits[i0:i1]
        items = []
        for q in sorted({e[0] for e in group}):
            lv = live[q]
            c0 = min([b // chunk for s, b, _ in group if s == q] + [n_chunks])
            c1 = max([lv[-1] // chunk if lv else 0] + [b // chunk for s, b, _ in edits[:i1] if s == q])
            for c in range(c0, c1 + 1):
                base = bisect.bisect_left(lv, c * chunk)
                base += sum(1 if p >= 0 else -1 for s, b, p in edits[:i1] if s == q and b < c * chunk)
                items.append((q, c, base, c == c1))
        for k in range(0, len(items), max_items):
            launches.append((group, items[k:k + max_items]))
    return launches


def _meta_kernel(table, live_page, live_blk, n_live, mb, group, items, chunk=1024):
    """k_meta: each item applies its chunk's edits, then writes the chunk's live
    blocks at the host's position; every access is checked against the arrays."""
    for q, c, base, last in items:
        j0 = c * chunk
        for s, b, p in group:
            if s == q and j0 <= b < j0 + chunk:
                table[q][b] = p
        off = base
        for j in range(j0, min(mb, j0 + chunk)):
            if table[q][j] >= 0:
                assert 0 <= off < mb
                live_page[q][off], live_blk[q][off] = table[q][j], j
                off += 1
        if last:
            n_live[q] = off


@pytest.mark.parametrize("mb,n_seq", [(64, 3), (1024, 2), (4096, 2), (65536, 1)])
def test_metadata_chunk_rebuild_equals_full_rebuild(mb, n_seq):
    """Deletions and insertions (single and in batches of more than 128 edits,
    across sequences): the chunked metadata rebuild leaves the dense live
    lists and counts equal to a full rebuild from the table."""
    import bisect
    import random
    rnd = random.Random(mb)
    table = [[-1] * mb for _ in range(n_seq)]
    live_page = [[-7] * mb for _ in range(n_seq)]
    live_blk = [[-7] * mb for _ in range(n_seq)]
    n_live = [0] * n_seq
    live = [[] for _ in range(n_seq)]
    free = list(range(n_seq * mb))
    rnd.shuffle(free)

    def apply(edits):
        for group, items in _meta_items(live, edits, mb):
            _meta_kernel(table, live_page, live_blk, n_live, mb, group, items)
        for s, b, p in edits:                      # the host update after the launches
            if p >= 0:
                bisect.insort(live[s], b)
            else:
                live[s].remove(b)
        for q in range(n_seq):
            assert n_live[q] == len(live[q])
            assert live_blk[q][:n_live[q]] == live[q]
            assert live_page[q][:n_live[q]] == [table[q][j] for j in live[q]]

    # a batch insert of many blocks (several groups of 128 edits, several sequences)
    first = [(q, b, free.pop()) for q in range(n_seq) for b in rnd.sample(range(mb), min(mb, 300))]
    apply(first)
    for _ in range(40):                              # single edits anywhere, as the store does them
        q = rnd.randrange(n_seq)
        if live[q] and rnd.random() < 0.6:
            apply([(q, rnd.choice(live[q]), -1)])
        else:
            absent = rnd.randrange(mb)
            if absent not in live[q]:
                apply([(q, absent, free.pop())])
    apply([(q, b, -1) for q in range(n_seq) for b in list(live[q])[::3]])   # a batch of deletes


@pytest.mark.parametrize("dh", [32, 64, 128])
def test_encoder_output_staging(dh):
    """The encoder's output rows pass through LDS in the key-plane layout, a
    slot whose byte address has bit SWB set (7; 9 at d_h = 32) holding its
    8-byte halves swapped: every (row, dim) lands in one place, the 16-byte reads
    (halves swapped back) and the transposed gather of a page insert find each
    dim where it was written, and each 16-lane group of an 8-byte write (the
    lanes one pass serves, over 128 bytes of banks) touches each bank once.
    Without the swap the same check fails: two rows of a group share a slot
    modulo 128 bytes."""
    BT, KRB = 64, dh * 2
    key_at = lambda r, c: plan().ap_key_at(dh, r, c)
    SWB = 9 if dh == 32 else 7

    def layout(swap):
        where, clean = {}, True
        for wave, dt in itertools.product(range(4), range(dh // 16)):
            for g in range(4):
                banks = []
                for lane in range(16 * g, 16 * g + 16):
                    qrow, d0 = wave * 16 + (lane & 15), dt * 16 + (lane >> 4) * 4
                    slot = key_at(qrow, d0 >> 3)
                    off = slot + (((d0 >> 2) & 1) ^ (((slot >> SWB) & 1) if swap else 0)) * 8
                    assert 0 <= off and off + 8 <= BT * KRB
                    for i in range(4):
                        assert off + 2 * i not in where
                        where[off + 2 * i] = (qrow, d0 + i)
                    banks += [(off // 4) % 32, (off // 4 + 1) % 32]
                clean &= len(banks) == len(set(banks))
        return where, clean

    assert not layout(False)[1]
    where, clean = layout(True)
    assert clean and len(where) == BT * dh
    for row, c8 in itertools.product(range(BT), range(dh // 8)):       # 16-byte reads, halves swapped back
        slot = key_at(row, c8)
        elems = [where[slot + 2 * e] for e in range(8)]
        if (slot >> SWB) & 1:
            elems = elems[4:] + elems[:4]
        assert elems == [(row, c8 * 8 + e) for e in range(8)]
    for d, r in itertools.product(range(dh), range(BT)):               # the page insert's transposed gather
        slot = key_at(r, d >> 3)
        assert where[slot + (((d & 7) * 2) ^ (((slot >> SWB) & 1) * 8))] == (r, d)


@pytest.mark.parametrize("D", [512, 768, 1024, 2048])
def test_rows_value_operand_transpose_read(D):
    """The row reader's value MFMA (16x16x16) takes B[k][n] = row k of the
    16-row chunk, dim d0 + n, in lane l = 16 (k // 4) + n as element k % 4.
    ds_read_b64_tr_b16 gives lane j of each 16-lane group element i of the
    8 bytes that lane 4 i + j // 4 of the group addressed, taking element
    j % 4 of them (the lane layout measured on gfx950 with LDS holding each
    element's index).  Each lane addresses row l // 4, dims d0 + 4 (l % 4):
    every lane then holds its operand, and every address lies in the chunk."""
    MP = D + 16
    for d0 in range(0, D, 16):
        addr = [(l // 4) * MP + d0 + 4 * (l % 4) for l in range(64)]
        for l in range(64):
            assert 0 <= addr[l] and addr[l] % 4 == 0 and l // 4 < 16 and d0 + 4 * (l % 4) + 4 <= D
            g, j = l // 16, l % 16
            for i in range(4):
                src = 16 * g + 4 * i + j // 4
                assert addr[src] + j % 4 == (4 * g + i) * MP + d0 + j


@pytest.mark.parametrize("D", [512, 768, 1024, 2048])
def test_rows_chunk_pitch_banks(D):
    """The row reader's chunk pitch in LDS is D + 16 bf16.  Bank model (the
    one that fits a one-wave probe of these reads at pads of 8, 16 and 24
    elements: only 16 is conflict-free): 128 banks of 4 bytes, a 16-byte
    read served 32 lanes at a time, a transposing 8-byte read 64 lanes at a
    time.  Under it the score reads (row l % 16, 16 bytes at 16 (l // 16))
    and the transposing value reads (row l // 4, 8 bytes at 8 (l % 4)) touch
    each bank at most once per pass, a 16-byte pad does not, and two chunk
    stages fit in LDS beside the reduction buffers."""
    def clean(pad):
        P = 2 * (D + pad)
        for half in range(2):
            banks = [((l % 16) * P + (l // 16) * 16) // 4 % 128 + i
                     for l in range(32 * half, 32 * half + 32) for i in range(4)]
            if len(set(b % 128 for b in banks)) != len(banks):
                return False
        banks = [((l // 4) * P + (l % 4) * 8) // 4 % 128 + i for l in range(64) for i in range(2)]
        return len(set(b % 128 for b in banks)) == len(banks)
    assert clean(16) and not clean(8) and not clean(24)
    stage = 16 * (D + 16) * 2
    assert 2 * stage + 2 * 4 * 256 * 4 + 2 * 256 * 2 + 2 * 16 * 4 + 64 <= 160 * 1024


@pytest.mark.parametrize("nc", [1, 2, 3, 4])
def test_fused_self_attention_indexing(nc):
    """k_qkv_attn (d = 256 nc, d_h = 32, one workgroup of 8 waves per (block,
    head)): every global and LDS offset stays in its buffer; the chunk
    partials cover (chunk, row, column) exactly once for the chunks that
    exist, and the ordered sum writes every staged q|k|v value once."""
    D, DH, NCOL, CT, BT, RT = 256 * nc, 32, 96, 6, 64, 2
    H = D // DH
    part = [0] * (nc * BT * NCOL)
    for w in range(8):
        c, r0 = w >> 1, (w & 1) * RT * 16
        if c >= nc:
            continue
        for lane in range(64):
            kofs = (lane >> 4) * 8
            for i in range(RT):
                row = r0 + i * 16 + (lane & 15)
                assert row < BT
                for t in range(8):
                    col = c * 256 + kofs + t * 32
                    assert col + 8 <= D                  # x row [blk*64 + row][col .. col+7]
            for h in (0, H - 1):
                for j in range(CT):
                    wrow = (j >> 1) * D + h * DH + (j & 1) * 16 + (lane & 15)
                    assert wrow < 3 * D
                    assert c * 256 + kofs + (8 - 1) * 32 + 8 <= D
            for i in range(RT):
                for j in range(CT):
                    base = (c * BT + r0 + i * 16 + (lane & 15)) * NCOL + j * 16 + 4 * (lane >> 4)
                    for e in range(4):
                        part[base + e] += 1
            if lane < 16:
                for i in range(RT):
                    assert c * BT + r0 + i * 16 + lane < nc * BT    # st0 / st1
    assert part == [1] * len(part)
    stage = [0] * (BT * NCOL)
    for q in range(BT * NCOL // 4):
        row, c0 = q // (NCOL // 4), (q % (NCOL // 4)) * 4
        for ch in range(nc):
            assert (ch * BT + row) * NCOL + c0 + 4 <= nc * BT * NCOL
        for e in range(4):
            stage[row * NCOL + c0 + e] += 1
    assert stage == [1] * len(stage)
    # attention: waves 0..3, query rows 16 w + l % 16; q fragments and the
    # key / value rows read from the stage (row stride 96, k at 32, v at 64)
    for w in range(4):
        for lane in range(64):
            qr = (w * 16 + (lane & 15)) * NCOL + (lane >> 4) * 8
            assert qr + 8 <= BT * NCOL
    cpr, nk = DH // 8, BT * (DH // 8)
    nj = nk + (BT // 2) * cpr
    assert nj <= 512                                        # one job per thread
    for j in range(nj):
        if j < nk:
            assert DH + (j // cpr) * NCOL + (j % cpr) * 8 + 8 <= BT * NCOL
        else:
            pr, c8 = (j - nk) // cpr, (j - nk) % cpr
            assert 2 * DH + (2 * pr + 1) * NCOL + c8 * 8 + 8 <= BT * NCOL
    # output rows: head h in columns [32 h, 32 h + 32)
    for lane in range(64):
        for dt in range(DH // 16):
            assert (H - 1) * DH + dt * 16 + (lane >> 4) * 4 + 4 <= D
    lds = 2 * BT * DH * 2 + nc * BT * NCOL * 4 + BT * NCOL * 2 + 2 * D * 2 + 2 * nc * BT * 4
    assert lds <= 160 * 1024


@pytest.mark.parametrize("M,K,N", [(1, 1024, 50257), (16, 768, 50257), (40, 768, 50257), (64, 1024, 50257),
                                   (64, 256, 8192), (33, 512, 9000), (32, 2048, 50257), (1, 2048, 50257)])
def test_wide_head_indexing(M, K, N):
    """k_linear_wide (fp32 maps of <= 64 rows, K <= 2048, N >= 8192, the x
    rows in LDS: at most 32 rows at K = 2048): the x rows fit the LDS tile,
    every weight row read is < N, every chunk's column range stays inside K,
    and the two tiles of each wave cover the output columns exactly once."""
    RT, XP = (M + 15) // 16, K + 8
    NCH = K // 256
    assert RT * 16 * XP * 2 <= 160 * 1024
    n_tiles = (N + 15) // 16
    grid = (n_tiles + 15) // 16
    cover = [0] * N
    for wg in range(grid):
        for wave in range(8):
            t0 = (wg * 8 + wave) * 2
            if t0 >= n_tiles:
                continue
            second = t0 + 1 < n_tiles
            tiles = [t0, t0 + 1 if second else t0]
            for lane in range(64):
                kofs = (lane >> 4) * 8
                for t in tiles:
                    assert 0 <= min(t * 16 + (lane & 15), N - 1) < N
                for c in range(NCH):
                    assert c * 256 + 7 * 32 + kofs + 8 <= K           # weights and x of chunk c
                    for i in range(RT):
                        assert (i * 16 + (lane & 15)) * XP + kofs + c * 256 + 7 * 32 + 8 <= RT * 16 * XP
            for j, t in enumerate(tiles):
                if j == 1 and not second:
                    break
                for g4 in range(4):
                    for e in range(4):
                        n = t * 16 + 4 * g4 + e
                        if n < N:
                            cover[n] += 1
    assert cover == [1] * N
