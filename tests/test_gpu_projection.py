"""GPU parity of the fused suffix QKV projection + rotary embedding + KV append.

cw_qkv_rope_append runs through the C ABI on seeded synthetic inputs and is
compared with the fp64 oracle (oracle.projection for q/k/v, oracle.paged for
where k and v land in the cache):

* every output element within |got - exp| <= 2^-8 |exp| + 1e-3. The kernel
  rounds each result once to bf16 (half an ulp: 2^-9 relative); fp32
  accumulation of `hidden` exact bf16 products with random signs adds about
  sqrt(hidden) 2^-24 |y| (< 1e-5 at hidden 8192), the fp32 cos/sin table
  another 2^-24 relative. The bound leaves 2x on the rounding term and 100x
  on the rest.
* every cache element that is not a suffix slot keeps its bits exactly;
  suffix slots whose block id lies outside the pool are not written.

Small cases compare everything; the model-sized batches compare sampled rows
(first / last row of every request and random ones) plus the untouched bytes
of the whole cache.
"""
import math

import numpy as np
import pytest
import test_gpu_parity as GP
import torch

from oracle import paged as OP
from oracle import projection as PR
from paper_2606_19667_amd import batch as B
from paper_2606_19667_amd import cw, inputs
from paper_2606_19667_amd import workload as W

pytestmark = pytest.mark.gpu

REL = 2.0 ** -8
ABS = 1e-3
BS = 16


def _say(msg):
    print(msg, flush=True)


def _bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def _f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def _close(got, exp, what):
    got = np.asarray(got, np.float64)
    err = np.abs(got - exp)
    bound = REL * np.abs(exp) + ABS
    worst = float((err - bound).max()) if err.size else -1.0
    _say(f"{what}: n={err.size} max_abs={float(err.max()) if err.size else 0:.3e} "
         f"mean_abs={float(err.mean()) if err.size else 0:.3e} worst_margin={worst:.3e}")
    assert np.isfinite(got).all(), what
    assert (err <= bound).all(), (what, worst)


def _image(cache, new, bt, cu, plen, layout):
    """Expected cache image; slots whose block id is outside the pool are dropped
    (written to a padding block that is cut off again)."""
    nb = cache.shape[0]
    bt2 = np.where((bt >= 0) & (bt < nb), bt, nb)
    ext = np.concatenate([cache, np.zeros_like(cache[:1])])
    return OP.kv_append_image(ext, new, bt2, cu, plen, BS, layout)[:nb]


class Case:
    """A ragged batch, its inputs and the library's outputs."""

    def __init__(self, name, hq, hkv, D, hidden, bt, cu, plen, num_blocks, seed, bias=True, base=500000.0):
        self.name, self.hq, self.hkv, self.D, self.hidden = name, hq, hkv, D, hidden
        self.bt = np.asarray(bt, np.int32)
        self.cu = np.asarray(cu, np.int32)
        self.plen = np.asarray(plen, np.int32)
        self.base = base
        T = int(self.cu[-1])
        nf = (hq + 2 * hkv) * D
        self.x = inputs.normal_bf16((seed, 101), (T, hidden))
        self.w = inputs.scaled_normal_bf16((seed, 102), (nf, hidden), hidden ** -0.5)
        self.b = inputs.scaled_normal_bf16((seed, 103), (nf,), 0.5) if bias else None
        self.k0 = inputs.normal_bf16((seed, 104), (num_blocks, hkv, BS, D))
        self.v0 = inputs.normal_bf16((seed, 105), (num_blocks, hkv, BS, D))
        self.pos = PR.suffix_positions(self.cu, self.plen)

    def run(self):
        meta = cw.BatchMeta(self.bt, self.cu, self.plen, self.hq, self.hkv, self.D)
        n_pos = int(self.pos.max()) + 1 if self.pos.size else 1
        rope = torch.from_numpy(cw.rope_table(n_pos, self.D, self.base)).cuda()
        self.kc, self.vc = self.k0.cuda(), self.v0.cuda()
        _say(f"qkv_rope_append {self.name}: T={int(self.cu[-1])} hidden={self.hidden} "
             f"Hq={self.hq} Hkv={self.hkv} D={self.D} bias={self.b is not None}")
        q = cw.qkv_rope_append(meta, self.x.cuda(), self.w.cuda(), rope, self.kc, self.vc,
                               bias=None if self.b is None else self.b.cuda())
        torch.cuda.synchronize()
        self.q = q
        return self

    def expected(self, rows):
        rows = np.asarray(rows, np.int64)
        return PR.qkv_rope(self.x[torch.as_tensor(rows)], self.w, self.pos[rows], self.hq, self.hkv, self.D,
                           self.base, self.b)

    def written_mask(self):
        T = int(self.cu[-1])
        ones = np.ones((T, self.hkv, self.D), bool)
        mk = _image(np.zeros(self.k0.shape, bool), ones, self.bt, self.cu, self.plen, "slot_d")
        mv = _image(np.zeros(self.v0.shape, bool), ones, self.bt, self.cu, self.plen, "slot_d")
        return mk, mv

    def check_untouched(self):
        mk, mv = self.written_mask()
        assert np.array_equal(_bits(self.kc)[~mk], _bits(self.k0)[~mk]), self.name
        assert np.array_equal(_bits(self.vc)[~mv], _bits(self.v0)[~mv]), self.name
        return mk, mv

    def check_full(self):
        T = int(self.cu[-1])
        q, k, v = self.expected(np.arange(T))
        _close(_f64(self.q), q, self.name + " q")
        mk, mv = self.check_untouched()
        ek = _image(_f64(self.k0), k, self.bt, self.cu, self.plen, "slot_d")
        ev = _image(_f64(self.v0), v, self.bt, self.cu, self.plen, "slot_d")
        _close(_f64(self.kc)[mk], ek[mk], self.name + " k cache")
        _close(_f64(self.vc)[mv], ev[mv], self.name + " v cache")

    def check_sampled(self, seed=0, n_random=64):
        rng = np.random.default_rng(seed)
        rows = set()
        for r in range(len(self.plen)):
            c0, c1 = int(self.cu[r]), int(self.cu[r + 1])
            if c1 > c0:
                rows.update({c0, c1 - 1})
        T = int(self.cu[-1])
        rows.update(int(t) for t in rng.integers(0, T, size=n_random))
        rows = np.array(sorted(rows))
        q, k, v = self.expected(rows)
        _close(_f64(self.q[torch.as_tensor(rows, device=self.q.device)]), q, self.name + " q (sampled rows)")
        self.check_untouched()
        kc, vc = _f64(self.kc), _f64(self.vc)
        gk, gv, ek, ev = [], [], [], []
        req = np.searchsorted(self.cu, rows, side="right") - 1
        for i, (t, r) in enumerate(zip(rows, req)):
            p = int(self.pos[t])
            blk = int(self.bt[r, p // BS])
            if 0 <= blk < kc.shape[0]:
                gk.append(kc[blk, :, p % BS, :])
                gv.append(vc[blk, :, p % BS, :])
                ek.append(k[i])
                ev.append(v[i])
        _close(np.stack(gk), np.stack(ek), self.name + " k cache (sampled rows)")
        _close(np.stack(gv), np.stack(ev), self.name + " v cache (sampled rows)")


def _ragged(name, hq, hkv, D, hidden, plen, slen, seed, holes=(), spare=3, **kw):
    """Blocks of every request drawn from a random permutation of the pool;
    holes: (request, logical block, id) entries overwritten afterwards."""
    rng = inputs.rng((seed, 106))
    nblk = [math.ceil((p + s) / BS) for p, s in zip(plen, slen)]
    nb = sum(nblk) + spare
    perm = rng.permutation(nb)
    bt = np.full((len(plen), max(1, max(nblk))), -1, np.int32)
    o = 0
    for r, n in enumerate(nblk):
        bt[r, :n] = perm[o:o + n]
        o += n
    for r, j, v in holes:
        bt[r, j] = v
    cu = np.concatenate([[0], np.cumsum(slen)]).astype(np.int32)
    return Case(name, hq, hkv, D, hidden, bt, cu, plen, nb, seed, **kw)


SMALL = [
    # tiny shape: 6 heads of 64 = 384 features (a partial feature tile), one request
    ("tiny-d64", 4, 1, 64, 256, [64], [32], {}),
    # several token tiles with a ragged tail, empty and one-row requests, bias off
    ("ragged-d128", 8, 2, 128, 512, [0, 48, 16, 0, 320, 32], [300, 0, 1, 17, 129, 211], {"bias": False}),
    # group 1, 3 heads = 384 features (partial tile), one and two hidden steps
    ("g1-h32", 1, 1, 128, 32, [0, 16], [40, 230], {}),
    ("g1-h64", 1, 1, 128, 64, [32, 16], [70, 190], {"base": 10000.0}),
    # three hidden steps, D = 64 with many heads
    ("d64-h96", 16, 4, 64, 96, [16, 0], [260, 5], {}),
    # Qwen2.5-7B-shaped heads (28 Q / 4 KV, hidden 3584, bias)
    ("qwen7b-heads", 28, 4, 128, 3584, [832, 96], [97, 250], {"base": 1e6}),
]


@pytest.mark.parametrize("name,hq,hkv,D,hidden,plen,slen,kw", SMALL, ids=[c[0] for c in SMALL])
def test_qkv_rope_append_matches_oracle(name, hq, hkv, D, hidden, plen, slen, kw):
    _ragged(name, hq, hkv, D, hidden, plen, slen, seed=7, **kw).run().check_full()


def test_blocks_outside_the_pool_are_skipped():
    # request 0's second block is -1, request 1's first is past the pool: nothing lands there
    c = _ragged("holes", 8, 2, 128, 128, [0, 16], [40, 33], seed=9, holes=[(0, 1, -1), (1, 1, 10 ** 6)])
    c.run().check_full()
    assert c.written_mask()[0].sum() == (40 - 16 + 33 - 16) * 2 * 128


def test_empty_batch_writes_nothing():
    c = _ragged("empty", 8, 2, 128, 128, [16, 32], [0, 0], seed=3)
    c.run()
    assert c.q.shape == (0, 8, 128)
    assert np.array_equal(_bits(c.kc), _bits(c.k0)) and np.array_equal(_bits(c.vc), _bits(c.v0))


def test_position_zero_query_is_the_plain_projection():
    # at p = 0 the rotation is the identity: q and k equal y rounded to bf16
    c = _ragged("p0", 4, 1, 64, 64, [0], [1], seed=4)
    c.run()
    y = PR.project(c.x, c.w, c.b)[0]
    _close(_f64(c.q)[0].reshape(-1), y[:4 * 64], "p0 q = y")


def test_llama8b_single_full_size():
    w = W.llama8b_single()
    s = B.schedule(w)
    c = Case(w.name, 32, 8, 128, 4096, s.block_table, s.cu_suffix, s.prefix_len, s.num_blocks, seed=11)
    c.run().check_full()


def test_llama8b_trace_batch16_sampled():
    w = W.llama8b_trace_batch(seed=0, batch=16)
    s = B.schedule(w)
    c = Case(w.name, 32, 8, 128, 4096, s.block_table, s.cu_suffix, s.prefix_len, s.num_blocks, seed=12)
    c.run().check_sampled()


def test_llama70b_long_sampled():
    w = W.long_context("high", batch=3)
    s = B.schedule(w)
    c = Case(w.name, 64, 8, 128, 8192, s.block_table, s.cu_suffix, s.prefix_len, s.num_blocks, seed=13,
             bias=False)
    c.run().check_sampled()


RAGGED = [
    # (query heads, KV heads, head_dim, hidden, prefixes, suffixes)
    (1, 1, 128, 96, [0], [1], {}),
    (8, 2, 128, 1056, [16, 0], [9, 8], {"bias": False}),
    (2, 1, 64, 672, [0, 48], [15, 1], {}),
    (28, 4, 128, 160, [0], [31], {}),
    (28, 4, 128, 2080, [32], [33], {}),
    (28, 4, 64, 160, [0, 16, 0], [30, 0, 35], {"bias": False}),
    (28, 4, 128, 1056, [0, 0], [64, 65], {}),
    (28, 4, 64, 1056, [16], [200], {}),
    (28, 4, 128, 1056, [0, 48], [129, 171], {}),
    (28, 4, 64, 2080, [0], [500], {"bias": False}),
    (28, 4, 128, 2080, [0, 16], [257, 190], {}),
    (28, 4, 64, 544, [0], [1100], {}),
    (28, 4, 128, 544, [0, 32, 0], [700, 1, 499], {}),
    (28, 4, 64, 1056, [0], [2100], {"bias": False}),
    (28, 4, 128, 1056, [0, 0], [1025, 1075], {}),
    (64, 16, 64, 544, [0, 16, 0, 0], [2500, 0, 1999, 2], {}),
]


@pytest.mark.parametrize("hq,hkv,D,hidden,plen,slen,kw", RAGGED,
                         ids=[f"{c[0]}-{c[1]}-{c[2]}-h{c[3]}-t{sum(c[5])}" for c in RAGGED])
def test_ragged_heads_and_hidden(hq, hkv, D, hidden, plen, slen, kw):
    _ragged(f"ragged T={sum(slen)}", hq, hkv, D, hidden, plen, slen, seed=21, **kw).run().check_full()


@pytest.mark.parametrize("T", [15, 60, 700, 1300])
def test_results_at_8_byte_alignment(T):
    """The epilogue stores 16 bytes at a time; results whose storage starts at 8
    bytes past a multiple of 16 get the same bits."""
    c = _ragged(f"8-byte aligned T={T}", 24, 4, 128, 160, [16], [T], seed=26).run()
    meta = cw.BatchMeta(c.bt, c.cu, c.plen, c.hq, c.hkv, c.D)
    rope = torch.from_numpy(cw.rope_table(int(c.pos.max()) + 1, c.D, c.base)).cuda()

    def shifted(t):
        flat = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")
        view = flat[4:].view(t.shape)
        view.copy_(t)
        assert view.data_ptr() % 16 == 8
        return view
    q, kc, vc = shifted(torch.zeros_like(c.q)), shifted(c.k0), shifted(c.v0)
    cw.qkv_rope_append(meta, c.x.cuda(), c.w.cuda(), rope, kc, vc, bias=c.b.cuda(), q_out=q)
    torch.cuda.synchronize()
    for got, expect in ((q, c.q), (kc, c.kc), (vc, c.vc)):
        assert np.array_equal(_bits(got), _bits(expect)), c.name


# Kernel of each tile shape (features x tokens), and row counts that select it with
# 25 / 5 heads of 128 (4,480 features) and 27 / 3 of 64 (2,112): neither a multiple
# of 256. The row counts are edges of the tile's range and of tiles of tokens.
TILES = {
    "32x16": ("qkv_stream_kernel<{D}, 1, 1, 4, 6, 2, 1>", {128: [1, 15, 16], 64: [1, 17, 47]}),
    "32x32": ("qkv_stream_kernel<{D}, 1, 2, 4, 5, 2, 2>", {128: [17, 31, 32], 64: [63, 65, 96]}),
    "32x64": ("qkv_stream_kernel<{D}, 1, 4, 2, 6, 2, 2>", {128: [33, 63, 64], 64: [97, 127, 129]}),
    "64x64": ("qkv_stream_kernel<{D}, 2, 4, 2, 5, 2, 2>", {128: [65, 127, 129], 64: [193, 255, 257]}),
    "128x128": ("qkv_block_kernel<{D}>", {128: [193, 257, 511], 64: [449, 513, 897]}),
    "256x128": ("qkv_tile_kernel<{D}>", {128: [897, 1023, 1025], 64: [1921, 2049]}),
    "256x256": ("qkv_rope_append_kernel<{D}>", {128: [1793, 2049], 64: [3841, 4097]}),
}
HEADS = {128: (25, 5), 64: (27, 3)}


def _tile_of(names):
    """Tile shape and head_dim of the projection kernel among `names`."""
    return [(tile, D) for tile, (kernel, rows) in TILES.items() for D in rows
            if any(kernel.format(D=D) in n for n in names)]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("tile", TILES)
def test_every_tile_shape(tile, D):
    """Each shape at the edges of its tiles, with one to 17 steps of hidden, whole
    and half (hidden below 160 never takes the 32 x 16 tile)."""
    kernel, rows = TILES[tile]
    for n, T in enumerate(rows[D]):
        for hidden in [160, 672, 1056] if tile == "32x16" else [32, 64, 96, 160, 1056]:
            cut = T // 3
            slen, plen = ([cut, 0, T - cut], [16, 48, 0]) if cut else ([T], [32])
            c = _ragged(f"{tile} T={T} hidden={hidden} D={D}", *HEADS[D], D, hidden, plen, slen, seed=21,
                        bias=n % 2 == 0)
            assert _tile_of(GP.kernels(c.run)) == [(tile, D)], c.name
            c.check_full() if T * hidden < 1e6 else c.check_sampled()


@pytest.mark.parametrize("hidden", [32, 96, 192])
@pytest.mark.parametrize("D", [64, 128])
def test_persistent_ring_runs_on_across_tiles(hidden, D):
    """More tiles than workgroups (1.75 rounds) at one, two and three steps a tile:
    a tile's first copies go out during the tile before it."""
    hq, hkv = (128, 64) if D == 64 else (64, 32)
    c = _ragged(f"rounds-h{hidden}-d{D}", hq, hkv, D, hidden, [0, 16, 0, 0], [900, 0, 699, 2], seed=22)
    assert _tile_of(GP.kernels(c.run)) == [("256x256", D)]
    c.check_sampled(n_random=400)


@pytest.mark.parametrize("hidden", [96, 1056])
@pytest.mark.parametrize("D", [64, 128])
def test_rows_alone_equal_rows_in_a_batch(D, hidden):
    """A request projected by itself gives the bits that it gets in a batch, with
    every tile shape (each sums over hidden in the same order)."""
    hq, hkv = HEADS[D]
    slen = [1, 17, 40, 70, 100, 200, 300, 480, 950, 2200] if D == 64 else [1, 17, 40, 70, 200, 300, 480, 950]
    plen = [16 * (i % 4) for i in range(len(slen))]
    c = _ragged(f"batch of {len(slen)}", hq, hkv, D, hidden, plen, slen, seed=25)
    seen = set(_tile_of(GP.kernels(c.run)))
    for r, (n, P) in enumerate(zip(slen, plen)):
        c0 = int(c.cu[r])
        one = _ragged(f"request of {n}", hq, hkv, D, hidden, [P], [n], seed=25)
        one.x, one.w, one.b = c.x[c0:c0 + n], c.w, c.b
        seen |= set(_tile_of(GP.kernels(one.run)))
        assert np.array_equal(_bits(one.q), _bits(c.q[c0:c0 + n])), (one.name, "q")
        for name in ("kc", "vc"):
            got, all_ = _bits(getattr(one, name)), _bits(getattr(c, name))
            pos = P + np.arange(n)
            rows = got[one.bt[0][pos // BS], :, pos % BS]
            assert np.array_equal(rows, all_[c.bt[r][pos // BS], :, pos % BS]), (one.name, name)
    # (32 x 16 is not taken at hidden 96)
    assert seen == {(t, D) for t in TILES if hidden > 96 or t != "32x16"}, seen


def _many_requests(total, seed):
    """Suffix lengths 0 to 5, half of them 0, that add up to `total`, with a run of
    40 empty requests and one of 40 one-row requests."""
    rng = inputs.rng((seed, 107))
    s = [1] * min(40, total) + [0] * 40
    while sum(s) < total:
        s.append(min(int(rng.integers(-4, 6).clip(0)), total - sum(s)))
    rng.shuffle(s[:20])
    return s + [0] * 20, [16 * int(p) for p in rng.integers(0, 4, size=len(s) + 20)]


@pytest.mark.parametrize("total", [16, 30, 60, 140, 300, 450, 1200, 2100])
@pytest.mark.parametrize("D", [64, 128])
def test_many_short_and_empty_requests(total, D):
    """Tiles of every size over more requests than the lookup walks one by one."""
    slen, plen = _many_requests(total, total)
    _ragged(f"many-requests-{len(slen)}", 28, 4, D, 160, plen, slen, seed=23).run().check_full()


def test_empty_requests_cost_little():
    """The lookup of a token's request does not grow with the empty requests before
    it: 20,000 of them between two requests take less than 4 times the call's time
    without them (one after the other they took 25 times as long)."""
    def call(slen):
        plen = [16] * len(slen)
        c = _ragged(f"{len(slen)} requests", 8, 2, 128, 256, plen, slen, seed=24)
        meta = cw.BatchMeta(c.bt, c.cu, c.plen, c.hq, c.hkv, c.D)
        rope = torch.from_numpy(cw.rope_table(int(c.pos.max()) + 1, c.D, c.base)).cuda()
        x, w, kc, vc = c.x.cuda(), c.w.cuda(), c.k0.cuda(), c.v0.cuda()
        best = math.inf
        for _ in range(8):   # (a call before it takes the host's check of the batch out of the time)
            torch.cuda.synchronize()
            torch.cuda._sleep(5_000_000)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            cw.qkv_rope_append(meta, x, w, rope, kc, vc)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    short, long = call([300, 300]), call([300] + [0] * 20000 + [300])
    _say(f"two requests {short * 1e3:.1f} us, with 20,000 empty ones between {long * 1e3:.1f} us")
    assert long < 4 * short
