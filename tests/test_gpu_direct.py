"""The direct form of the exact compressor (every element read in every pass,
taken by gradients of at most 6,291,456 elements) against the oracle, at the
sizes and values where its pieces, records and rules change: chunk and vector
edges, more than 64 and more than 1,024 tensors, many keys inside one 22-bit
prefix (equal, different, in pieces that store counts in place of keys),
1-bit sums taken by slices, and a context that alternates with the candidate
form."""
import numpy as np
import pytest
import torch

import oracle
from paper_1704_05021_amd import gd
from parity import check_case

pytestmark = pytest.mark.gpu


def _layout(rng, n, tensors):
    return [0] + np.sort(rng.integers(0, n + 1, tensors - 1)).tolist() + [n]


@pytest.mark.parametrize("tensors", [1, 5, 64, 65, 1025])
@pytest.mark.parametrize("n", [1, 3, 1023, 4096, 4097, 16_387, 1_000_003, 4_718_592, 4_718_593, 6_291_456])
def test_sizes(n, tensors):
    rng = np.random.default_rng(n + tensors)
    off = _layout(rng, n, tensors)
    g = (rng.standard_t(3, n) * 1e-3).astype(np.float32)
    r = (rng.normal(0, 1e-3, n) * (rng.random(n) < 0.5)).astype(np.float32)
    comp = gd.Compressor(off)
    for per, quant, drop in ((False, gd.GD_QUANT_SIGN_MEAN, 0.99), (True, False, 0.9))[:2 if n < 4_000_000 else 1]:
        check_case(g, r, off, drop, per, quant, comp=comp, what=f"n={n} T={tensors} per={per}")


@pytest.mark.parametrize("spread", [1, 2, 40, 512, 3000], ids=lambda s: f"{s}_values")
@pytest.mark.parametrize("per_tensor", [False, True], ids=["global", "per_tensor"])
def test_many_keys_in_one_prefix(per_tensor, spread):
    # `spread` neighbouring binary32 values share the threshold's prefix (512 low
    # bits), far more of them than one piece stores as keys; both forms in turn
    rng = np.random.default_rng(spread)
    n = 60_000
    off = [0, 7, 30_001, n]
    g = (np.float32(1.0).view(np.uint32) + rng.integers(0, spread, n).astype(np.uint32)).view(np.float32)
    g = g * np.where(rng.random(n) < 0.5, -1, 1).astype(np.float32)
    g[rng.random(n) < 0.02] *= 4.0
    comp = gd.Compressor(off)
    for drop in (0.99, 0.5):
        for debug in (0, 3, 0):
            check_case(g, np.zeros(n, np.float32), off, drop, per_tensor, gd.GD_QUANT_THRESHOLD, comp=comp,
                       debug_bracket=debug, what=f"spread={spread} drop={drop} debug={debug}")


@pytest.mark.parametrize("spread", [17, 512, 512 * 40, 512 * 256, 512 * 600], ids=lambda s: f"{s}_values")
def test_lists_and_counts_of_keys(spread):
    # keys in the threshold's prefix per piece of 4,096 elements: all of them (counts
    # are stored), about 100 (counts), 16 (counts in some pieces, lists in others) and 7
    # (lists); segments that begin and end with pieces of 196 and 312 elements, too
    # short for counts, of one such piece, and of many pieces
    rng = np.random.default_rng(spread)
    off = [0, 3_900, 12_600, 12_700, 700_001]
    n = off[-1]
    g = (np.float32(1.0).view(np.uint32) + rng.integers(0, spread, n).astype(np.uint32)).view(np.float32)
    g = g * np.where(rng.random(n) < 0.5, -1, 1).astype(np.float32)
    comp = gd.Compressor(off)
    for per in (False, True):
        for drop in (0.99, 0.7, 0.3):
            check_case(g, np.zeros(n, np.float32), off, drop, per, False, comp=comp, what=f"spread={spread} per={per} drop={drop}")


@pytest.mark.parametrize("quant", [gd.GD_QUANT_SIGN_MEAN, gd.GD_QUANT_GLOBAL_MEAN], ids=["sign_mean", "global_mean"])
@pytest.mark.parametrize("keep", [65_536, 65_537])
def test_sums_by_slices(quant, keep):
    rng = np.random.default_rng(keep)
    n = 400_000
    off = [0, 100, 100, 300_000, n]
    g = rng.normal(0, 1e-3, n).astype(np.float32)
    check_case(g, np.zeros(n, np.float32), off, 1.0 - keep / n, False, quant, what=f"keep={keep}")
    assert gd.keep_count(n, 1.0 - keep / n) in (keep, keep - 1)


@pytest.mark.parametrize("n", [5, 4_098, 300_003])
def test_pull_from_copy(n):
    rng = np.random.default_rng(n)
    p = rng.normal(0, 1e-2, n).astype(np.float32)
    copy = np.where(rng.random(n) < 0.9, p, p + rng.normal(0, 1e-3, n)).astype(np.float32)
    off = _layout(rng, n, 3)
    comp = gd.Compressor(off)
    for per in (False, True):
        for drop in (0.99, 0.5):  # the second keeps zeros
            pt, ct = torch.from_numpy(p).cuda(), torch.from_numpy(copy).cuda()
            out = comp.compress_pull(pt, ct, drop, per_tensor=per)
            torch.cuda.synchronize()
            o, oc = oracle.compress_pull(p, copy, off, drop, per_tensor=per)
            assert np.array_equal(out.idx[:out.k].cpu().numpy().view(np.uint32), o.idx)
            assert np.array_equal(out.val[:out.k].cpu().numpy().view(np.uint32), o.val.view(np.uint32))
            assert np.array_equal(ct.cpu().numpy().view(np.uint32), oc.view(np.uint32))
            assert np.array_equal(out.tensor_counts[:comp.T].cpu().numpy().view(np.uint32), o.tensor_counts)


@pytest.mark.parametrize("quant", [gd.GD_QUANT_SIGN_MEAN, gd.GD_QUANT_GLOBAL_MEAN, gd.GD_QUANT_THRESHOLD],
                         ids=["sign_mean", "global_mean", "threshold"])
@pytest.mark.parametrize("tensors", [3, 900, 1023, 1024, 5000])
def test_sums_over_many_tensors(tensors, quant):
    # slices of 4,096 sent entries inside one tensor, across a few and across
    # thousands (empty ones among them): tensors of at most and more than 32
    # entries in a slice, one that spans several slices, few entries in all
    rng = np.random.default_rng(tensors)
    sizes = rng.choice([0, 1, 5, 31, 32, 33, 64, 400], tensors)
    sizes[rng.integers(0, tensors, 2)] = [30_000, 6_000]
    off = [0] + np.cumsum(sizes).tolist()
    g = rng.normal(0, 1e-3, off[-1]).astype(np.float32)
    comp = gd.Compressor(off)
    for per, drop in ((False, 0.0), (True, 0.0), (False, 0.3), (True, 0.5), (False, 0.99), (False, 1.0)):
        check_case(g, np.zeros_like(g), off, drop, per, quant, comp=comp, what=f"T={tensors} per={per} drop={drop}")


@pytest.mark.parametrize("run", [1, 2, 63, 64, 65, 66, 200], ids=lambda r: f"runs_of_{r}")
def test_counts_of_crowded_tensors(run):
    # one threshold over tensors that start together (all but the last empty): at
    # the first element, at a unit's start, inside a unit (two runs in a row, then a
    # tensor per element over three units), at the last element and past it
    n = 10_000
    off = [0] * run + [700] * run + [1024] * run + [1500] * run + [1501] * (run + 1) + list(range(3_000, 6_072))
    off += [8191] * run + [n - 1] * run + [n] * run
    rng = np.random.default_rng(run)
    g = rng.normal(0, 1e-3, n).astype(np.float32)
    comp = gd.Compressor(off)
    for drop in (0.99, 0.5, 0.0):
        check_case(g, np.zeros_like(g), off, drop, False, False, comp=comp, what=f"run={run} drop={drop}")


@pytest.mark.parametrize("layout", ["empty_in_a_row", "one_element_each"])
def test_crowded_tensors_cost_no_more_than_in_the_candidate_form(layout):
    n, t = 6_144_000, 20_000
    off = [0] + ([n // 2] * t if layout == "empty_in_a_row" else list(range(1, t))) + [n]
    comp = gd.Compressor(off)
    g = torch.randn(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    out = comp.alloc_out(0.99)

    def us(mode):
        comp.debug_force_bracket(mode)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times = []
        for _ in range(9):
            r = torch.zeros_like(g)
            torch.cuda.synchronize()
            ev[0].record()
            comp.compress(g, r, 0.99, out=out)
            ev[1].record()
            torch.cuda.synchronize()
            times.append(1e3 * ev[0].elapsed_time(ev[1]))
        comp.debug_force_bracket(0)
        return sorted(times)[4]

    direct, candidates = us(0), us(5)
    # about a half and a tenth; 44 and 1.5 times as long where a lane took one tensor after another
    assert direct < 1.2 * candidates, f"{direct:.0f} us, candidate form {candidates:.0f} us"


@pytest.mark.parametrize("debug", [0, 1], ids=["direct", "candidates"])
def test_state_of_segments_that_keep_nothing(debug):
    # 50 entries at 99% drop, and an empty tensor: the state is this call's, not an
    # earlier one's that kept half of them
    off = [0, 50, 50, 100_000]
    rng = np.random.default_rng(5)
    g = np.zeros(off[-1], np.float32)
    g[::7] = rng.normal(0, 1, g[::7].size).astype(np.float32)  # half kept needs zeros
    comp = gd.Compressor(off)
    for drop in (0.5, 0.99):
        check_case(g, np.zeros_like(g), off, drop, True, False, comp=comp, debug_bracket=debug, what=f"drop={drop}")
    segs = comp.debug_state()[0]
    for s in segs[:2]:
        assert (s["thr"], s["need"], s["zero"], s["miss"], s["clo"]) == (0xFFFFFFFF, 0, 0, 0, 0), s
    assert segs[2]["thr"] not in (0, 0xFFFFFFFF) and segs[2]["zero"] == 0


@pytest.mark.parametrize("quant", [gd.GD_QUANT_NONE, gd.GD_QUANT_SIGN_MEAN, gd.GD_QUANT_COLUMN_MEAN],
                         ids=["plain", "sign_mean", "column_mean"])
def test_captured_call(quant):
    # replayed with other calls on the same context between the replays
    rng = np.random.default_rng(quant)
    off = [0, 1_000, 1_000, 60_000, 90_001]
    n = off[-1]
    comp = gd.Compressor(off)
    comp.set_columns([10, 1, 100, 1])
    g = rng.normal(0, 1e-3, n).astype(np.float32)
    gt, rt = torch.from_numpy(g).cuda(), torch.zeros(n, device="cuda")
    out = comp.alloc_out(0.99, quant=quant)
    r2 = torch.zeros(n, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        comp.compress(gt, rt, 0.99, quant=quant, out=out)
    for step in range(5):
        r = rt.cpu().numpy()
        graph.replay()
        torch.cuda.synchronize()
        o = oracle.compress(g, r, off, 0.99, per_tensor=False, quant=quant, columns=[10, 1, 100, 1])
        k = o.idx.size
        assert out.k == k
        assert np.array_equal(out.idx[:k].cpu().numpy().view(np.uint32), o.idx), step
        assert np.array_equal(out.val[:k].cpu().numpy().view(np.uint32), o.val.view(np.uint32)), step
        assert np.array_equal(out.tensor_counts.cpu().numpy().view(np.uint32), o.tensor_counts), step
        # centres are fp64 sums in another order, rounded to binary32: the residual of a
        # sent entry is off by the centre's rounding, 2^-23 of at most 1e-2
        np.testing.assert_allclose(rt.cpu().numpy(), o.residual, rtol=0, atol=0 if not quant else 2.0 ** -23 * 1e-2)
        comp.compress(gt, r2, 0.5, per_tensor=True, quant=quant)
        comp.compress_sampled(gt, r2, 0.9, sample_ppm=100_000, quant=quant)
