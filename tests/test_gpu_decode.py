"""GPU decoder (kp_trace_reduce, through the C ABI) against the CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

import inputs
from inputs import PHASE_END as E
from inputs import PHASE_START as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kp():
    import paper_2505_21661_amd as kp

    return kp


def check(raw, oracle_mod, use_hdr=False, threads=8):
    from tests.gpu_util import assert_stats_equal, gpu_decode_bytes

    want = oracle_mod.decode_bytes(raw, threads)
    got = gpu_decode_bytes(raw, use_hdr=use_hdr)
    assert_stats_equal(want, got, oracle_mod)


def test_hand_patterns(kp, oracle_mod):
    cases = [
        ([[(S, 0, 10), (E, 0, 30), (S, 1, 40), (E, 1, 100)]], 2, 16),
        ([[(S, 0, 10), (S, 1, 20), (E, 1, 50), (E, 0, 90)]], 2, 16),
        ([[(S, 0, 0), (E, 0, 5), (S, 0, 8), (E, 0, 16), (S, 0, 20), (E, 0, 21)]], 1, 16),
        ([[(S, 0, 0), (E, 0, 10)], [(S, 1, 5), (S, 0, 12), (E, 1, 15), (E, 0, 20)]], 2, 16),
        ([[(S, 0, 0), (E, 0, 10)], [(S, 0, 5), (E, 0, 15)]], 1, 16),
        ([[(S, 0, 0), (E, 0, 10), (S, 1, 20), (E, 1, 30), (S, 0, 40), (E, 0, 50), (S, 1, 60)]], 2, 4),
        ([[(S, 0, 0), (S, 0, 7), (E, 0, 10), (E, 0, 30)]], 1, 16),
        ([[], []], 2, 8),
        # equal timestamps across waves and inside a wave
        ([[(S, 0, 5), (E, 0, 5), (S, 1, 5), (E, 1, 9)], [(S, 1, 5), (E, 1, 9), (S, 0, 9), (E, 0, 9)],
          [(S, 0, 5), (S, 1, 5), (E, 0, 9), (E, 1, 9)]], 2, 8),
    ]
    for evs, R, cap in cases:
        for flush in (False, True):
            wg = inputs.events_to_wg(evs, cap, flush=flush)
            raw = inputs.encode_trace([wg], len(evs), R, cap, rec_cost=1, flush=flush)
            check(raw, oracle_mod)
            check(raw, oracle_mod, use_hdr=True)


def test_clock_wrap_and_span_overflow(kp, oracle_mod):
    wg = inputs.events_to_wg([[(S, 0, 0xFFFFFFF0), (E, 0, 0x10)]], 8, t_end=1000 + (1 << 32) + 100)
    check(inputs.encode_trace([wg], 1, 1, 8), oracle_mod)


@pytest.mark.parametrize("seed", range(24))
def test_messy_traces(kp, oracle_mod, seed):
    waves = [1, 2, 3, 4, 7, 8, 16][seed % 7]
    n_regions = [1, 3, 5, 16, 17, 32][seed % 6]
    cap = [2, 8, 16, 64, 256][seed % 5]
    raw = inputs.messy_trace(1000 + seed, n_wg=9, waves=waves, n_regions=n_regions, cap_wave=cap,
                             p_bad=0.03 if seed % 3 else 0.0, allow_nonmono=bool(seed % 2),
                             flush=(seed % 4 == 3))
    check(raw, oracle_mod, use_hdr=bool(seed & 1))


def test_small_gemm_shape_trace(kp, oracle_mod):
    raw, _ = inputs.gen_trace(inputs.spec_small_gemm_shape())
    check(raw, oracle_mod)


@pytest.mark.parametrize("log2n,wrap", [(17, False), (20, False), (20, True), (22, False)])
def test_decode_workload_scaled(kp, oracle_mod, log2n, wrap):
    raw, _ = inputs.gen_trace(inputs.spec_decode_standalone(log2n, wrap=wrap))
    check(raw, oracle_mod, use_hdr=True)


@pytest.mark.parametrize("W,R,cap,total", [(4, 5, 1024, 1500), (8, 20, 1024, 1024), (16, 16, 1024, 700),
                                             (2, 32, 4096, 4096), (5, 3, 512, 512), (1, 2, 16384, 20000)])
def test_other_geometries(kp, oracle_mod, W, R, cap, total):
    spec = inputs.TraceSpec(n_wg=37, waves=W, n_regions=R, cap_wave=cap, total_per_wave=total, total_var=total // 3,
                            seed=W * 100 + R, dist="lognormal", p0=5.0, p1=1.2, p_orphan=0.03, p_swap=0.002)
    raw, _ = inputs.gen_trace(spec)
    check(raw, oracle_mod)


@pytest.mark.parametrize("p0", [0.0, 1.0, 2.0, 3.0, 4.0, 5.0, 6.5, 8.0, 10.0, 12.0, 14.0])
def test_spans_from_a_few_ticks_to_many_million(kp, oracle_mod, p0):
    """The overlap sweep bins a workgroup's records into time cells whose width follows the workgroup's
    span; spans from fewer ticks than cells to 2^27 ticks take every form of that width (and, at the
    long end, the wide merge keys), and the phase offsets give every workgroup a different span."""
    for W, cap, seed in ((8, 128, 1), (3, 1024, 2)):
        spec = inputs.TraceSpec(n_wg=24, waves=W, n_regions=6, cap_wave=cap, total_per_wave=cap, seed=seed + int(10 * p0),
                                dist="lognormal", p0=p0, p1=0.7, gap_max=1 if p0 < 3 else 32, phase_min=0,
                                phase_max=int(2 ** min(p0 + 2, 12)) - 1, p_orphan=0.01)
        raw, _ = inputs.gen_trace(spec)
        n_wg = int(raw[2])
        hdr = raw[16:16 + 32 * n_wg].reshape(n_wg, 32).astype(np.uint64)
        span = (hdr[:, 4] | (hdr[:, 5] << np.uint64(32))) - (hdr[:, 2] | (hdr[:, 3] << np.uint64(32)))
        assert span.max() < 2 ** 32
        check(raw, oracle_mod)


@pytest.mark.parametrize("n_wg,W,R,cap", [
    (256, 1, 8, 256), (257, 1, 8, 256), (257, 1, 9, 256), (257, 2, 17, 128), (256, 2, 17, 128),      # 256 records
    (256, 4, 3, 256), (300, 4, 8, 256), (300, 4, 16, 256), (300, 4, 17, 256), (300, 16, 32, 32),    # up to 1024
    (256, 8, 32, 512), (260, 8, 8, 512), (260, 8, 16, 512), (260, 8, 17, 512), (260, 16, 8, 256),  # up to 4096
    (3300, 16, 8, 16), (1500, 16, 32, 16), (4100, 1, 1, 2), (513, 3, 5, 64), (5000, 5, 7, 32)])
def test_every_split_of_the_decoder(kp, oracle_mod, n_wg, W, R, cap):
    """The number of recorded workgroups, of record slots and of regions decide how many threads decode a workgroup, how
    many records a lane takes and how many workgroups share one set of totals: both sides of every line, clean and damaged
    traces, crowded and sparse clocks.  (Most of these are over after one turn.)"""
    for p0, seed in ((1.0, 1), (5.0, 2), (11.0, 3)):
        spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=R, cap_wave=cap, total_per_wave=cap, total_var=cap // 2, seed=seed,
                                dist="lognormal", p0=p0, p1=1.0, gap_max=1 if p0 < 3 else 32, p_orphan=0.02, p_swap=0.01 if cap >= 16 else 0.0)
        raw, _ = inputs.gen_trace(spec)
        check(raw, oracle_mod, use_hdr=True)
    raw = inputs.messy_trace(n_wg + W, n_wg=min(n_wg, 600), waves=W, n_regions=R, cap_wave=min(cap, 64), p_bad=0.01, allow_nonmono=False)
    check(raw, oracle_mod, use_hdr=True)


# one or two geometries (up to 15 waves and 16) of every form that can be given more recorded workgroups than its decoder
# workgroups and their teams take at a time, with 256 CUs; the forms for at most as many as CUs are the ones that cannot
@pytest.mark.parametrize("n_wg,W,R,cap", [
    (300, 8, 16, 1024), (301, 16, 20, 512),                                                      # 1024 threads, 256 at a time
    (1100, 8, 8, 256), (1050, 16, 8, 128), (801, 8, 16, 256), (790, 16, 9, 128), (601, 8, 17, 256), (555, 16, 32, 128),  # 256 threads
    (3301, 4, 3, 128), (3109, 16, 8, 32), (3302, 4, 16, 128), (3111, 16, 11, 32), (1701, 4, 17, 128), (1600, 16, 32, 32),  # a wave, 16 records per lane
    (4501, 2, 8, 64), (3300, 4, 16, 64), (3333, 16, 9, 16), (2201, 2, 17, 64), (2100, 16, 32, 16)])                  # a wave, four records per lane
def test_every_form_of_the_decoder_over_several_turns(kp, oracle_mod, n_wg, W, R, cap):
    """What a decoder workgroup carries from one recorded workgroup into the next: requests, sums that are reset behind
    their last use, totals; with damaged workgroups between clean ones."""
    from tests.gpu_util import damaged_between_clean_trace

    check(damaged_between_clean_trace(n_wg, n_wg, W, R, cap), oracle_mod, use_hdr=True)


# rings of at least the 1024 (256 with four records per lane) slots that a hardware wave takes, of at least the 128 of one of
# its rounds, and smaller ones, for the kernels with 1024 threads, 256, and one wave, each with up to 16 regions and with more
@pytest.mark.parametrize("n_wg,W,R,cap", [
    (300, 8, 16, 2048), (260, 16, 20, 512), (260, 2, 5, 1024), (260, 8, 16, 512), (260, 16, 9, 64),       # 16 records per lane
    (300, 1, 5, 1024), (300, 4, 16, 128), (300, 16, 20, 32),
    (40, 8, 5, 512), (40, 4, 5, 256), (40, 4, 5, 128), (40, 8, 5, 64), (40, 1, 3, 256), (40, 2, 3, 64), (300, 2, 8, 128),  # four
    (40, 1, 20, 4096), (40, 8, 20, 512), (40, 4, 20, 256), (40, 4, 32, 128), (40, 16, 20, 64), (40, 1, 20, 256), (40, 2, 20, 64),  # more than 16 regions
    (400, 8, 16, 64), (401, 8, 16, 64), (1400, 3, 17, 128), (1401, 3, 17, 128), (300, 1, 3, 1024),  # either side of the line between 256 threads and one wave
    (260, 8, 16, 1024), (260, 4, 24, 2048), (260, 16, 32, 512), (20, 1, 3, 8192), (260, 3, 16, 2048),  # 512 threads
    (300, 16, 16, 128), (300, 2, 20, 1024), (300, 1, 3, 2048), (1500, 2, 8, 1024)])  # 128, the last one not
def test_the_oldest_record_anywhere_in_the_ring(kp, oracle_mod, n_wg, W, R, cap):
    """Records are paired where they lie, in the order of a ring that begins with its oldest one: rings that wrapped by any
    number of records or not at all, oldest records that are ENDs, STARTs and ENDs of a pair at the two ends of a ring and of
    a hardware wave's share; with records outside the slot of their seq, seqs that occur twice and bad records, and with
    regions inside regions."""
    from tests.gpu_util import nested_trace

    spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=R, cap_wave=cap, total_per_wave=3 * cap, total_var=2 * cap + cap // 2, seed=cap + W,
                            dist="exp", p0=40.0, gap_max=4, p_orphan=0.1, p_swap=0.002)
    raw, _ = inputs.gen_trace(spec)
    check(raw, oracle_mod, use_hdr=True)
    raw = raw.copy()
    slots = raw[16 + 32 * n_wg:].reshape(n_wg, W, cap, 2)
    rng = np.random.default_rng(cap)
    for wg in range(n_wg):
        seg, a = slots[wg, int(rng.integers(0, W))], int(rng.integers(0, cap - 1))
        if wg % 5 == 1:    # a seq that occurs twice
            seg[a + 1, 0] = (seg[a + 1, 0] & ~np.uint32(0xFFFFF)) | (seg[a, 0] & np.uint32(0xFFFFF))
        elif wg % 5 == 2:  # a bad record
            seg[a, 0] |= np.uint32(0x7F000000)
        elif wg % 5 == 3:  # the records at the two ends of the ring, each in the other's slot
            seg[[0, cap - 1]] = seg[[cap - 1, 0]]
    check(raw, oracle_mod, use_hdr=True)
    check(nested_trace(cap, W, R, cap, depth=min(3, R), inner=4), oracle_mod, use_hdr=True)


def test_empty_trace(kp, oracle_mod):
    check(inputs.encode_trace([], 4, 3, 8), oracle_mod)


def test_errors(kp):
    raw, _ = inputs.gen_trace(inputs.spec_small_gemm_shape())
    n_wg, W, R, cap = (int(x) for x in raw[2:6])
    dev = torch.from_numpy(raw.view(np.int32)).cuda()
    out = torch.zeros(kp.kp_stats_bytes(n_wg, W, R), dtype=torch.uint8, device="cuda")
    with pytest.raises(kp.KperfError) as e:
        kp.kp_trace_reduce(dev, n_wg * W * cap + 1, out)
    assert e.value.status == kp.KP_ERR_BAD_TRACE
    bad = raw.copy(); bad[0] ^= 4
    with pytest.raises(kp.KperfError) as e:
        kp.kp_trace_reduce(torch.from_numpy(bad.view(np.int32)).cuda(), n_wg * W * cap, out)
    assert e.value.status == kp.KP_ERR_BAD_TRACE
    # more record slots per workgroup than any kernel takes; more regions than the tag names
    with pytest.raises(kp.KperfError) as e:
        kp.kp_trace_reduce_hdr(dev, 16 * (1 << 16), kp.make_hdr(1, 16, 4, 1 << 16), out)
    assert e.value.status == kp.KP_ERR_UNSUPPORTED_SHAPE
    with pytest.raises(kp.KperfError) as e:
        kp.kp_trace_reduce_hdr(dev, n_wg * W * cap, kp.make_hdr(n_wg, W, 129, cap), out)
    assert e.value.status == kp.KP_ERR_BAD_TRACE
    # host header that disagrees with the device header: flagged in the stats block, no statistics
    kp.kp_trace_reduce_hdr(dev, n_wg * W * cap, kp.make_hdr(n_wg, W, R + 1, cap),
                           torch.zeros(kp.kp_stats_bytes(n_wg, W, R + 1), dtype=torch.uint8, device="cuda"))
    st_buf = torch.zeros(kp.kp_stats_bytes(n_wg, W, R + 1), dtype=torch.uint8, device="cuda")
    kp.kp_trace_reduce_hdr(dev, n_wg * W * cap, kp.make_hdr(n_wg, W, R + 1, cap), st_buf)
    torch.cuda.synchronize()
    st = kp.parse_stats(st_buf)
    assert st["status"] == 1 and st["n_pairs"] == 0


def test_repeated_calls_are_deterministic(kp, oracle_mod):
    from tests.gpu_util import gpu_decode_bytes

    raw, _ = inputs.gen_trace(inputs.spec_decode_standalone(19))
    dev = torch.from_numpy(raw.view(np.int32)).cuda()
    first = gpu_decode_bytes(raw, dev_raw=dev)
    for _ in range(3):
        assert np.array_equal(first, gpu_decode_bytes(raw, use_hdr=True, dev_raw=dev))


def test_decode_workload_full_size(kp, oracle_mod):
    """The benchmark's decode workload at its full size (2^28 records, 16384 workgroups x 8 waves x
    2048 records, 16 regions) in the launch configuration bench.py times (kp_trace_reduce_hdr,
    kp_trace_pairs_hdr, kp_trace_waits_hdr and kp_pairs_stages): the whole statistics block, every
    timeline row, the whole waits block and the whole stage table, bit for bit."""
    import os

    spec = inputs.spec_decode_standalone(28)
    raw, _ = inputs.gen_trace(spec)
    n = spec.n_slots
    dev_raw = torch.from_numpy(raw.view(np.int32)).cuda()
    hdr = kp.make_hdr(spec.n_wg, spec.waves, spec.n_regions, spec.cap_wave)
    out = torch.full((kp.kp_stats_bytes(spec.n_wg, spec.waves, spec.n_regions),), 0xAB, dtype=torch.uint8, device="cuda")
    kp.kp_trace_reduce_hdr(dev_raw, n, hdr, out)
    rows = torch.full((kp.kp_pairs_bytes(spec.n_wg, spec.waves, spec.waves * spec.cap_wave),), 0xA5, dtype=torch.uint8,
                      device="cuda")
    kp.kp_trace_pairs_hdr(dev_raw, n, hdr, rows)
    waits = torch.full((kp.kp_waits_bytes(spec.n_wg, spec.waves, spec.n_regions),), 0x5A, dtype=torch.uint8, device="cuda")
    kp.kp_trace_waits_hdr(dev_raw, n, hdr, waits)
    max_iter = 64
    stages = torch.full((kp.kp_stages_bytes(spec.n_wg, spec.n_regions, max_iter),), 0x3C, dtype=torch.uint8, device="cuda")
    kp.kp_pairs_stages(rows, spec.n_wg, spec.waves, spec.waves * spec.cap_wave, spec.n_regions, max_iter, stages)
    torch.cuda.synchronize()
    from tests.gpu_util import assert_stats_equal

    want = oracle_mod.decode_bytes(raw, min(16, os.cpu_count() or 1))
    assert_stats_equal(want, out.cpu().numpy(), oracle_mod)
    st = kp.parse_stats(out)
    assert st["n_slots_valid"] == n and st["n_overlap_wgs"] == spec.n_wg and st["n_invalid"] == 0
    del out, want
    want_rows = oracle_mod.pairs_raw(raw, fill=0xA5)
    got_rows = rows.cpu().numpy()
    assert np.array_equal(want_rows, got_rows)
    want_stages = oracle_mod.stages_raw(want_rows, spec.n_wg, spec.waves, spec.cap_wave, spec.n_regions, max_iter)
    assert np.array_equal(want_stages, stages.cpu().numpy())
    del want_rows, got_rows, want_stages
    assert np.array_equal(oracle_mod.waits_raw(raw), waits.cpu().numpy())


def test_events_around_the_main_kernel(kp, oracle_mod):
    """kp_trace_reduce_hdr_events: the same statistics, and two events of the caller's recorded around the
    replay kernel (their distance is below that of events around the whole call)."""
    from tests.gpu_util import assert_stats_equal

    raw, _ = inputs.gen_trace(inputs.spec_decode_standalone(20))
    n_wg, W, R, cap = (int(x) for x in raw[2:6])
    dev = torch.from_numpy(raw.view(np.int32)).cuda()
    out = torch.full((kp.kp_stats_bytes(n_wg, W, R),), 0x5A, dtype=torch.uint8, device="cuda")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    torch.cuda.synchronize()
    hdr = kp.make_hdr(n_wg, W, R, cap)
    ev[0].record()
    kp.kp_trace_reduce_hdr_events(dev, n_wg * W * cap, hdr, out, ev[1], ev[2])
    ev[3].record()
    torch.cuda.synchronize()
    assert_stats_equal(oracle_mod.decode_bytes(raw, 8), out.cpu().numpy(), oracle_mod)
    assert 0.0 < ev[1].elapsed_time(ev[2]) <= ev[0].elapsed_time(ev[3])
    kp.kp_trace_reduce_hdr_events(dev, n_wg * W * cap, hdr, out, None, None)   # events are optional
    torch.cuda.synchronize()
    with pytest.raises(ValueError):
        kp.kp_trace_reduce_hdr_events(dev, n_wg * W * cap, hdr, out, torch.cuda.Event(enable_timing=True), None)


def test_sequence_numbers_that_wrap(kp, oracle_mod):
    """Waves that wrote more than 2^20 records: the 20-bit sequence numbers wrap around inside the surviving
    tail of the ring (a generated trace with a multiple of the ring size added to every sequence number and
    to the waves' record counts)."""
    W, cap, n_wg = 8, 2048, 5
    spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=16, cap_wave=cap, total_per_wave=2600, total_var=400,
                            seed=32, dist="exp", p0=30.0, gap_max=4, phase_max=10, p_orphan=0.01, p_swap=0.002)
    raw, _ = inputs.gen_trace(spec)
    shift = (1 << 20) - cap
    raw = raw.copy()
    hdrs = raw[16:16 + 32 * n_wg].reshape(n_wg, 32)
    assert (hdrs[:, 8:8 + W] > cap).all()
    hdrs[:, 8:8 + W] += shift
    recs = raw[16 + 32 * n_wg:].reshape(-1, 2)
    recs[:, 0] = (recs[:, 0] & 0xFFF00000) | ((recs[:, 0] + shift) & 0xFFFFF)
    check(raw, oracle_mod)
    check(raw, oracle_mod, use_hdr=True)


@pytest.mark.parametrize("W,R,cap", [(12, 32, 256), (8, 16, 512), (4, 3, 128), (2, 17, 64), (16, 20, 1024), (8, 5, 2048), (8, 40, 256)])
def test_records_of_one_clock(kp, oracle_mod, W, R, cap):
    """Few clocks, pairs of length 0 and regions inside regions: the records of one clock come in any order out of the
    counting sort, and the region-pair sums must not depend on it."""
    rng = np.random.default_rng(R)
    wgs = []
    for _ in range(20):
        waves = []
        for _w in range(W):
            wave, t = [], 0
            while len(wave) < cap - 6:
                t += int(rng.choice([0, 0, 0, 300]))
                order = [int(x) for x in rng.permutation(R)[:3]]
                for phase, regions in ((S, order), (E, order[::-1])):
                    for r in regions:
                        wave.append((phase, r, t))
                        t += int(rng.choice([0, 0, 0, 0, 7]))
            waves.append(wave)
        wgs.append(inputs.events_to_wg(waves, cap, flush=False))
    raw = inputs.encode_trace(wgs, W, R, cap, rec_cost=0)
    for _ in range(3):
        check(raw, oracle_mod, use_hdr=True)


@pytest.mark.parametrize("W,R,cap", [(4, 3, 1024), (2, 7, 1024), (8, 16, 2048), (16, 5, 1024), (1, 2, 16384)])
def test_a_long_gap_between_short_stretches(kp, oracle_mod, W, R, cap):
    """Records every few hundred ticks and one stretch of 2^21 ticks or more, which only the hardware wave that holds it
    adds up record by record: at every place of the sequence, and behind the last record, with regions open around it."""
    rng = np.random.default_rng(W * R)
    wgs = []
    for place in (0.0, 0.1, 0.35, 0.5, 0.77, 0.95, 1.0):
        waves = []
        for w in range(W):
            k = np.arange(cap - 4)
            t = k * 600 + rng.integers(0, 600, cap - 4) + np.where(k >= place * cap, (1 << 21) + 5000, 0)
            region = rng.integers(0, R - 1, cap) if w else np.zeros(cap, int)
            inner = [(E if i % 2 else S, int(region[i // 2]), int(t[i])) for i in k]
            waves.append([(S, R - 1, 0)] + inner + [(E, R - 1, int(t[-1]) + 7 * w)])
        wg = inputs.events_to_wg(waves, cap, flush=False)
        wg["t_end"] += (1 << 21) if place == 1.0 else 0
        wgs.append(wg)
    raw = inputs.encode_trace(wgs, W, R, cap, rec_cost=2)
    check(raw, oracle_mod, use_hdr=True)


def test_headers_read_back_by_several_threads(kp, oracle_mod):
    """Every thread reads the headers of its own traces back, on a stream of its own with other work ahead (one read longer
    than the host looks for it) or without."""
    import threading

    failures = []

    def replay(i):
        try:
            stream = torch.cuda.Stream()
            busy = torch.randn(4096, 4096, device="cuda")
            for turn in range(6):
                raw = inputs.messy_trace(900 + 10 * i + turn, n_wg=3 + turn, waves=1 + i, n_regions=2 + i, cap_wave=32)
                n_wg, W, R, cap = (int(x) for x in raw[2:6])
                dev = torch.from_numpy(raw.view(np.int32)).cuda()
                out = torch.zeros(kp.kp_stats_bytes(n_wg, W, R), dtype=torch.uint8, device="cuda")
                torch.cuda.synchronize()
                with torch.cuda.stream(stream):
                    for _ in range(4 if turn % 2 else 0):
                        busy = busy @ busy * 1e-4
                    kp.kp_trace_reduce(dev, n_wg * W * cap, out)
                stream.synchronize()
                if not np.array_equal(oracle_mod.decode_bytes(raw), out.cpu().numpy()):
                    failures.append((i, turn))
        except Exception as e:  # noqa: BLE001
            failures.append((i, repr(e)))

    threads = [threading.Thread(target=replay, args=(i,)) for i in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures, failures


def test_a_trace_in_pinned_host_memory(kp, oracle_mod):
    """Memory of another kind than the device's, which the C ABI takes: its header comes by the runtime's copy."""
    raw = inputs.messy_trace(950, n_wg=5, waves=3, n_regions=4, cap_wave=32)
    n_wg, W, R, cap = (int(x) for x in raw[2:6])
    pinned = torch.empty(raw.size, dtype=torch.int32, pin_memory=True)
    pinned.copy_(torch.from_numpy(raw.view(np.int32)))
    out = torch.zeros(kp.kp_stats_bytes(n_wg, W, R), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert kp.lib().kp_trace_reduce(pinned.data_ptr(), n_wg * W * cap, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert np.array_equal(oracle_mod.decode_bytes(raw), out.cpu().numpy())


def test_a_thread_that_read_a_header_ends_during_a_capture(kp, oracle_mod):
    """The end of such a thread is no concern of another thread's capture."""
    import threading

    raw = inputs.messy_trace(960, n_wg=5, waves=3, n_regions=4, cap_wave=32)
    n_wg, W, R, cap = (int(x) for x in raw[2:6])
    n, dev = n_wg * W * cap, torch.from_numpy(raw.view(np.int32)).cuda()
    outs = [torch.zeros(kp.kp_stats_bytes(n_wg, W, R), dtype=torch.uint8, device="cuda") for _ in range(2)]
    hdr = kp.make_hdr(n_wg, W, R, cap, int(raw[6]), int(raw[7]))
    kp.kp_trace_reduce_hdr(dev, n, hdr, outs[0])
    torch.cuda.synchronize()
    read, end = threading.Event(), threading.Event()

    def reader():
        kp.kp_trace_reduce(dev, n, outs[1])
        torch.cuda.synchronize()
        read.set()
        end.wait(30)

    thread = threading.Thread(target=reader)
    thread.start()
    assert read.wait(30)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kp.kp_trace_reduce_hdr(dev, n, hdr, outs[0])
        end.set()
        thread.join()
        kp.kp_trace_reduce_hdr(dev, n, hdr, outs[0])
    want = oracle_mod.decode_bytes(raw)
    assert np.array_equal(want, outs[1].cpu().numpy())
    for _ in range(3):
        outs[0].fill_(0x77)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(want, outs[0].cpu().numpy())


def restart_trace(seed, n_wg, W, R, cap, most):
    """All waves are in region 0 and restart it now and then: up to `most` of them end it and start it again on one tick, on
    which another wave may open or close a further region.  Two dozen workgroups, over and over: where in the clock-sorted
    sequence a tick lies differs from one to the next."""
    rng = np.random.default_rng(seed)
    distinct = []
    for i in range(min(n_wg, 24)):
        waves = [[(S, 0, 40 * w)] for w in range(W)]
        inner = [0] * W  # the further region a wave has open
        t = 40 * W
        for _ in range(i):
            t += 400
            if R > 1 and len(waves[i % W]) + 4 < cap:
                waves[i % W] += [(S, 1 + i % (R - 1), t), (E, 1 + i % (R - 1), t + 200)]
        for _ in range(200):
            t += 400
            able = [w for w in range(W) if inner[w] == 0 and len(waves[w]) + 5 <= cap]
            again = [int(w) for w in rng.permutation(able)[:int(rng.integers(1, most + 1))]]
            for w in again:
                waves[w] += [(E, 0, t), (S, 0, t)]
            other = int(rng.integers(0, W))
            if R > 1 and other not in again and rng.random() < 0.7 and (inner[other] or len(waves[other]) + 5 <= cap):
                r = inner[other] or int(rng.integers(1, R))
                waves[other].append((E if inner[other] else S, r, t))
                inner[other] = 0 if inner[other] else r
            if not able and not any(inner):
                break
        for w in range(W):
            t += 40
            waves[w] += ([(E, inner[w], t)] if inner[w] else []) + [(E, 0, t)]
            assert len(waves[w]) <= cap
        distinct.append(inputs.events_to_wg(waves, cap, flush=False))
    return inputs.encode_trace([distinct[i % len(distinct)] for i in range(n_wg)], W, R, cap, rec_cost=1)


# with up to 15 waves the counts of open waves have four bits per region; every number of threads and of records per lane
@pytest.mark.parametrize("n_wg,W,R,cap", [
    (40, 15, 2, 16), (40, 15, 16, 64), (40, 15, 2, 64), (40, 14, 3, 256), (40, 15, 16, 256),                    # four records per lane
    (260, 15, 2, 16), (450, 15, 2, 64), (450, 8, 3, 64), (450, 12, 16, 64), (260, 15, 3, 128), (260, 9, 16, 128),  # one wave, 128 threads
    (260, 12, 2, 256), (260, 15, 16, 256), (30, 15, 3, 512), (30, 8, 16, 1024), (30, 9, 2, 1024),               # 256, 512, 1024 threads
    (40, 16, 3, 64), (30, 16, 16, 1024), (30, 7, 3, 256),                                                        # five bits; counts that always fit
    (40, 15, 32, 64), (450, 15, 17, 64), (30, 12, 24, 256), (30, 16, 32, 256),                                   # more than 16 regions
    (30, 15, 40, 256), (300, 15, 40, 128), (30, 16, 100, 128)])                                                   # more than 32
def test_regions_that_restart_on_a_tick(kp, oracle_mod, n_wg, W, R, cap):
    """An END and the START of the same region in one wave on one clock: between the two of them a region is open in one wave more
    or fewer than the workgroup has, and neither the region nor its neighbours in the counts may be taken for open or closed."""
    for most in (1, 2, 8, W):
        check(restart_trace(most, n_wg, W, R, cap, most), oracle_mod, use_hdr=True)


@pytest.mark.parametrize("n_wg,W,R,cap", [
    (40, 4, 3, 16), (40, 8, 5, 64), (40, 4, 5, 128), (40, 2, 5, 512), (300, 2, 8, 32), (450, 8, 16, 64), (450, 2, 5, 128),
    (300, 8, 16, 128), (300, 4, 5, 1024), (30, 8, 16, 1024), (30, 16, 5, 1024), (30, 16, 20, 512), (30, 3, 40, 512)])
@pytest.mark.parametrize("dropped", [(1 << 20) - 7, 1 << 20, 3 << 20, (16 << 20) + 37, (5 << 20) - 200])
def test_long_captures(kp, oracle_mod, n_wg, W, R, cap, dropped):
    """Waves that dropped 2^20 records or more, or nearly so that seq wraps inside the ring: clean, and with records that name another
    wave: the one that a sum of the wave's place in the tag and the full record number would give, in whole rings and from the
    place on where seq wraps."""
    spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=R, cap_wave=cap, total_per_wave=2 * cap, total_var=cap // 2, seed=cap + W, dist="exp",
                            p0=30.0, gap_max=4, p_orphan=0.02, p_swap=0.002 if cap >= 128 else 0.0)
    raw, _ = inputs.gen_trace(spec)
    raw = raw.copy()
    heads = raw[16:16 + 32 * n_wg].reshape(n_wg, 32)
    slots = raw[16 + 32 * n_wg:].reshape(n_wg, W, cap, 2)
    number = slots[..., 0] & np.uint32(0xFFFFF)
    shift = dropped - dropped % cap  # (a record stays in its slot)
    assert (heads[:, 8:8 + W] > cap).all() and int(number.max()) + shift < 1 << 32
    heads[:, 8:8 + W] += np.uint32(shift)
    number = number + np.uint32(shift)
    slots[..., 0] = (slots[..., 0] & np.uint32(0xFFF00000)) | (number & np.uint32(0xFFFFF))
    check(raw, oracle_mod, use_hdr=True)
    for wg in range(0, n_wg, 2):
        for w in range(W) if wg % 6 == 0 else [wg // 2 % W]:
            other = np.uint32(w) + (number[wg, w] >> np.uint32(20)) & np.uint32(0xF)
            slots[wg, w, :, 0] = (slots[wg, w, :, 0] & np.uint32(0xFF0FFFFF)) | (other << np.uint32(20))
    check(raw, oracle_mod, use_hdr=True)


@pytest.mark.parametrize("n_wg,W,R,cap", [(40, 2, 3, 256), (40, 4, 5, 1024), (40, 8, 20, 512), (300, 2, 5, 1024), (300, 1, 16, 2048), (300, 4, 24, 1024),
                                          (130, 4, 16, 2048), (130, 8, 5, 2048), (130, 1, 20, 16384), (40, 8, 5, 64), (450, 2, 16, 512), (40, 3, 40, 512)])
@pytest.mark.parametrize("ends_round", [True, False])
def test_rings_written_further_than_the_header_says(kp, oracle_mod, n_wg, W, R, cap, ends_round):
    """A wave's count is 1 to 127 records short: as many slots of its ring hold records newer than the count covers, which are
    invalid, in the place of the oldest that it does.  The overrun ends at a multiple of 128 slots, or anywhere."""
    spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=R, cap_wave=cap, total_per_wave=3 * cap if ends_round else 3 * cap + cap // 3,
                            total_var=0 if ends_round else cap // 2, seed=cap + W, dist="exp", p0=30.0, gap_max=4, p_orphan=0.02)
    raw, _ = inputs.gen_trace(spec)
    raw = raw.copy()
    heads = raw[16:16 + 32 * n_wg].reshape(n_wg, 32)
    assert not ends_round or (heads[:, 8:8 + W] == 3 * cap).all()
    for wg in range(n_wg):
        if wg % 10 != 9:
            heads[wg, 8 + wg % W] -= np.uint32([1, 2, 3, 31, 64, 65, 100, 126, 127][wg % 10])
    check(raw, oracle_mod, use_hdr=True)
