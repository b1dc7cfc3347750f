"""The workloads on which this library's speed is measured.

A program that profiles a kernel region by region does two things with the library: it runs the recording
targets (GEMM, attention), with the record sites on and, for the overhead figure, off; and it replays the
traces (statistics, timeline rows, asynchronous waits, stage table and critical path).  The cases below are
those calls from the smallest problem on which the method is tried out to the largest it is quoted on.

Kinds of case, each with the sizes it takes:
  gemm      C = A B, bf16, m x n x k, in one of the record modes below
  attention O = softmax(scale Q K^T) V, bf16, [b, h, s, 128], causal or not, same modes
  reduce    statistics block of a trace
  timeline  one row per paired START/END
  waits     END-before-barrier / START-after-barrier gaps
  path      timeline rows -> stage table -> critical path, the three calls in a row

What a recording writes besides its result is returned as the tags of its records and the record counts; the
clock values next to the tags are measurements and differ from run to run.
"""
import math

import torch

import paper_2505_21661_amd as kp

# record modes: bits of region_mask next to the regions themselves
MODES = {
    "off": 0,                               # the uninstrumented kernel
    "all": 0,                               # every region, ring in LDS, one stream per wave
    "staged": kp.KP_MASK_PHASES,            # large-tile GEMM: five regions, the stages of a K step apart
    "staged_off": kp.KP_MASK_PHASES,        # the same schedule without record sites
    "groups": kp.KP_MASK_WAVE_GROUP,        # one stream per four waves
    "realtime": kp.KP_MASK_REALTIME,        # constant-rate clock
    "flush": kp.KP_MASK_FLUSH,              # ring copied out whenever it is full
    "collab": kp.KP_MASK_COLLAB,            # 64-lane stores, hardware ids
}


def listed():
    return [
        # the smallest recorded GEMM: tried out first, 16 workgroups, launch latency counts
        {"name": "gemm_small_recorded", "kind": "gemm", "m": 256, "n": 256, "k": 256, "mode": "all", "ring": 512},
        # sizes off the 256 grid, as odd model dimensions give them: the 64x64 tile, sites off
        {"name": "gemm_ragged_plain", "kind": "gemm", "m": 2112, "n": 1984, "k": 2080, "mode": "off", "ring": 0},
        # the problem the recording overhead is quoted on, default schedule, recorded
        {"name": "gemm_large_recorded", "kind": "gemm", "m": 4096, "n": 4096, "k": 4096, "mode": "all", "ring": 4096},
        # stage-by-stage K step with its five regions, on a matrix that is not square
        {"name": "gemm_staged_recorded", "kind": "gemm", "m": 2048, "n": 4096, "k": 4096, "mode": "staged", "ring": 4096},
        # one short sequence, few heads: fewer workgroups than compute units
        {"name": "attention_short_plain", "kind": "attention", "b": 1, "h": 12, "s": 1152, "causal": False, "mode": "off", "ring": 0},
        # the attention problem of the overhead figure, ring of 1024 records that wraps
        {"name": "attention_large_recorded", "kind": "attention", "b": 4, "h": 32, "s": 4096, "causal": True, "mode": "all", "ring": 1024},
        # trace of the smallest recorded GEMM's kind: 12288 records
        {"name": "reduce_small", "kind": "reduce", "wgs": 64, "waves": 4, "cap": 128, "regions": 3, "fill": "short", "host_header": True},
        # trace of one large recorded GEMM, header read back from the device
        {"name": "reduce_one_kernel", "kind": "reduce", "wgs": 256, "waves": 8, "cap": 512, "regions": 5, "fill": "wrapped", "host_header": False},
        # the largest trace replayed: 2^28 records, 0.1 % of them out of order
        {"name": "reduce_large", "kind": "reduce", "wgs": 16384, "waves": 8, "cap": 2048, "regions": 16, "fill": "full", "host_header": True},
        # many regions and long rings: what the LDS-resident decoder does not take
        {"name": "reduce_many_regions", "kind": "reduce", "wgs": 1024, "waves": 8, "cap": 4096, "regions": 48, "fill": "wrapped", "host_header": True},
        # three waves, rings partly filled
        {"name": "waits_odd", "kind": "waits", "wgs": 9000, "waves": 3, "cap": 1024, "regions": 7, "fill": "short", "host_header": True},
        # rows, stage table and critical path of a long capture
        {"name": "path_large", "kind": "path", "wgs": 4096, "waves": 8, "cap": 2048, "regions": 16, "fill": "full", "host_header": True},
    ]


def draw(rng):
    def spread(lo, hi):  # evenly over the logarithm
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def recorded(modes, rings):
        mode = rng.choice(modes)
        return {"mode": mode, "ring": 0 if mode in ("off", "staged_off") else rng.choice(rings)}

    kind = rng.choice(["gemm", "gemm", "attention", "attention", "reduce", "reduce", "reduce", "timeline", "waits", "path"])
    modes = ["off", "all", "all", "groups", "realtime", "flush", "collab"]
    if kind == "gemm":
        m, n, k = 64 * spread(1, 64), 64 * spread(1, 64), 32 * spread(1, 128)
        if rng.random() < 0.5:  # on the 256 grid; from 16 tiles on it is the large tile that takes it
            m, n, k = 256 * -(-m // 256), 256 * -(-n // 256), 64 * -(-k // 64)
            if (m // 256) * (n // 256) >= 16:
                modes = modes + ["staged", "staged_off"]
        return {"kind": kind, "m": m, "n": n, "k": k, **recorded(modes, [512, 1024, 2048])}
    if kind == "attention":
        b, h, s = rng.randint(1, 4), spread(1, 32), 128 * spread(1, 32)
        causal = b * h * s * s > 1 << 30 or rng.random() < 0.5
        return {"kind": kind, "b": b, "h": h, "s": s, "causal": causal, **recorded(modes, [512, 1024, 2048])}
    waves = rng.choice([1, 2, 3, 4, 5, 7, 8, 8, 12, 16])
    regions = rng.choice([1, 2, 3, 4, 5, 7, 11, 16, 16, 24, 32])
    cap = 1 << rng.randint(4, 14 - (waves - 1).bit_length())
    slots = 1 << rng.randint(12, 25 if kind == "path" else 26)
    if kind == "reduce" and rng.random() < 0.3:  # outside what the LDS-resident decoder takes
        regions = rng.choice([16, 40, 64, 100, 128])
        cap = 1 << rng.randint(8 if regions > 32 else 15 - (waves - 1).bit_length(), 17 - (waves - 1).bit_length())
        if regions <= 32 and waves * cap <= 16384:
            cap *= 2
        slots = 1 << rng.randint(14, 24)
    wgs = max(1, min(65536, slots // (waves * cap)) - rng.randint(0, 3))
    return {"kind": kind, "wgs": wgs, "waves": waves, "cap": cap, "regions": regions,
            "fill": rng.choice(["full", "short", "wrapped"]), "host_header": rng.random() < 0.7}


# ---- recorded kernels ------------------------------------------------------------------------------------

def _recording(case, n_wg, waves, regions, records):
    """region_mask, trace buffer and the view of its records that a recording defines.  records: what a wave
    writes; the slots past them hold unspecified bytes and are left out of the view."""
    mode = case["mode"]
    mask = MODES[mode]
    if mode in ("off", "staged_off"):
        return {"mask": mask, "trace": None, "cap": 0, "defined": []}
    mask |= (1 << regions) - 1
    streams = waves // 4 if mode == "groups" else waves
    cap = case["ring"]
    cap_wave = cap // streams
    trace = torch.zeros(kp.kp_trace_bytes(n_wg, streams, cap), dtype=torch.uint8, device="cuda")
    words = trace.view(torch.int32)
    counts = words[16:16 + 32 * n_wg].view(n_wg, 32)[:, 8:24]
    tags = words[16 + 32 * n_wg:].view(n_wg, streams, cap_wave, 2)[:, :, :min(cap_wave, records), 0]
    return {"mask": mask, "trace": trace, "cap": cap, "defined": [counts, tags]}


def _gemm(case, seed):
    m, n, k = case["m"], case["n"], case["k"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    a = torch.randn(m, k, generator=gen, device="cuda").to(torch.bfloat16)
    b = torch.randn(k, n, generator=gen, device="cuda").to(torch.bfloat16)
    c = torch.zeros(m, n, dtype=torch.bfloat16, device="cuda")
    n_wg, waves, regions = kp.kp_gemm_launch_shape(m, n, k)
    if case["mode"] == "staged":
        regions = 5
    # two records per region and K step; the large tile's epilogue region comes once
    records = 2 * (regions - 1) * (k // 64) + 2 if waves == 8 else 2 * regions * (k // 32)
    rec = _recording(case, n_wg, waves, regions, records)

    def call():
        kp.kp_gemm_instrumented(a, b, c, m, n, k, rec["mask"], rec["trace"], rec["cap"])
        return [c] + rec["defined"]

    return call


def _attention(case, seed):
    b, h, s, causal = case["b"], case["h"], case["s"], case["causal"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn(b, h, s, 128, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    o = torch.zeros_like(q)
    n_wg, waves, regions = kp.kp_attn_launch_shape(b, h, s, 128)
    blocks = s // 128
    rec = _recording(case, n_wg, waves, regions, 12 * blocks)
    if causal and rec["trace"] is not None:
        # query block i (0 the first; workgroups are numbered head by head, last block first) writes 12 (i + 1)
        # records per wave: the blocks that fill as many slots as the longest one does
        counts, tags = rec["defined"]
        filled = sum(1 for i in range(blocks) if 12 * (i + 1) >= tags.shape[2])
        rec["defined"] = [counts, tags.view(b * h, blocks, *tags.shape[1:])[:, :filled]]
    scale = 1.0 / math.sqrt(128.0)

    def call():
        kp.kp_attn_instrumented(q, k, v, o, b, h, s, 128, causal, scale, rec["mask"], rec["trace"], rec["cap"])
        return [o] + rec["defined"]

    return call


# ---- traces -------------------------------------------------------------------------------------------------

def _trace(case, seed):
    """A raw trace in device memory: per wave the regions follow one another, lognormal(6, 1) durations, gaps of
    1..32 ticks, about 1 % of the records are STARTs without END; full rings have 0.1 % of their slots out of place."""
    wgs, waves, cap, regions, fill = case["wgs"], case["waves"], case["cap"], case["regions"], case["fill"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    hdr = kp.make_hdr(wgs, waves, regions, cap, rec_cost=20)
    raw = torch.zeros(kp.kp_trace_bytes(wgs, waves, waves * cap), dtype=torch.uint8, device="cuda")
    raw[:64] = torch.frombuffer(bytearray(bytes(hdr)), dtype=torch.uint8).cuda()
    heads = raw[64:64 + 128 * wgs].view(torch.int64).view(wgs, 16)
    records = raw[64 + 128 * wgs:].view(torch.int32).view(wgs * waves, cap, 2)
    longest = cap // 2 + cap // 16 + 4  # region instances of a wave: enough for a whole ring
    step = max(1, (1 << 24) // (longest * waves)) * waves

    def ints(lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=gen, device="cuda")

    end_of_wg = []
    total_of_wave = []
    for s0 in range(0, wgs * waves, step):
        rows = min(step, wgs * waves - s0)
        if fill == "full":
            total = torch.full((rows, 1), cap, dtype=torch.int64, device="cuda")
        elif fill == "short":
            total = ints(cap // 4, cap + 1, rows, 1)
        else:
            total = cap + ints(0, 3 * cap, rows, 1)
        held = total.clamp(max=cap)
        first = total - held
        z = torch.randn(rows, longest, generator=gen, device="cuda")
        dur = torch.exp(6.0 + z).long().clamp(min=1)
        gap = ints(1, 33, rows, longest)
        single = torch.rand(rows, longest, generator=gen, device="cuda") < 2.0 / 101.0
        count = 2 - single.long()
        rank = count.cumsum(1) - count
        offset = ints(0, regions, rows, 1)
        if fill == "wrapped":  # the ring may begin with an END whose START is gone
            rank -= ints(0, 2, rows, 1)
        advance = dur + gap
        begin = advance.cumsum(1) - advance + ints(0, 4096, rows, 1)
        region = (torch.arange(longest, device="cuda") + offset) % regions
        wave = ((torch.arange(rows, device="cuda") + s0) % waves).unsqueeze(1)
        rest = (region << 24) | (wave << 20)
        here = records[s0:s0 + rows]
        flat = here.view(rows * cap, 2)
        base = torch.arange(rows, device="cuda").unsqueeze(1) * cap
        for is_end in (0, 1):
            r = rank + is_end
            keep = (r >= 0) & (r < held)
            if is_end:
                keep &= ~single
            seq = first + r
            at = (base + (seq & (cap - 1)))[keep]
            flat[at, 0] = ((rest | (seq & 0xFFFFF)) - (is_end << 31))[keep].to(torch.int32)
            flat[at, 1] = (begin + dur * is_end)[keep].to(torch.int32)
        if fill == "full" and cap >= 16:  # one pair of slots in every hundred or so blocks of 16 trades places
            block = here.view(rows * (cap // 16), 16, 2)
            hit = (torch.rand(block.shape[0], generator=gen, device="cuda") < 0.008).nonzero().squeeze(1)
            x = ints(0, 8, hit.numel())
            y = x + ints(1, 9, hit.numel())
            kept = block[hit, x].clone()
            block[hit, x] = block[hit, y]
            block[hit, y] = kept
        end_of_wg.append((begin + dur).amax(1).view(-1, waves).amax(1))
        total_of_wave.append(total.view(-1, waves))
    t0 = ints(1 << 30, 1 << 40, wgs)
    heads[:, 0] = torch.arange(wgs, device="cuda")
    heads[:, 1] = t0
    heads[:, 2] = t0 + torch.cat(end_of_wg) + 64
    heads.view(torch.int32)[:, 8:8 + waves] = torch.cat(total_of_wave).to(torch.int32)
    return hdr, raw


def _iterations(case):
    return max(1, min(64, case["cap"] // (2 * case["regions"]) + 1))


def _replay(case, seed):
    hdr, raw = _trace(case, seed)
    wgs, waves, cap, regions, host = case["wgs"], case["waves"], case["cap"], case["regions"], case["host_header"]
    n = wgs * waves * cap

    def block(size):
        return torch.zeros(size, dtype=torch.uint8, device="cuda")

    if case["kind"] == "reduce":
        out = block(kp.kp_stats_bytes(wgs, waves, regions))
        result = [out.view(torch.int64)]

        def call():
            if host:
                kp.kp_trace_reduce_hdr(raw, n, hdr, out)
            else:
                kp.kp_trace_reduce(raw, n, out)
            return result
    elif case["kind"] == "waits":
        out = block(kp.kp_waits_bytes(wgs, waves, regions))
        result = [out.view(torch.int64)]

        def call():
            if host:
                kp.kp_trace_waits_hdr(raw, n, hdr, out)
            else:
                kp.kp_trace_waits(raw, n, out)
            return result
    else:
        pairs = block(kp.kp_pairs_bytes(wgs, waves, waves * cap))
        result = [pairs.view(torch.int32)]
        more = case["kind"] == "path"
        its = _iterations(case)
        if more:
            stages = block(kp.kp_stages_bytes(wgs, regions, its))
            paths = block(kp.kp_critical_bytes(wgs, regions))
            result += [stages.view(torch.int32), paths.view(torch.int64)]

        def call():
            if host:
                kp.kp_trace_pairs_hdr(raw, n, hdr, pairs)
            else:
                kp.kp_trace_pairs(raw, n, pairs)
            if more:
                kp.kp_pairs_stages(pairs, wgs, waves, waves * cap, regions, its, stages)
                kp.kp_stages_critical(stages, wgs, regions, its, paths)
            return result
    return call


def prepare(case, seed):
    """Inputs, output buffers and (for the recording kernels) the trace buffer of one call."""
    make = {"gemm": _gemm, "attention": _attention}.get(case["kind"], _replay)
    return make(case, seed)


def run(state):
    return state()


def work(case):
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 2 * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    if kind == "attention":
        b, h, s = case["b"], case["h"], case["s"]
        return {"bytes": 8 * b * h * s * 128, "flops": 4 * b * h * s * s * 128 // (2 if case["causal"] else 1)}
    wgs, waves, cap, regions = case["wgs"], case["waves"], case["cap"], case["regions"]
    share = {"full": 1.0, "short": 0.625, "wrapped": 1.0}[case["fill"]]  # of the slots that hold a record
    read = 128 * wgs + 8 * share * wgs * waves * cap
    rows = 16 * 0.99 * share * wgs * waves * cap / 2
    if kind in ("reduce", "waits"):
        return {"bytes": int(read + 16 * wgs * waves * regions), "flops": 0}
    if kind == "timeline":
        return {"bytes": int(read + rows), "flops": 0}
    table = 16 * wgs * regions * _iterations(case)
    return {"bytes": int(read + 2 * rows + 2 * table + 32 * wgs), "flops": 0}


def tolerance(case):
    # bf16 results of fp32 sums.  Against the same in 64 bits the GEMM is off by 1.7e-3 (the rounding of its
    # results; 0.4 % at most in one value), the attention by 1.9e-3 to 2.3e-3 (the same and the rounding of the
    # probabilities; 1 % to 2.5 %); four times that.
    if case["kind"] == "gemm":
        return {"rel": 7e-3, "max": 0.016}
    if case["kind"] == "attention":
        return {"rel": 9e-3, "max": 0.1}
    return "exact"  # integers
