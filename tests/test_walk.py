"""Walk launches (stream mode, AUTO fusion): a whole operation in one launch.

Sizes sit where the launch changes shape: one lane group per vector or several
(2, 4: 256 lanes; 8, 16: 64 per group), a remainder of a group's positions,
truncated parts, chunks that fill a workgroup or share one, a partial last
vector, the smallest chunk and the largest rank count a walk is taken for and
the first beyond; which launch ran is asserted.  Bar: the same bits as the CPU
oracle's PAT order, and as the step kernels (fusion off) on the same inputs.
"""

import os
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

import synth
from oracle import native
from paper_2506_20252_amd import build as B
from paper_2506_20252_amd import pat

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TORCH = {"int32": torch.int32, "float32": torch.float32, "bfloat16": torch.bfloat16}
DIST = {"int32": "int32_pm2p20", "float32": "f32_normal", "bfloat16": "bf16_normal"}
WIDTH = {"int32": np.uint32, "float32": np.uint32, "bfloat16": np.uint16}


def bits(t):
    if t.dtype == torch.bfloat16:
        return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    return t.contiguous().cpu().numpy().view(np.uint32)


def rows(n, elems, dtype, layout):
    """N rows of `elems` elements: rows of one tensor, the same in descending
    order or shuffled, rows one element off a 16-byte boundary with a gap
    between them, or N allocations."""
    dev = torch.device("cuda:0")
    if layout in ("reversed", "shuffled"):
        r = rows(n, elems, dtype, "rows")[::-1]
        return r if layout == "reversed" else [r[i] for i in np.random.default_rng(n).permutation(n)]
    if layout == "separate":
        return [torch.empty(elems, dtype=TORCH[dtype], device=dev) for _ in range(n)]
    skew, gap = (1, 3) if layout == "skewed" else (0, 0)
    flat = torch.empty(n * (elems + gap) + skew, dtype=TORCH[dtype], device=dev)
    return [flat[skew + r * (elems + gap): skew + r * (elems + gap) + elems] for r in range(n)]


@pytest.fixture(scope="module")
def walk_asm(tmp_path_factory):
    if not os.path.exists(B.hipcc()):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / "walk.s"
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [B.hipcc(), *flags, "--cuda-device-only", "-S", "-I", os.path.join(ROOT, "include"),
           os.path.join(B.CSRC, "walk.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-2000:]
    return out.read_text()


def test_walk_kernels_keep_their_slots_in_registers(walk_asm):
    """No scratch memory, no packed fp32; VGPRs within what a workgroup's
    declared size allows (512 per SIMD lane: 128 at 1024 lanes)."""
    names = re.findall(r"^\s+\.name:\s+(\S+)$", walk_asm, re.M)
    priv = [int(x) for x in re.findall(r"^\s+\.private_segment_fixed_size:\s+(\d+)$", walk_asm, re.M)]
    vgpr = [int(x) for x in re.findall(r"^\s+\.vgpr_count:\s+(\d+)$", walk_asm, re.M)]
    assert names and len(names) == len(priv) == len(vgpr)
    assert not [(n, p) for n, p in zip(names, priv) if p]
    assert not [(n, v) for n, v in zip(names, vgpr) if v > 128]
    assert not re.search(r"\bv_pk_(add|mul|fma)_f32\b", walk_asm)


def test_overlap_checks_agree_with_the_definition():
    """Which pointer sets are refused, whatever layout check answers: receive
    buffers overlapping each other or another rank's send buffer, or their own
    other than in place.  Without a GPU an accepted call ends at the first
    device call (PAT_ERR_HIP), before any address is used."""
    if torch.cuda.is_available():
        pytest.skip("the addresses are made up: only where nothing can be launched")
    rng = np.random.default_rng(11)
    seen = set()
    for trial in range(4000):
        n, count, gather = int(rng.integers(2, 7)), int(rng.integers(1, 9)), bool(rng.integers(2))
        chunk = 4 * count
        sb, rb = (chunk, n * chunk) if gather else (n * chunk, chunk)
        base = 0x10000
        kind = int(rng.integers(4))
        gap = 4 * int(rng.integers(0, 3))
        big = max(sb, rb) + gap
        if kind == 0:  # rows side by side
            send = [base + r * (sb + gap) for r in range(n)]
            recv = [base + n * (sb + gap) + r * (rb + gap) for r in range(n)]
        elif kind == 1:  # in place
            outer = [base + r * big for r in range(n)]
            inner = [o + r * chunk for r, o in enumerate(outer)]
            send, recv = (inner, outer) if gather else (outer, inner)
        elif kind == 2:  # interleaved
            send = [base + r * (sb + rb + gap) for r in range(n)]
            recv = [s + sb for s in send]
        else:
            send = [base + 4 * int(rng.integers(0, 40 * n)) for _ in range(n)]
            recv = [base + 4 * int(rng.integers(0, 40 * n)) for _ in range(n)]
        if rng.integers(2):  # one pointer moved, or two swapped
            side = send if rng.integers(2) else recv
            i, j = (int(x) for x in rng.integers(0, n, 2))
            if rng.integers(2):
                side[i] += 4 * int(rng.integers(-3, 4))
            else:
                side[i], side[j] = side[j], side[i]
        ok = all(abs(recv[a] - recv[b]) >= rb for a in range(n) for b in range(a))
        for a in range(n):
            for b in range(n):
                if send[a] < recv[b] + rb and recv[b] < send[a] + sb:
                    alias = send[a] == recv[b] + b * chunk if gather else recv[b] == send[a] + a * chunk
                    ok = ok and a == b and alias
        if gather:
            st = pat.pat_allgather(send, recv, count, "float32", n, None)
        else:
            st = pat.pat_reducescatter(send, recv, count, "float32", pat.PAT_SUM, n, None)
        assert st == (pat.PAT_ERR_HIP if ok else pat.PAT_ERR_INVALID_ARGUMENT), (trial, kind, gather, send, recv)
        seen.add((kind, ok))
    assert seen >= {(0, True), (0, False), (1, True), (1, False), (2, True), (3, False)}


@pytest.mark.gpu
@pytest.mark.parametrize("n,count,dtype,layout", [
    (2, 16, "float32", "rows"), (3, 17, "bfloat16", "skewed"), (5, 1000, "int32", "separate"),
    (8, 4096, "float32", "rows"), (9, 4095, "bfloat16", "rows"), (16, 1024, "float32", "skewed"),
    (13, 70001, "bfloat16", "rows"), (64, 16384, "float32", "rows"), (65, 1023, "float32", "separate"),
    (128, 8191, "float32", "rows"), (127, 129, "bfloat16", "skewed"), (129, 2049, "int32", "rows"),
    (200, 520, "float32", "rows"), (257, 250, "bfloat16", "rows"), (300, 75, "float32", "skewed"),
    (513, 67, "float32", "rows"), (1000, 64, "float32", "rows"), (1025, 33, "bfloat16", "rows"),
    (2049, 16, "float32", "rows"), (4096, 18, "bfloat16", "rows"), (4097, 16, "bfloat16", "rows"),
    (31, 15, "float32", "rows"), (16, 64, "float32", "rows"), (32, 1024, "int32", "rows"),
    (128, 1024, "float32", "rows"), (64, 1024, "int32", "rows"), (1024, 64, "float32", "rows"), (20, 1000, "bfloat16", "reversed"), (64, 333, "float32", "shuffled"),
    (65, 40, "int32", "shuffled"), (300, 64, "float32", "reversed"), (600, 24, "bfloat16", "shuffled"),
    # pointer tables, chunks that share a workgroup: 1 to 5 groups in the last
    # part, whole and not; 4 and 2 lane groups, a whole tree
    (1027, 17, "float32", "shuffled"), (1029, 24, "int32", "shuffled"), (1031, 16, "float32", "reversed"),
    (1033, 20, "float32", "shuffled"), (1030, 17, "bfloat16", "shuffled"), (1034, 18, "bfloat16", "separate"),
    (200, 1320, "int32", "shuffled"), (300, 519, "bfloat16", "shuffled"), (250, 1058, "bfloat16", "shuffled"),
    (128, 4118, "bfloat16", "shuffled"), (7, 30, "float32", "shuffled"),
    # keyed read orders in workgroups of 256 lanes: 2 lane groups and nontemporal
    # accesses, 4 and cached ones
    (128, 4096, "float32", "rows"), (32, 2048, "float32", "rows"), (64, 4096, "int32", "rows"),
    # a chunk's own workgroups: many lane groups, pointer tables
    (300, 1024, "float32", "rows"), (300, 1000, "float32", "shuffled"), (100, 4096, "int32", "shuffled"),
    (257, 1000, "bfloat16", "shuffled"), (600, 260, "bfloat16", "reversed"),
])
@pytest.mark.parametrize("entry", ["reducescatter", "reducescatter_noalloc"])
def test_walked_reducescatter(n, count, dtype, layout, entry):
    seed = 0x3A1C + 7 * n + count
    print(f"[gpu] walk {entry} n={n} count={count} {dtype} {layout} seed={seed:#x}", file=sys.stderr, flush=True)
    st, info = pat.pat_plan_info(pat.PAT_REDUCESCATTER, n, count, dtype)
    if entry == "reducescatter_noalloc" and info["slot_bytes_total"] > 200 << 20:
        entry = "reducescatter"
    stream = torch.cuda.current_stream()
    pat.check(pat.pat_set_exec_mode("stream"))
    send, recv = rows(n, n * count, dtype, layout), rows(n, count, dtype, layout)
    for x in range(n):
        synth.fill(send[x], DIST[dtype], seed, x)
    S, R = pat.pointer_array(send), pat.pointer_array(recv)
    outs = []
    for fusion in ("auto", "off"):
        for r in recv:
            r.view(torch.uint8).fill_(0xA5)
        walks = fusion == "auto" and count >= 16 and n <= 4096
        pat.check(pat.pat_set_top_fusion(fusion))
        try:
            assert pat.pat_launch_info(pat.PAT_REDUCESCATTER, n, count, dtype)[1]["walk"] == walks
            pat.check(pat.pat_trace_start_as_run(10000))
            pat.check(getattr(pat, "pat_" + entry)(S, R, count, dtype, pat.PAT_SUM, n, stream))
            torch.cuda.synchronize()
            kinds = [k for _, _, k, _ in pat.pat_trace_read(10000)[1]]
        finally:
            pat.check(pat.pat_set_top_fusion("auto"))
        if entry == "reducescatter":  # the other one is not traced
            assert kinds == [2] if walks else kinds and 2 not in kinds
        outs.append(np.stack([bits(r) for r in recv]))
    np.testing.assert_array_equal(outs[0], outs[1])
    want = native.reducescatter(dtype, n, count, dist=DIST[dtype], seed=seed)["pat"]
    np.testing.assert_array_equal(outs[0], want.view(WIDTH[dtype]).reshape(n, count))


@pytest.mark.gpu
@pytest.mark.parametrize("coll", ["allgather", "reducescatter"])
def test_trace_as_run_times_the_walk(coll):
    """pat_trace_start_as_run records the launch an untraced call makes: one
    walk, with the bytes it needs."""
    n, count = 24, 32768
    print(f"[gpu] trace as run {coll} n={n} count={count}", file=sys.stderr, flush=True)
    pat.check(pat.pat_set_exec_mode("stream"))
    stream = torch.cuda.current_stream()
    s_elems, r_elems = (count, n * count) if coll == "allgather" else (n * count, count)
    send, recv = rows(n, s_elems, "float32", "rows"), rows(n, r_elems, "float32", "rows")
    for x in range(n):
        synth.fill(send[x], "f32_normal", 3, x)
    args = (count, "float32") if coll == "allgather" else (count, "float32", pat.PAT_SUM)
    pat.check(pat.pat_trace_start_as_run(3))
    for _ in range(3):
        pat.check(getattr(pat, "pat_" + coll)(send, recv, *args, n, stream))
    st, launches = pat.pat_trace_read(3)
    pat.check(st)
    assert [(b, k, s) for _, b, k, s in launches] == [(4.0 * count * n * (n + 1), 2, 0)] * 3
    assert all(ms > 0 for ms, _, _, _ in launches)


@pytest.mark.gpu
def test_walk_over_a_pointer_table_is_not_the_slower_path(monkeypatch):
    """Rows at no regular spacing, more ranks than a launch carries pointers
    for, chunks that share a workgroup: a walk takes no longer than the step
    schedule (0.8 of its time measured; 1.7 when a lane waited for its address
    before every group of loads).  Shortest of 5 rounds of 20 calls each."""
    n, count = 1025, 24
    print(f"[gpu] walk and steps timed n={n} count={count}", file=sys.stderr, flush=True)
    pat.check(pat.pat_set_exec_mode("stream"))
    stream = torch.cuda.current_stream()
    send, recv = rows(n, n * count, "float32", "shuffled"), rows(n, count, "float32", "shuffled")
    for s in send:
        s.zero_()
    S, R = pat.pointer_array(send), pat.pointer_array(recv)
    us = {"1": [], "0": []}
    for _ in range(6):
        for walk in us:
            monkeypatch.setenv("PAT_WALK", walk)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                pat.check(pat.pat_reducescatter(S, R, count, "float32", pat.PAT_SUM, n, stream))
            b.record()
            b.synchronize()
            us[walk].append(a.elapsed_time(b) * 50)
    walk, steps = (min(us[k][1:]) for k in ("1", "0"))  # the first round loads the kernels
    print(f"[gpu]   walk {walk:.1f} us, steps {steps:.1f} us", file=sys.stderr, flush=True)
    assert walk <= 1.2 * steps


@pytest.mark.gpu
@pytest.mark.parametrize("n,count,dtype,order", [
    (7, 1001, "float32", "rows"), (40, 203, "bfloat16", "rows"), (12, 64, "int32", "rows"),
    # keyed orders, 2 and 8 lane groups; pointer tables, chunks that share a
    # workgroup or fill their own; a whole tree in many workgroups
    (128, 4096, "float32", "rows"), (128, 1024, "int32", "rows"), (66, 33, "float32", "shuffled"),
    (100, 4099, "bfloat16", "shuffled"), (9, 500003, "float32", "rows"), (40, 77, "int32", "shuffled"),
])
def test_walked_reducescatter_in_place_and_special_values(n, count, dtype, order):
    """In place (rank r receives into its own chunk r), with infinities, NaN,
    negative zeros and subnormals among the inputs: the step kernels' bits
    (any NaN for a NaN), and send buffers otherwise untouched."""
    print(f"[gpu] walk in place n={n} count={count} {dtype} {order}", file=sys.stderr, flush=True)
    row = list(range(n))  # rank r's buffer is row row[r]
    if order == "shuffled":
        row = [int(x) for x in np.random.default_rng(n).permutation(n)]
    pat.check(pat.pat_set_exec_mode("stream"))
    stream = torch.cuda.current_stream()
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    src = torch.empty((n, n * count), dtype=TORCH[dtype], device="cuda:0")
    if dtype == "int32":
        src.random_(-(1 << 31), 1 << 31, generator=gen)
    else:
        src.normal_(generator=gen)
        for k, v in enumerate((float("inf"), float("-inf"), float("nan"), -0.0, 1e-40)):
            src[k % n, k::17] = v
        src[:, 3::29] = -0.0
    got = []
    for fusion in ("auto", "off"):
        send = src.clone()
        pat.check(pat.pat_set_top_fusion(fusion))
        try:
            pat.check(pat.pat_reducescatter([send[x] for x in row], [send[x, r * count:] for r, x in enumerate(row)],
                                            count, dtype, pat.PAT_SUM, n, stream))
            torch.cuda.synchronize()
        finally:
            pat.check(pat.pat_set_top_fusion("auto"))
        got.append(send)
    for r, x in enumerate(row):  # only chunk r of rank r's row may change
        for t in got:
            for part in (slice(0, r * count), slice((r + 1) * count, None)):
                assert torch.equal(t[x, part].view(torch.uint8), src[x, part].view(torch.uint8))
    a, b = (t.clone() for t in got)
    if dtype != "int32":
        assert torch.equal(a.isnan(), b.isnan())
        a[a.isnan()] = 0
        b[b.isnan()] = 0
    assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("path", ["steps", "walk over a table"])
def test_pointer_tables_of_queued_calls(path, monkeypatch):
    """Eleven calls on one plan, each with buffers of its own, queued behind
    work that takes longer than queueing them: the library's four staging sets
    come round again while earlier uploads are still pending, and every call
    must still find its own addresses."""
    n, count, calls = 70, 200, 11
    print(f"[gpu] queued calls n={n} count={count} {path}", file=sys.stderr, flush=True)
    if path == "steps":
        monkeypatch.setenv("PAT_WALK", "0")
    pat.check(pat.pat_set_exec_mode("stream"))
    stream = torch.cuda.current_stream()
    bufs = [(rows(n, n * count, "float32", "shuffled"), rows(n, count, "float32", "shuffled")) for _ in range(calls)]
    for k, (send, recv) in enumerate(bufs):
        for x in range(n):
            synth.fill(send[x], "f32_normal", 40 + k, x)
            recv[x].fill_(float("nan"))
    args = [(pat.pointer_array(send), pat.pointer_array(recv)) for send, recv in bufs]
    pat.check(pat.pat_reducescatter(*args[0], count, "float32", pat.PAT_SUM, n, stream))  # the plan is made
    bufs[0][1][0].fill_(float("nan"))
    busy = torch.zeros(1 << 28, device="cuda:0")
    torch.cuda.synchronize()
    for _ in range(50):  # about 20 ms
        busy.add_(1)
    for S, R in args:
        pat.check(pat.pat_reducescatter(S, R, count, "float32", pat.PAT_SUM, n, stream))
    torch.cuda.synchronize()
    for k, (_, recv) in enumerate(bufs):
        want = native.reducescatter("float32", n, count, dist="f32_normal", seed=40 + k)["pat"]
        np.testing.assert_array_equal(np.stack([bits(r) for r in recv]), want.view(np.uint32).reshape(n, count))


@pytest.mark.gpu
@pytest.mark.parametrize("n,count,dtype,layout", [
    (6, 1024, "int32", "rows"), (24, 1001, "bfloat16", "separate"), (128, 4096, "float32", "rows"),
    (70, 100, "float32", "shuffled"),
])
def test_captured_walks(n, count, dtype, layout):
    """The no-allocation entry point under graph capture, as a walk: addresses
    at a stride, in the launch, and in the library's table (after a call that
    put them there).  Replays between eager work and synchronizations, each on
    new inputs, give the eager call's bits."""
    print(f"[gpu] captured walk n={n} count={count} {dtype} {layout}", file=sys.stderr, flush=True)
    pat.check(pat.pat_set_exec_mode("stream"))
    assert pat.pat_launch_info(pat.PAT_REDUCESCATTER, n, count, dtype)[1]["walk"] == 1
    send, recv = rows(n, n * count, dtype, layout), rows(n, count, dtype, layout)
    eager = rows(n, count, dtype, "rows")
    S, R, E = (pat.pointer_array(b) for b in (send, recv, eager))
    for x in range(n):
        synth.fill(send[x], DIST[dtype], 1, x)
    stream = torch.cuda.current_stream()
    pat.check(pat.pat_reducescatter_noalloc(S, R, count, dtype, pat.PAT_SUM, n, stream))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        st = pat.pat_reducescatter_noalloc(S, R, count, dtype, pat.PAT_SUM, n, torch.cuda.current_stream())
    pat.check(st)
    for rep in range(4):
        for x in range(n):
            synth.fill(send[x], DIST[dtype], 100 + rep, x)
            recv[x].view(torch.uint8).fill_(0xA5)
        graph.replay()
        if rep % 2:
            torch.cuda.synchronize()
        pat.check(pat.pat_reducescatter(S, E, count, dtype, pat.PAT_SUM, n, stream))
        torch.cuda.synchronize()
        for x in range(n):
            np.testing.assert_array_equal(bits(recv[x]), bits(eager[x]))
        want = native.reducescatter(dtype, n, count, dist=DIST[dtype], seed=100 + rep)["pat"]
        np.testing.assert_array_equal(np.stack([bits(r) for r in recv]), want.view(WIDTH[dtype]).reshape(n, count))


@pytest.mark.gpu
@pytest.mark.parametrize("n,count,dtype", [
    (2, 1, "bfloat16"), (3, 1, "float32"), (5, 7, "bfloat16"), (9, 3, "int32"), (13, 1001, "bfloat16"),
    (24, 4096, "bfloat16"), (37, 999, "float32"), (64, 1023, "bfloat16"), (130, 33, "float32"),
    (300, 17, "bfloat16"), (300, 1024, "float32"), (1000, 63, "float32"), (1025, 2, "bfloat16"),
])
@pytest.mark.parametrize("layout", ["rows", "skewed", "separate", "inplace", "reversed", "shuffled"])
def test_walked_allgather(n, count, dtype, layout):
    """Every receive row is the concatenation: chunks smaller and larger than
    a vector and a tile, rows that start anywhere in a line, receivers that
    share a workgroup side by side or a period apart; nothing outside the rows
    changes."""
    print(f"[gpu] walk allgather n={n} count={count} {dtype} {layout}", file=sys.stderr, flush=True)
    dev = torch.device("cuda:0")
    pat.check(pat.pat_set_exec_mode("stream"))
    stream = torch.cuda.current_stream()
    skew, gap = {"skewed": (3, 5), "inplace": (1, 1)}.get(layout, (0, 0))
    whole = torch.empty(n * (n * count + gap) + skew, dtype=TORCH[dtype], device=dev).random_(0, 100)
    recv = [whole[skew + r * (n * count + gap): skew + r * (n * count + gap) + n * count] for r in range(n)]
    if layout in ("separate", "reversed", "shuffled"):
        recv = rows(n, n * count, dtype, layout)
    send = rows(n, count, dtype, "rows" if layout == "inplace" else layout)
    for x in range(n):
        synth.fill(send[x], DIST[dtype], 77 + n, x)
    want = torch.cat([s.clone() for s in send])
    if layout == "inplace":
        for x in range(n):
            recv[x][x * count:(x + 1) * count] = send[x]
        send = [recv[x][x * count:(x + 1) * count] for x in range(n)]
    mark = torch.ones(whole.numel(), dtype=torch.bool, device=dev)
    for r in range(n):
        mark[skew + r * (n * count + gap): skew + r * (n * count + gap) + n * count] = False
    outside = whole[mark].clone()
    pat.check(pat.pat_trace_start_as_run(10))
    pat.check(pat.pat_allgather(pat.pointer_array(send), pat.pointer_array(recv), count, dtype, n, stream))
    torch.cuda.synchronize()
    assert [k for _, _, k, _ in pat.pat_trace_read(10)[1]] == [2]  # a walk
    bad = [r for r in range(n) if not torch.equal(recv[r].view(torch.uint8), want.view(torch.uint8))]
    assert not bad, bad[:8]
    assert torch.equal(whole[mark], outside)


@pytest.mark.gpu
def test_walks_beyond_one_grid():
    """Operations of more workgroups than one grid takes (2^31 lanes) run as
    several launches: an all-gather into 40 GiB and a reduce-scatter of 2 ranks
    with more than 2^31 vectors, against plain torch."""
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    pat.check(pat.pat_set_exec_mode("stream"))
    pat.check(pat.pat_finalize())
    n, count = 200, 262144
    print(f"[gpu] walk allgather n={n} count={count} float32 (40 GiB)", file=sys.stderr, flush=True)
    send = torch.randn(n, count, device=dev)
    recv = torch.empty(n, n * count, device=dev)
    pat.check(pat.pat_allgather(list(send), list(recv), count, "float32", n, stream))
    torch.cuda.synchronize()
    assert not [r for r in range(n) if not torch.equal(recv[r], send.reshape(-1))]
    del send, recv
    pat.check(pat.pat_finalize())
    torch.cuda.empty_cache()
    n, count = 2, 4 * (1 << 30) + 1027
    print(f"[gpu] walk reducescatter n={n} count={count} float32", file=sys.stderr, flush=True)
    send = torch.empty(n, n * count, device=dev).uniform_(-1, 1)
    recv = torch.empty(n, count, device=dev)
    pat.check(pat.pat_reducescatter(list(send), list(recv), count, "float32", pat.PAT_SUM, n, stream))
    torch.cuda.synchronize()
    step = 1 << 28
    for r in range(n):
        for i in range(0, count, step):
            j = min(i + step, count)
            assert torch.equal(recv[r, i:j], send[r, r * count + i:r * count + j] + send[1 - r, r * count + i:r * count + j])
    del send, recv
    pat.check(pat.pat_finalize())
    torch.cuda.empty_cache()
