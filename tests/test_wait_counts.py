"""The hand-counted vector-memory waits of the prefill kernels' operand pipelines and of the decode kernel's activation
copy, checked without a GPU.

1. A host-side model (tests/ring_model/ring_check.cpp, plain C++) replays the kernels' per-thread issue order for every
   instantiation the library launches and every step count up to 48, with the constants of the header the kernels
   themselves use (csrc/bl_gemm_ring.hpp), under the ISA's rule "operations complete in issue order, vmcnt(n) = at most n
   outstanding": every LDS read of an activation tile must lie behind a barrier that followed the tile's completion,
   every overwrite of a stage behind a barrier that followed its last read -- whether the compiler keeps the dead weight
   loads of the loop's tail or removes them.  With the tail's count set to the main loop's (the kernel's earlier form)
   the model must fail: that is the mistake it is there to catch.  The kernel for few tokens, whose waves have stages of
   their own and no barrier, is replayed in the same way, and must fail with one operation more left outstanding.
2. The model's premise -- which loads each step issues -- is checked against the compiler's output: the kernels are
   compiled to assembly for gfx950 and every barrier of the K loop must be preceded by the expected wait and by the
   expected number of global -> LDS requests and weight loads since the barrier before it.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16144_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ring") / "ring_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                           os.path.join(ROOT, "tests", "ring_model", "ring_check.cpp"), "-o", exe])
    return exe


def test_model_accepts_the_kernels_wait_counts(model):
    r = subprocess.run([model], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "0 failing cases" in r.stdout


def test_model_rejects_the_main_loop_count_in_the_tail(model):
    r = subprocess.run([model, "--old-tail"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 1
    n = int(re.search(r"(\d+) failing cases", r.stdout).group(1))
    assert n > 0


def test_model_rejects_a_wait_that_leaves_one_more_outstanding(model):
    r = subprocess.run([model, "--slack"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 1 and int(re.search(r"(\d+) failing cases", r.stdout).group(1)) > 0


def _functions(asm_path):
    cur, out = None, {}
    with open(asm_path) as f:
        for line in f:
            m = re.match(r"^(_Z\S+):", line)
            if m:
                cur = m.group(1)
                out[cur] = []
            elif line.startswith(".Lfunc_end"):
                cur = None
            elif cur:
                out[cur].append(line.strip())
    return out


def _barriers(lines):
    """Per s_barrier: (vmcnt of the last wait since the previous barrier, global->LDS loads, 128-bit loads since it)."""
    seq, lds, w, wait = [], 0, 0, None
    for l in lines:
        if l.startswith("global_load_lds_dwordx4"):
            lds += 1
        elif l.startswith("global_load_dwordx4"):
            w += 1
        elif l.startswith("s_waitcnt"):
            m = re.search(r"vmcnt\((\d+)\)", l)
            if m:
                wait = int(m.group(1))
        elif l.startswith("s_barrier"):
            seq.append((wait, lds, w))
            lds, w, wait = 0, 0, None
    return seq


def _loops(lines):
    """The bodies between a label and a branch back to it."""
    at = {l.split(":")[0]: i for i, l in enumerate(lines) if l.startswith(".LBB")}
    bodies = []
    for i, l in enumerate(lines):
        m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", l)
        if m and at.get(m.group(1), i) < i:
            bodies.append(lines[at[m.group(1)]:i])
    return bodies


def _compile_to_asm(tmp, name, extra=()):
    out = str(tmp / (name + ".s"))
    cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-Wno-unused-command-line-argument", *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           "-S", "--cuda-device-only", "-o", out, os.path.join(CSRC, name)]
    subprocess.run(cmd, check=True, stderr=subprocess.DEVNULL, timeout=600)
    return out


def _check_tiles(name, seq, mb, h, wk, wn):
    """The barriers of a tile's code: a prologue, the main loop's eight steps and the tail's, wherever the compiler laid them."""
    nt, lead = (h + 1) // 2, 4
    wr = 8 if nt == 1 else 4
    rq = -(-(wk * 2 * mb) // (wn * wk))          # requests per loader thread and step
    younger, younger_tail, prologue = (lead - 2) * (rq + nt), (lead - 2) * rq, (lead - 3) * rq
    # prologue: the weight ring's first tiles and the first kLead requests, a wait that leaves kPrologueWait outstanding
    assert seq[0][1] == lead * rq and seq[0][2] == (wr - 1) * nt and seq[0][0] is not None and seq[0][0] <= prologue, (name, seq[0])
    main = [b for b in seq[1:] if b[0] == younger]
    tail = [b for b in seq[1:] if b[0] == younger_tail]
    assert len(main) == 8 and len(tail) == 7, (name, seq)
    for wait, lds, w in main:          # a step of the main loop: kRQ requests, at least the kNT weight loads
        assert lds == rq and w >= nt, (name, seq)
    for wait, lds, w in tail:          # a step of the tail: kRQ requests; its weight loads may be gone
        assert lds == rq, (name, seq)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_compiled_prefill_kernels_issue_what_the_model_assumes(tmp_path):
    fns = _functions(_compile_to_asm(tmp_path, "bl_gemm.hip"))
    seen = 0
    for name, lines in fns.items():
        m = re.search(r"gemm_(?:batch_)?kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)E", name)
        if m:
            seen += 1
            _check_tiles(name, _barriers(lines), *(int(x) for x in m.groups()))
    assert seen == 14                      # seven forms, single and batched


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_compiled_few_token_kernels_issue_what_the_model_assumes(tmp_path):
    """No barrier in the loop: the requests between the function's start and the first barrier are D steps ahead of it and one
    step's inside it, the loop waits for 0 or kYounger of them and has no other vector memory operation."""
    fns = _functions(_compile_to_asm(tmp_path, "bl_gemm_narrow.hip"))
    forms = {(16, 1): 2, (16, 2): 2, (32, 1): 2, (32, 2): 1, (32, 4): 1, (64, 4): 1}      # (T, RH): D
    seen = 0
    for name, lines in fns.items():
        m = re.search(r"gemm_narrow_kernelILi(\d+)ELi(\d)ELi8ELi(\d)E", name)
        if not m:
            continue
        seen += 1
        t, rh, d = (int(x) for x in m.groups())
        assert forms[t, rh] == d
        per_step = rh + t // 8
        end = next(i for i, l in enumerate(lines) if l.startswith("s_barrier"))
        loop = lines[:end]
        requests = [i for i, l in enumerate(loop) if l.startswith("global_load_lds_dwordx4")]
        assert len(requests) == (d + 1) * per_step, name
        for l in loop[requests[0]:]:
            assert not re.match(r"(scratch_|buffer_|flat_|global_store|global_atomic)", l), (name, l)
        # ordinary loads: the scales, before the first request or behind the loop, whose products end it or lie before it
        last = max(i for i, l in enumerate(loop) if l.startswith("v_mfma") or i in set(requests))
        for i, l in enumerate(loop):
            if re.match(r"global_load_dword\b", l):
                assert i < requests[0] or i > last, (name, l)
        waits = {int(w) for l in loop[requests[0]:last] for w in re.findall(r"vmcnt\((\d+)\)", l)}
        assert waits == ({0, (d - 1) * per_step} if d > 1 else {0}), (name, waits)
    assert seen == 6


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_compiled_decode_copy_waits_for_the_copy_only(tmp_path):
    fns = _functions(_compile_to_asm(tmp_path, "bl_gemv.hip", ("-mllvm", "-amdgpu-kernarg-preload-count=7")))
    seen = 0
    for name, lines in fns.items():
        # QMODE 1 (activations copied into LDS), either kind of weight load, not the publishing form (which issues
        # the copy last and waits for everything)
        if not re.search(r"decode_mfma_kernelILi\dELi1ELb\dELb\dELb0E", name):
            continue
        seen += 1
        first = _barriers(lines)[0]
        # the copy's requests, then exactly the 6 weight tiles of the first batch, and a wait that lets those 6 fly
        assert first[1] >= 1 and first[2] == 6 and first[0] == 6, (name, first)
    assert seen == 16


def _check_paired_extras(name, lines, loops, forms):
    """What stands between the products and ahead of them: the LDS address register is written once for up to four requests, always with
    the pause they need behind it and by nobody else; one division, the mapping to tiles, ahead of the first request."""
    code = [l for l in lines if l and not l.startswith((";", ".")) and not l.endswith(":")]
    for i, l in enumerate(code):
        if re.search(r"\bm0\b", l):
            assert l.startswith("s_mov_b32 m0,") and code[i + 1] == "s_nop 0" and code[i + 2].startswith("global_load_lds_dwordx4"), (name, code[i:i + 3])
    writes = sorted(sum(l.startswith("s_mov_b32 m0,") for l in body) for body in loops)
    assert writes == sorted(s * -(-(h + 4 * mb // wn) // 4) for mb, h, wn, wk, s in forms), (name, writes)
    first = next(i for i, l in enumerate(code) if l.startswith("global_load_lds_dwordx4"))
    assert sum("v_rcp" in l for l in code[:first]) == 1, name


def test_paired_kernels_waits_hold_and_one_operation_less_does_not(tmp_path):
    """csrc/bl_gemm_pair.hip: the issue order of every form replayed with the constants of the kernel's header (see
    tests/ring_model/pair_check.cpp), and with every wait one operation too generous, which must fail."""
    exe = str(tmp_path / "pair_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                           os.path.join(ROOT, "tests", "ring_model", "pair_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "0 failing cases" in r.stdout, r.stdout[-2000:]
    assert subprocess.run([exe, "--slack"], capture_output=True, timeout=120).returncode == 1


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_compiled_paired_kernels_issue_what_the_model_assumes(tmp_path):
    """The main loop of every form, and both of the two-width kernel, by its back edge: S steps, each with one step's requests, the
    wait that the header names and a barrier; and no other vector memory operation behind the first request but the output's stores."""
    fns = _functions(_compile_to_asm(tmp_path, "bl_gemm_pair.hip"))
    seen = 0
    for name, lines in fns.items():
        m = re.search(r"pair_gemm_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d+)E", name)
        if m:
            forms = [tuple(int(x) for x in m.groups())]
        elif "mixed_pair_gemm_kernel" in name:
            forms = [(2, 2, 4, 1, 4), (2, 1, 4, 1, 4)]
        else:
            continue
        seen += 1
        # per form: S steps of H + 4 MB / WN requests and a wait that leaves the S - 3 steps requested last on their way
        want = [[((s - 3) * (h + 4 * mb // wn), h + 4 * mb // wn, 0)] * s for mb, h, wn, wk, s in forms]
        # (the main loop is straight code; a tail's steps, laid out in any order with branches between them, are not)
        loops = [body for body in _loops(lines)
                 if any(l.startswith("s_barrier") for l in body) and not any(re.match(r"s_c?branch", l) for l in body)]
        got = [_barriers(body) for body in loops]
        assert sorted(got) == sorted(want), (name, got)
        _check_paired_extras(name, lines, loops, forms)
        # what the compiler sees is loaded before the first request (the scales) and nothing after it
        requests = [i for i, l in enumerate(lines) if l.startswith("global_load_lds_dwordx4")]
        others = [i for i, l in enumerate(lines) if re.match(r"(scratch_|flat_|global_store|global_atomic|buffer_load|global_load_dword(x2|x4)?\b)", l)]
        if len(forms) == 1:
            assert all(i < requests[0] for i in others), (name, [lines[i] for i in others])
        else:   # two tiles' code, one behind the other: each loads its scales ahead of its own first request
            assert not any(re.match(r"(scratch_|flat_|global_store|global_atomic|buffer_load)", lines[i]) for i in others), name
            for body in _loops(lines):
                assert not any(re.match(r"global_load_dword(x2|x4)?\b", l) for l in body if any(x.startswith("s_barrier") for x in body)), name
    assert seen == 8


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_compiled_paired_kernels_of_one_workgroup_per_unit_issue_what_the_model_assumes(tmp_path):
    """bl_gemm_pair_wide.hip, looked at as the paired kernels above: S steps per trip, each with one step's requests, the header's
    wait and a barrier, and nothing else behind the first request but the output's stores."""
    fns = _functions(_compile_to_asm(tmp_path, "bl_gemm_pair_wide.hip"))
    seen = 0
    for name, lines in fns.items():
        m = re.search(r"pair_gemm_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d+)E", name)
        if not m:
            continue
        seen += 1
        mb, h, wn, wk, s = (int(x) for x in m.groups())
        want = [((s - 3) * (h + 4 * mb // wn), h + 4 * mb // wn, 0)] * s
        loops = [body for body in _loops(lines)
                 if any(l.startswith("s_barrier") for l in body) and not any(re.match(r"s_c?branch", l) for l in body)]
        got = [_barriers(body) for body in loops]
        assert got == [want], (name, got)
        _check_paired_extras(name, lines, loops, [(mb, h, wn, wk, s)])
        requests = [i for i, l in enumerate(lines) if l.startswith("global_load_lds_dwordx4")]
        others = [i for i, l in enumerate(lines) if re.match(r"(scratch_|flat_|global_store|global_atomic|buffer_load|global_load_dword(x2|x4)?\b)", l)]
        assert all(i < requests[0] for i in others), (name, [lines[i] for i in others])
    assert seen == 2


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_compiled_token_attention_keeps_a_chunk_half_on_its_way(tmp_path):
    """bl_decoder.hip's walk over the cache: a loop with one run of requests for the next keys and one for the next values, kVecs
    each, in which no wait is for fewer than the kVecs requests issued last; and no instance spills a register."""
    asm = _compile_to_asm(tmp_path, "bl_decoder.hip")
    fns = _functions(asm)
    spills = dict(re.findall(r"\.amdhsa_kernel (\S+)\n(?:.*\n)*?\s+\.amdhsa_private_segment_fixed_size (\d+)", open(asm).read()))
    seen = 0
    for name, lines in fns.items():
        m = re.search(r"attn_chunk_kernelILi(\d+)ELi(\d+)E", name)
        if not m:
            continue
        seen += 1
        w, maxd = (int(x) for x in m.groups())
        vecs = 64 * (maxd // w) // 256
        assert spills[name] == "0", (name, spills[name])
        load = "global_load_dwordx%d" % (w // 2)
        bodies = [body for body in _loops(lines) if any(l.startswith(load) for l in body)]
        walk = min(bodies, key=len)
        runs, waits, since = [], [], vecs
        for l in walk:
            if l.startswith(load):
                runs = runs + [1] if since else runs[:-1] + [runs[-1] + 1]
                since = 0
            elif l.startswith("s_waitcnt"):
                since = 1
                waits += [int(x) for x in re.findall(r"vmcnt\((\d+)\)", l)]
            assert not re.match(r"(scratch_|flat_|buffer_|s_barrier)", l), (name, l)
        assert runs == [vecs, vecs] and min(waits) == vecs, (name, runs, waits)
    assert seen == 4
