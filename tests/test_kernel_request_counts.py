"""The small-M kernels and the row-walking kernel wait on vector-memory requests with hand-counted
`s_waitcnt vmcnt(n)`; n is built from the number of requests that fetch one row tile.  This
test compiles the kernels to gfx950 assembly (no GPU needed) and checks that the requests
the compiler emitted are whole multiples of that number, so a request added to or dropped
from the tile fetch without the count following fails here, on the CPU, and not as a wrong
sum on the GPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_11582_amd", "csrc")


def _hipcc():
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return None


def _assembly(source, directory):
    """A source compiled to gfx950 assembly, split into (kernel name, body) pairs."""
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not found")
    asm = str(directory / (source + ".s"))
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                          "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "--cuda-device-only", "-S",
                          os.path.join(CSRC, source), "-o", asm], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    parts = re.split(r"\n(_Z\w+):[^\n]*\n", open(asm).read())
    return [(name, body.split(".Lfunc_end")[0]) for name, body in zip(parts[1::2], parts[2::2])]


@pytest.fixture(scope="module")
def smallm_asm(tmp_path_factory):
    return _assembly("egt_mfma_smallm.hip", tmp_path_factory.mktemp("asm"))


def _lane_loops(body):
    """Loops over the lanes of a wave around a request (what the compiler makes of a resource or a uniform offset that it
    does not know to be uniform: one request per distinct value)."""
    lines, labels, found = body.split("\n"), {}, 0
    for k, ln in enumerate(lines):
        m = re.match(r"(\.LBB\w+):", ln)
        if m:
            labels[m.group(1)] = k
        m = re.search(r"s_cbranch_execnz (\.LBB\w+)", ln)
        if m and m.group(1) in labels:
            loop = "\n".join(lines[labels[m.group(1)]:k])
            found += bool(k - labels[m.group(1)] < 60 and re.search(r"\bbuffer_load", loop) and re.search(r"v_readfirstlane", loop) and "saveexec" in loop)
    return found


def test_tile_requests_of_the_small_m_kernels_match_the_wait_counts(smallm_asm):
    text = open(os.path.join(CSRC, "egt_mfma_smallm.hip")).read()
    loads = re.search(r"static constexpr int LOADS = KIND == EGT_VAL_INT4 \? (\d+) : 1 \+ VW;", text)
    vw = re.search(r"static constexpr int VW = KIND == EGT_VAL_INT4 \? 1 : (\d+);", text)
    assert loads and vw, "ATile::LOADS / ATile::VW are not where this test reads them"
    per_tile = {0: int(loads.group(1)), 1: 1 + int(vw.group(1))}          # by value kind
    # no hand-written count survives beside the constant
    assert not re.search(r"wait_vmem<[^>]*\b[2-9]\b[^>]*>", text), "a literal request count in a wait"
    seen = 0
    for name, body in smallm_asm:
        m = re.search(r"k_sparse_smallm_ks(?:_batch|_joint)?ILi(\d)ELi(\d+)ELi(\d+)E", name)   # KIND, NT, NIT
        if not m:
            continue
        kind, nit = int(m.group(1)), int(m.group(3))
        requests = [ln for ln in body.split("\n") if re.search(r"\bbuffer_load_dword", ln)]
        tile_requests = [ln for ln in requests if " lds" not in ln]           # X goes straight to LDS: counted apart
        assert tile_requests, name
        assert len(tile_requests) % (nit * per_tile[kind]) == 0, (name, len(tile_requests), nit, per_tile[kind])
        waits = {int(v) for v in re.findall(r"vmcnt\((\d+)\)", body)}
        assert max(waits) <= 2 * nit * per_tile[kind], (name, sorted(waits))   # at most two phases of tiles pending
        assert _lane_loops(body) == 0, name
        seen += 1
    assert seen >= 60


def test_requests_of_the_row_split_stack_kernel_match_its_wait_counts(smallm_asm):
    # k_smallm_rows<NG, Q, W> allows exactly the Q * LOADS requests of the next round's A tiles to stay pending at
    # the top of a round; the round body is compiled twice (two sets of fetch registers) after a prologue of two rounds
    text = open(os.path.join(CSRC, "egt_mfma_smallm.hip")).read()
    loads = int(re.search(r"static constexpr int LOADS = KIND == EGT_VAL_INT4 \? (\d+) : 1 \+ VW;", text).group(1))
    seen = 0
    for name, body in smallm_asm:
        m = re.search(r"k_smallm_rowsILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", name)       # NG, Q, W, N1
        if not m:
            continue
        ng, q, w, n1 = (int(v) for v in m.groups())
        per_round, x_per_round = q * loads, ng * q * (16 if n1 else 8) // w      # (1:4: a request of X per token, 2:4: per pair)
        requests = [ln for ln in body.split("\n") if re.search(r"\bbuffer_load_dword", ln)]
        to_lds = [ln for ln in requests if " lds" in ln]
        assert len(requests) - len(to_lds) == 4 * per_round, (name, len(requests), len(to_lds))   # rounds 0, 1 and j + 2 twice
        assert len(to_lds) == 3 * x_per_round, (name, len(to_lds))                                # X(0) and X(j + 1) twice
        waits = [int(v) for v in re.findall(r"vmcnt\((\d+)\)", body)]
        assert waits.count(per_round) >= 2 and max(waits) <= 2 * per_round + x_per_round + 1, (name, sorted(set(waits)))
        assert len(re.findall(r"\bs_barrier\b", body)) == 2, name
        assert not re.search(r"\bscratch_|\bflat_", body), name
        seen += 1
    assert seen == 5


def test_waits_of_the_stack_kernel_count_only_requests_that_are_there(smallm_asm):
    # k_stack_tiles<NG, T, QW, NARROW, N1>: a round of the loop lets the 4 T requests of the next round's weights stay pending;
    # the odd last round, on whose way the compiler may leave requests out, waits for all of them
    seen = 0
    for name, body in smallm_asm:
        m = re.search(r"k_stack_tilesILi(\d+)ELi(\d)E", name)
        if not m:
            continue
        lines = body.split("\n")
        barriers = [k for k, ln in enumerate(lines) if re.search(r"\bs_barrier\b", ln)]
        # (the waits of the source, not those that the compiler adds)
        waits = [re.match(r"\s*s_waitcnt vmcnt\((\d+)\)\s*$", ln) if "ASMSTART" in lines[k - 1] else None for k, ln in enumerate(lines)]
        before = [next(int(waits[j].group(1)) for j in range(k, -1, -1) if waits[j]) for k in barriers]
        per_round = 4 * int(m.group(2))
        assert sorted(before) == [0, per_round, per_round], (name, before)
        asked = len([ln for ln in lines if re.search(r"\bbuffer_load_dword", ln) and " lds" not in ln])
        assert asked == 4 * per_round, (name, asked)     # rounds 0 and 1, and j + 2 twice
        assert _lane_loops(body) == 0 and not re.search(r"\bscratch_|\bflat_", body), name
        seen += 1
    assert seen == 7


def _prologue(body, wait):
    """(requests of tiles, requests of x to LDS) in the straight line before the first `vmcnt(wait)`, up to the first
    barrier; a request that stands in both arms of a branch (lanes on, lanes off) writes one register and counts once."""
    lines = body.split("\n")
    end = next(k for k, ln in enumerate(lines) if re.search(r"vmcnt\(%d\)" % wait, ln))
    requests = [ln for ln in lines[:end] if re.search(r"\bbuffer_load", ln)]
    tiles = [ln for ln in requests if " lds" not in ln]
    first = next(k for k, ln in enumerate(lines) if ln in tiles)
    assert not any(" lds" in ln for ln in lines[first:end]), "x requested between the tiles"
    return {re.search(r"buffer_load_\w+ (\S+),", ln).group(1) for ln in tiles}, len(requests) - len(tiles)


def test_requests_of_the_products_held_in_registers_match_the_wait_count(tmp_path):
    # k_smallm_hold<QW, N1, NG, RING, ...>: x and then RING tiles of three requests each are asked for; the wait for x allows
    # exactly the tiles to stay pending
    seen = 0
    for name, body in _assembly("egt_mfma_smallm_hold.hip", tmp_path):
        m = re.search(r"k_smallm_holdILi(\d+)ELb(\d)ELi(\d+)ELi(\d+)E", name)
        if not m:
            continue
        ring = int(m.group(4))
        registers, to_lds = _prologue(body, 3 * ring)
        assert len(registers) == 3 * ring and to_lds >= 1, (name, registers, to_lds)
        assert _lane_loops(body) == 0 and not re.search(r"\bscratch_|\bflat_", body), name
        seen += 1
    assert seen >= 40


def test_requests_of_the_row_walking_kernel_match_the_wait_count(tmp_path):
    # k_rows<MP>: x, then two items of four tiles of two requests each
    text = open(os.path.join(CSRC, "egt_rows.hip")).read()
    tpi, loads = int(re.search(r"ROWS_TPI = (\d+);", text).group(1)), int(re.search(r"LOADS = (\d+);", text).group(1))
    seen = 0
    for name, body in _assembly("egt_rows.hip", tmp_path):
        if "k_rows" not in name:
            continue
        registers, to_lds = _prologue(body, 2 * tpi * loads)
        assert len(registers) == 2 * tpi * loads and to_lds == 1, (name, registers, to_lds)
        assert _lane_loops(body) == 0 and not re.search(r"\bscratch_|\bflat_", body), name
        seen += 1
    assert seen == 4


def test_requests_of_the_exact_codes_match_the_wait_count(tmp_path):
    # k_codes<FORM, CPL, UNITS, TPI, MP>: x, then a wave's tiles (rows of different lengths five requests each, dense rows two, the others three)
    text = open(os.path.join(CSRC, "egt_mfma_codes.hip")).read()
    dense, mixed, other = (int(v) for v in re.search(r"LOADS = DENSE \? (\d+) : MIXED \? (\d+) : (\d+);", text).groups())
    seen = 0
    for name, body in _assembly("egt_mfma_codes.hip", tmp_path):
        m = re.search(r"k_codes(?:_batch)?ILi(\d)ELi\d+ELi\d+ELi(\d)E", name)
        if not m:
            continue
        loads = int(m.group(2)) * {2: mixed, 3: dense}.get(int(m.group(1)), other)
        registers, to_lds = _prologue(body, loads)
        assert len(registers) == loads and to_lds == 1, (name, registers, to_lds)
        assert _lane_loops(body) == 0 and not re.search(r"\bscratch_|\bflat_", body), name
        seen += 1
    assert seen >= 40


def test_rows_past_the_last_one_are_requested_past_the_buffer_by_the_lane_offset(tmp_path):
    # k_codes: a wave's buffers begin at its first row, and the whole place of a request lies in its lane offset, which the range
    # check compares with the buffer's size.  A uniform offset beyond the size (the check subtracts it) is never there: only
    # the codes and index words of rows of different lengths have one, four requests a tile, from checked row pointers.
    seen = 0
    for name, body in _assembly("egt_mfma_codes.hip", tmp_path):
        m = re.search(r"k_codes(?:_batch)?ILi(\d)ELi\d+ELi\d+ELi(\d)E", name)
        if not m:
            continue
        requests = [ln for ln in body.split("\n") if re.search(r"\bbuffer_load", ln)]
        uniform = [ln for ln in requests if not re.search(r", 0 offen\b", ln)]
        assert requests and len(uniform) == (4 * int(m.group(2)) if m.group(1) == "2" else 0), (name, uniform)
        seen += 1
    assert seen >= 40


def test_requests_of_the_product_for_many_tokens_match_its_wait_counts(smallm_asm):
    # k_smallm_wide*<NG, NIT>: phases 0 and 1 are asked for ahead, a phase of the loop asks for its next but one after its first
    # unit of x, the odd last phase asks for no tiles and counts none (3 NIT requests a phase, 8 a unit of x)
    seen = 0
    for name, body in smallm_asm:
        m = re.search(r"k_smallm_wide(?:_batch|_ks_joint)?ILi(\d)ELi(\d)E", name)
        if not m:
            continue
        ng, na = int(m.group(1)), 3 * int(m.group(2))
        events = []
        lines = body.split("\n")
        for k, ln in enumerate(lines):
            w = re.match(r"\s*s_waitcnt vmcnt\((\d+)\)\s*$", ln)
            if w and "ASMSTART" in lines[k - 1]:
                events.append(int(w.group(1)))
            elif re.search(r"\bbuffer_load", ln):
                events.append("x" if " lds" in ln else "a")
        assert events.count("a") == 4 * na, (name, events.count("a"))
        assert events.count("x") == 8 * (2 + 3 * ng) and _lane_loops(body) == 0, name
        assert not re.search(r"\bscratch_|\bflat_", body), name
        waits = [e for e in events if isinstance(e, int)]
        allowed = {8, 8 + na, 8 + 2 * na, 0}
        assert set(waits) == allowed and waits.count(0) == 1 and waits.count(8 + 2 * na) >= 1, (name, waits)
        # the odd last phase: units whose wait counts x alone, and no tiles between them
        first = " ".join(str(e) for e in events).replace("x " * 8, "X ").replace("a " * na, "A ")
        assert first.startswith("X A X A "), (name, first[:60])
        assert ("8 X " * ng).strip() in first, (name, first)
        seen += 1
    assert seen == 20
