"""Structural checks of compiled kernels (no GPU needed): the streaming GEMM's hand-counted
waits, and the split-K hand-over of the projection's partial sums.

The kernel issues its ring loads as inline assembly and waits for them with hand-counted
`s_waitcnt vmcnt(N)`.  That is only correct while the compiler (a) adds no vector-memory
operation of its own to the loop, (b) never copies a ring register between its load and its
wait, and (c) does not hand a register of a load still in flight to other code behind the loop.
These properties are read off the generated assembly."""
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_00422_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# every instantiation that is launched (the tiles of csrc/gemm_tiles.h), each with plain codes, gated, and with
# nibble-packed codes (4 code copies per slice instead of 8): (channel tiles per wavefront, wavefronts that share K, ring
# depth) of the kernels with private rings ...
PRIVATE = [(1, 4, 4), (2, 4, 4), (2, 2, 4), (3, 2, 4)]
# ... and (channel tiles, ring depth, wavefronts side by side) of the kernels with one ring of codes
SHARED = [(1, 4, 2), (1, 4, 4), (2, 4, 4), (3, 4, 4), (4, 2, 4), (5, 4, 4)]
FORMS = [(0, 0), (1, 0), (0, 1)]                           # (gated, nibble-packed)


@pytest.fixture(scope="module")
def gemm_asm():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "gemm_prefill.s")
        cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
               "-o", out, os.path.join(CSRC, "gemm_prefill.hip")]
        subprocess.run(cmd, check=True, capture_output=True)
        text = open(out).read().split("\n")
    return text


def _kernel(text, name, args):
    pat = re.compile(rf"^_ZN.*{name}I{''.join(args)}E.*:")
    start = next(i for i, l in enumerate(text) if pat.match(l))
    end = next(i for i in range(start, len(text)) if "s_endpgm" in text[i])
    return text[start:end + 1]


def test_these_are_the_kernels_of_the_file(gemm_asm):
    def template_args(name):
        found = set()
        for l in gemm_asm:
            m = re.match(rf"^_ZN.*{name}I((?:L[ib]\d+E)+)E.*:", l)
            if m:
                found.add(tuple(map(int, re.findall(r"L[ib](\d+)E", m.group(1)))))
        return found
    assert template_args("gemm_prefill_direct_kernel") == {(*v, *f) for v in PRIVATE for f in FORMS}
    assert template_args("gemm_prefill_shared_kernel") == {(*v, *f) for v in SHARED for f in FORMS}


def _main_loop(lines):
    start = next(i for i, l in enumerate(lines) if "Loop Header" in l)
    label = lines[start].split(":")[0].strip()
    end = next(i for i in range(start + 1, len(lines)) if re.search(rf"s_cbranch\S*\s+{re.escape(label)}$", lines[i]))
    return start, end


@pytest.mark.parametrize("gated,a4", FORMS)
@pytest.mark.parametrize("ntl,wk,nb", PRIVATE)
def test_streaming_gemm_loop_structure(gemm_asm, ntl, wk, nb, gated, a4):
    lines = _kernel(gemm_asm, "gemm_prefill_direct_kernel", [f"Li{ntl}E", f"Li{wk}E", f"Li{nb}E", f"Lb{gated}E", f"Lb{a4}E"])
    copies = 4 if a4 else 8
    start, end = _main_loop(lines)
    loop = lines[start:end + 1]
    code = [l.strip() for l in loop if l.strip() and not l.strip().startswith((";", "."))]
    # nb slices per trip: nb x (NTL weight loads + 8 asynchronous code copies), nb x 4 x 2 NTL MFMAs
    assert sum(l.startswith("global_load_lds_dwordx4") for l in code) == copies * nb
    assert sum(l.startswith("global_load_dwordx4") for l in code) == nb * ntl
    assert sum(l.startswith("v_mfma_i32_32x32x32_i8") for l in code) == nb * 4 * 2 * ntl
    # the only vector-memory waits are the hand-counted ones, with the documented count
    waits = [l for l in code if l.startswith("s_waitcnt") and "vmcnt" in l]
    assert waits == [f"s_waitcnt vmcnt({(nb - 2) * (ntl + copies)})"] * nb
    # no other memory traffic and no register shuffling of ring or accumulator registers
    assert not any(l.startswith(("scratch_", "global_store", "buffer_", "flat_")) for l in code)
    assert not any(l.startswith(("v_mov_b32", "v_accvgpr")) for l in code)


@pytest.mark.parametrize("gated,a4", FORMS)
@pytest.mark.parametrize("ntl,wk,nb", PRIVATE)
def test_registers_of_loads_in_flight_stay_reserved(gemm_asm, ntl, wk, nb, gated, a4):
    lines = _kernel(gemm_asm, "gemm_prefill_direct_kernel", [f"Li{ntl}E", f"Li{wk}E", f"Li{nb}E", f"Lb{gated}E", f"Lb{a4}E"])
    _registers_of_loads_in_flight_stay_reserved(lines, ntl, nb)


def _registers_of_loads_in_flight_stay_reserved(lines, ntl, nb):
    start, end = _main_loop(lines)
    dest = set()
    for l in lines[start:end]:
        m = re.match(r"\s*global_load_dwordx4 v\[(\d+):(\d+)\]", l)
        if m:
            dest.update(range(int(m.group(1)), int(m.group(2)) + 1))
    assert len(dest) == 4 * nb * ntl
    drain = next(i for i in range(end, len(lines)) if "s_waitcnt vmcnt(0)" in lines[i])
    for l in lines[end + 1:drain]:
        l = l.strip()
        if not l or l.startswith((";", ".", "s_", "global_store", "ds_write", "scratch_store")):
            continue
        m = re.match(r"\S+\s+v\[(\d+):(\d+)\]", l) or re.match(r"\S+\s+v(\d+)()", l)
        if m:
            lo = int(m.group(1))
            hi = int(m.group(2)) if m.group(2) else lo
            assert not any(r in dest for r in range(lo, hi + 1)), f"writes a register of a load in flight: {l}"


@pytest.mark.parametrize("gated,a4", FORMS)
@pytest.mark.parametrize("ntl,nb,wn", SHARED)
def test_shared_ring_loop_structure(gemm_asm, ntl, nb, wn, gated, a4):
    """As above, and one barrier a slice, directly behind the counted wait; loads in flight keep their registers."""
    lines = _kernel(gemm_asm, "gemm_prefill_shared_kernel", [f"Li{ntl}E", f"Li{nb}E", f"Li{wn}E", f"Lb{gated}E", f"Lb{a4}E"])
    copies = (4 if a4 else 8) // wn
    start, end = _main_loop(lines)
    code = [l.strip() for l in lines[start:end + 1] if l.strip() and not l.strip().startswith((";", "."))]
    assert sum(l.startswith("global_load_lds_dwordx4") for l in code) == copies * nb
    assert sum(l.startswith("global_load_dwordx4") for l in code) == nb * ntl
    assert sum(l.startswith("v_mfma_i32_32x32x32_i8") for l in code) == nb * 4 * 2 * ntl
    waits = [i for i, l in enumerate(code) if l.startswith("s_waitcnt") and "vmcnt" in l]
    assert [code[i] for i in waits] == [f"s_waitcnt vmcnt({(nb - 2) * (ntl + copies)})"] * nb
    barriers = [i for i, l in enumerate(code) if l.startswith("s_barrier")]
    assert len(barriers) == nb
    for w, b in zip(waits, barriers):
        # the next slice's rows are read, and its predecessor's tile is filled again, behind the barrier only
        assert w < b and not any(l.startswith(("ds_read", "global_load_lds")) for l in code[w:b])
    assert not any(l.startswith(("scratch_", "global_store", "buffer_", "flat_", "v_mov_b32", "v_accvgpr")) for l in code)
    _registers_of_loads_in_flight_stay_reserved(lines, ntl, nb)


def _device_asm(src):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "out.s")
        cmd = [HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
               "-o", out, os.path.join(CSRC, src)]
        subprocess.run(cmd, check=True, capture_output=True)
        return [l.strip() for l in open(out).read().split("\n")]


@pytest.mark.parametrize("src,min_sites", [("psp_prefill.hip", 1), ("rotate_quant.hip", 2)])
def test_partial_sums_are_acknowledged_before_the_arrival_count(src, min_sites):
    """The workgroup that arrives last at the counter reads the other workgroups' partial tiles.
    Nothing but an explicit wait orders a workgroup's device-scope stores before its counter bump
    (a workgroup-scope fence emits none), so between the last such store and the returning atomic
    add there must be: a wait for all vector-memory operations, then the barrier, then the add."""
    lines = _device_asm(src)
    sites = 0
    for i, l in enumerate(lines):
        if not (l.startswith("global_atomic_add") and l.endswith("sc0")):
            continue                                   # (adds without return value are code sums)
        bar = next(j for j in range(i, 0, -1) if lines[j] == "s_barrier")
        st = next((j for j in range(bar, max(bar - 400, 0), -1)
                   if lines[j].startswith("global_store_dword") and lines[j].endswith("sc1")), None)
        if st is None:
            continue
        sites += 1
        waits = [j for j in range(st + 1, bar) if lines[j].startswith("s_waitcnt") and "vmcnt(0)" in lines[j]]
        assert waits, f"{src}: no vmcnt(0) wait between the partial stores (line {st}) and the barrier (line {bar})"
        assert not any(lines[j].startswith("global_store") for j in range(waits[-1], bar))
    assert sites >= min_sites


def test_decode_fallback_asks_early_only_where_a_wavefront_has_its_tile_alone():
    """gemm_decode_kernel<NT, MANY, EARLY>: operands of the epilogue held over the contraction cost registers
    (98: four wavefronts a SIMD) and, where wavefronts share K, loads that all but one of them throw away.  The
    forms that such workgroups are launched with stay at six wavefronts a SIMD (512 / 6 = 85 registers) and ask for nothing
    before the contraction but sign bits (16 bytes a lane) and code rows."""
    lines = _device_asm("gemm_decode.hip")
    for many in (0, 1):
        start = next(i for i, l in enumerate(lines) if re.match(rf"_ZN.*gemm_decode_kernelILi1ELb{many}ELb0E.*:", l))
        body = lines[start:next(i for i in range(start, len(lines)) if lines[i].startswith("s_endpgm"))]
        meta = next(i for i in range(start, len(lines)) if lines[i].startswith(".amdhsa_next_free_vgpr"))
        assert int(lines[meta].split()[1]) <= 84
        head = body[:next(i for i, l in enumerate(body) if l.startswith("s_barrier"))]
        assert any(l.startswith("global_load_dwordx4") for l in head)
        assert not any(re.match(r"global_load_(dword |dwordx2|ushort|short)", l) for l in head)


def test_last_workgroup_of_a_projection_tile_keeps_enough_slices_in_flight():
    """psp_prefill_kernel<BF16, NJT>: the partial sums of eight slices (four, of four vectors a thread: the counter of loads
    in flight holds 63) are requested before the first of them is waited for, whatever the number of vectors."""
    lines = _device_asm("psp_prefill.hip")
    for bf16 in (0, 1):
        for njt, least in ((1, 8 * 4), (2, 8 * 2 * 4), (4, 40)):
            start = next(i for i, l in enumerate(lines) if re.match(rf"_ZN.*psp_prefill_kernelILb{bf16}ELi{njt}E.*:", l))
            end = next(i for i in range(start, len(lines)) if lines[i].startswith(".amdhsa_next_free_vgpr"))
            run = best = 0
            for l in lines[start:end]:
                if l.startswith("global_load_dword ") and l.endswith("sc1"):
                    run += 1
                    best = max(best, run)
                elif l.startswith("s_waitcnt") and "vmcnt" in l:
                    run = 0
            assert best >= least, (bf16, njt, best)


# (token tiles, channel tiles, wavefronts, ring, workgroups a CU) of csrc/gemm_tiles.h
SPARSE = [(2, 2, 4, 4, 2), (2, 5, 4, 4, 1), (4, 4, 4, 4, 1)]


@pytest.fixture(scope="module")
def sparse_asm():
    return _device_asm("gemm_sparse.hip")


def _registers(l):
    """Vector registers an instruction names."""
    found = set()
    for m in re.finditer(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", l.split(";")[0]):
        lo = int(m.group(1) or m.group(3))
        found.update(range(lo, int(m.group(2) or lo) + 1))
    return found


@pytest.mark.parametrize("gated", [0, 1])
@pytest.mark.parametrize("tile", SPARSE)
def test_sparse_gemm_loop_structure(sparse_asm, tile, gated):
    """The sparse GEMM's loop loads nothing to registers from memory, waits for its asynchronous copies by a hand-counted
    number once a pair of contractions, and reads LDS by inline assembly: a register of such a read is named by nothing
    before the wait behind it."""
    mt, nt, wn, ring, resident = tile
    pat = re.compile(rf"_ZN.*gemm_sparse_kernelILi{mt}ELi{nt}ELi{wn}ELi{ring}ELi{resident}ELb{gated}E.*:")
    start = next(i for i, l in enumerate(sparse_asm) if pat.match(l))
    lines = sparse_asm[start:next(i for i in range(start, len(sparse_asm)) if sparse_asm[i].startswith(".amdhsa_next_free_vgpr"))]
    first = next(i for i, l in enumerate(lines) if l.startswith("v_smfmac"))
    last = max(i for i, l in enumerate(lines) if l.startswith("v_smfmac"))
    head = max(i for i in range(first) if lines[i].startswith(".LBB"))
    branch = next(i for i in range(last, len(lines)) if re.match(rf"s_cbranch\S*\s+{lines[head].split(':')[0]}$|s_branch\s+{lines[head].split(':')[0]}$", lines[i])
                  or lines[i].startswith("s_cbranch"))
    loop = [l for l in lines[head:branch] if l and not l.startswith((";", "."))]
    codes, weights = 2 * (32 * mt * 64) // 1024 // wn, (2 * nt + 3) // 4       # copies a pair and wavefront
    per = codes + weights
    assert sum(l.startswith("v_smfmac_i32_32x32x64_i8") for l in loop) == 8 * mt * nt
    assert sum(l.startswith("global_load_lds_dwordx4") for l in loop) == 4 * per
    assert not any(l.startswith(("scratch_", "global_store", "buffer_", "flat_", "v_accvgpr")) or
                   (l.startswith("global_load") and "_lds_" not in l) for l in loop)
    waits = [i for i, l in enumerate(loop) if l.startswith("s_waitcnt") and "vmcnt" in l]
    assert [loop[i] for i in waits] == [f"s_waitcnt vmcnt({(ring - 2) * per})"] * 4
    barriers = [i for i, l in enumerate(loop) if l.startswith("s_barrier")]
    assert len(barriers) == 4
    for w, b in zip(waits, barriers):
        assert w < b and not any(l.startswith(("ds_read", "global_load_lds")) for l in loop[w:b])
    # from the first asynchronous copy of the kernel on: the prologue's reads, then the loop twice (what is in flight at
    # its end meets its beginning)
    begin = next(i for i, l in enumerate(lines) if l.startswith("global_load_lds"))
    barrier = next(i for i in range(begin, len(lines)) if lines[i].startswith("s_barrier"))
    pro = next(i for i in range(barrier, len(lines)) if lines[i].startswith("ds_read"))
    for part in (lines[pro:head] if pro < head else [], loop + loop):
        pending = set()
        for l in part:
            if l.startswith("s_waitcnt") and "lgkmcnt(0)" in l:
                pending.clear()
                continue
            touched = _registers(l)
            assert not touched & pending, l
            if l.startswith("ds_read"):
                pending |= _registers(l.split(",")[0])
        assert not pending
    # the flags that are asked for before the copies stay untouched until the first counted wait
    flags = [i for i in range(begin) if lines[i].startswith("global_load_dword ")]
    assert len(flags) == 32 * mt // 16
    wait = next(i for i in range(begin, len(lines)) if lines[i].startswith("s_waitcnt") and "vmcnt" in lines[i])
    assert lines[wait] == f"s_waitcnt vmcnt({(ring - 1) * per})"
    for i in flags:
        regs = _registers(lines[i].split(",")[0])
        assert not any(_registers(l) & regs for l in lines[i + 1:wait])


def test_sparse_gemm_reads_h_from_lds_as_it_was_written(sparse_asm):
    """The gated epilogue leaves h in LDS as 32-bit pairs and other lanes read it; a 16-bit scalar read is one that the
    compiler may assume to be of something else, and so move in front of the writes."""
    assert any(l.startswith("ds_write_b32") or l.startswith("ds_write2_b32") for l in sparse_asm)
    assert not any(l.startswith(("ds_read_u16", "ds_read_i16")) for l in sparse_asm)


def test_rotation_in_fp32_keeps_the_summing_role_in_a_kernel_of_its_own():
    """rotate_quant_kernel<BF16, tiles, SUMS>: the role that adds up partial tiles (sixteen plain loads in flight) costs the
    rotation beside it 4 to 6 %, so the form that every other launch takes has none of it."""
    lines = _device_asm("rotate_quant.hip")
    forms = set()
    for i, l in enumerate(lines):
        m = re.match(r"_ZN.*rotate_quant_kernelILb([01])ELi(\d+)ELb([01])E.*:", l)
        if not m:
            continue
        forms.add(tuple(map(int, m.groups())))
        run = best = 0
        for x in lines[i:next(j for j in range(i, len(lines)) if lines[j].startswith(".amdhsa_next_free_vgpr"))]:
            if x.startswith("global_load_dword ") and not x.endswith("sc1"):
                run += 1
                best = max(best, run)
            elif x.startswith("s_waitcnt") and "vmcnt" in x:
                run = 0
        assert (best >= 16) == (m.group(3) == "1"), (m.groups(), best)
    assert forms == {(b, t, s) for b, s in ((0, 0), (1, 0), (1, 1)) for t in (2, 4, 16)}


@pytest.mark.parametrize("gated", [0, 1])
@pytest.mark.parametrize("tile", SPARSE)
def test_sparse_gemm_keeps_stores_in_flight_where_rows_start_anywhere(sparse_asm, tile, gated):
    """Rows of channels that do not start on whole vectors leave in stores of four as the others do, or, gated, eight at a
    time: read from LDS and stored value by value, they made the kernel slower than the dense one."""
    pat = re.compile(r"_ZN.*gemm_sparse_kernelI" + "".join(f"Li{x}E" for x in tile) + f"Lb{gated}E.*:")
    start = next(i for i, l in enumerate(sparse_asm) if pat.match(l))
    lines = sparse_asm[start:next(i for i in range(start, len(sparse_asm)) if sparse_asm[i].startswith(".amdhsa_next_free_vgpr"))]
    if not gated:
        assert sum(l.startswith("global_store_dwordx4") for l in lines) >= 8      # four of either kind in flight
    else:
        behind = [i for i, l in enumerate(lines) if l.startswith("global_store_short")]
        reads = sum(2 if l.startswith("ds_read2_") else 1 for l in lines[behind[0] - 200:behind[0]] if l.startswith("ds_read"))
        assert len(behind) == 8 and reads >= 8


@pytest.mark.parametrize("kernel,tile", [("direct", (1, 4, 4)), ("direct", (3, 2, 4)), ("shared", (1, 4, 4)), ("shared", (5, 4, 4))])
def test_epilogue_reads_a_tile_from_lds_before_it_stores(gemm_asm, kernel, tile):
    """A store is a branch, and what is read behind it waits by itself: of the four whole-line stores of a tile none has a read
    of LDS in front of it but the first.  (One by one, 512 columns to 11140 channels at 806 tokens took 25.9 us, 21.3 now.)"""
    pat = re.compile(rf"^_ZN.*gemm_prefill_{kernel}_kernelI" + "".join(f"Li{x}E" for x in tile) + "Lb0ELb0E.*:")
    start = next(i for i, l in enumerate(gemm_asm) if pat.match(l))
    end = next(i for i in range(start, len(gemm_asm)) if ".amdhsa_next_free_vgpr" in gemm_asm[i])
    lines = [l.strip() for l in gemm_asm[start:end]]
    last = max(i for i, l in enumerate(lines) if l.startswith("v_mfma_i32"))
    runs, run, read = [], 0, False
    for l in lines[last:]:
        if l.startswith("ds_write"):
            runs, run = runs + [run] if run else runs, 0
        elif l.startswith("ds_read"):
            read = True
        elif l.startswith("global_store_dwordx4"):
            if run and read:
                runs, run = runs + [run], 0
            run, read = run + 1, False
    runs.append(run)
    assert runs and all(n >= 4 for n in runs if n), runs
