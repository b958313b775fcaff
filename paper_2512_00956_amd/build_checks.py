"""Checks on the generated gfx950 assembly of the MXFP4 GEMMs that issue loads from inline asm.

The tiled one (csrc/mxfp4_gemm_frag.hip): its main-loop global loads are issued from inline asm with explicit vmcnt waits, so the compiler
does not know that their destination registers are written asynchronously.  The kernel is only
correct while
  (a) nothing in it spills to scratch,
  (b) every register of the two W sets has ONE physical assignment in the whole kernel (2 sets x
      CB x 4 fragment tuples + 2 x CB scale registers for a tile shape with CB column blocks per
      wave, each loaded at the same number of code sites): a second assignment would mean a
      register copy that may read a tuple whose load is still in flight,
  (c) the compiler adds no full drain (vmcnt(0) / lgkmcnt(0)) inside the pipelined loop, which
      holds exactly two K iterations and two barriers.
None of this can be said in the source, and a different compiler may break it silently, so the
build runs these checks on every compile and fails when one does not hold; the test suite runs
them again.

The canonical one (csrc/mxfp4_gemm_canon.hip) has no register destination in its asm, but its LDS
ring is filled behind the compiler's back.  It is only correct while every LDS read of a step stays
between the step's barrier and the next, with the explicit count of outstanding loads in front of
the barrier; it is only fast while nothing spills and nothing but the documented wait for the
scale loads drains the ring.

All kernels with matrix instructions: nothing interlocks their results against a read by another kind of instruction, so the
compiler counts wait states and adds s_nop.  It walks back from the read over every path, but each block only once: where a loop around the read is so
short that the walk reaches the instruction's block that way first, the direct path is not looked at any more, and the read
follows the product at once (seen in a kernel whose product ended a branch before a store to LDS, inside a loop over blocks of outputs: old values).
"""
from __future__ import annotations

import re
from collections import Counter


class InvariantError(RuntimeError):
    pass


def kernels(text: str) -> dict:
    """{kernel symbol: body} of every gemm_frag_kernel instantiation in the assembly."""
    parts = re.split(r"^(_ZN4wush\S*gemm_frag_kernel\S*):.*$", text, flags=re.M)
    return {parts[i]: parts[i + 1].split("s_endpgm")[0] for i in range(1, len(parts) - 1, 2)}


def check_lds_load_asm(text: str) -> None:
    """Direct-to-LDS loads issued from asm (csrc/mxfp4_gemm_frag.hip, csrc/mxfp4_gemm_canon.hip): each reads the m0 its own asm
    block wrote, with a wait state in between, and m0 has no other writer; no scalar address of one comes straight from a
    vector instruction (five wait states, which the compiler does not count for an asm)."""
    ins = [s for s in (line.split(";")[0].strip() for line in text.split("\n")) if s and not s.startswith((".", "#"))]
    loads = [k for k, s in enumerate(ins) if s.startswith("global_load_lds_")]
    if not loads:
        raise InvariantError("no direct-to-LDS load found")
    for k in loads:
        if not (ins[k - 2].startswith("s_mov_b32 m0,") and ins[k - 1].startswith("s_nop")):
            raise InvariantError(f"no wait state between the write of m0 and {ins[k]!r}: {ins[k - 2:k + 1]}")
        base = re.search(r"s\[(\d+):(\d+)\]", ins[k])
        for s in ins[max(0, k - 7):k]:
            m = re.match(r"v_read(?:first)?lane_b32 s(\d+),", s)
            if m and int(base.group(1)) <= int(m.group(1)) <= int(base.group(2)):
                raise InvariantError(f"{s!r} too close before {ins[k]!r}")
    if sum("m0" in re.findall(r"\w+", s) for s in ins) != len(loads):
        raise InvariantError("m0 is used outside the loads' asm blocks")


def shape(name: str):
    """(RB, CB) from the mangled template arguments ...ILb<f32>ELi<RB>ELi<CB>E..."""
    m = re.search(r"ILb[01]ELi(\d+)ELi(\d+)E", name)
    return int(m.group(1)), int(m.group(2))


def check_gemm_frag_asm(text: str, expected_kernels: int = 8) -> None:
    ks = kernels(text)
    if len(ks) != expected_kernels:
        raise InvariantError(f"expected {expected_kernels} gemm_frag_kernel instantiations, found {len(ks)}: {list(ks)}")
    for name, body in ks.items():
        RB, CB = shape(name)
        if "scratch_" in body:
            raise InvariantError(f"{name}: spills to scratch")
        frag = Counter(re.findall(r"global_load_dwordx4 (v\[\d+:\d+\])", body))
        scale = Counter(re.findall(r"global_load_dword (v\d+),", body))
        if len(frag) != 2 * CB * 4 or len(scale) != 2 * CB:
            raise InvariantError(f"{name}: {len(frag)} W fragment tuples and {len(scale)} scale registers "
                                 f"(expected {2 * CB * 4} and {2 * CB}): a W register changed its assignment")
        if len(set(frag.values())) != 1 or len(set(scale.values())) != 1:
            raise InvariantError(f"{name}: W registers are loaded at different numbers of code sites: {frag} {scale}")
        regs = [r for t in frag for r in range(*map(int, re.match(r"v\[(\d+):(\d+)\]", t).groups()))]
        if len(regs) != len(set(regs)):
            raise InvariantError(f"{name}: W fragment tuples overlap")
        m = re.search(r"Inner Loop Header.*?s_cbranch_scc1", body, flags=re.S)
        if not m:
            raise InvariantError(f"{name}: pipelined loop not found")
        loop = m.group(0)
        if loop.count("v_mfma_scale_f32_32x32x64_f8f6f4") != 2 * 4 * RB * CB:
            raise InvariantError(f"{name}: the loop does not hold two K iterations")
        if "vmcnt(0)" in loop or "lgkmcnt(0)" in loop:
            raise InvariantError(f"{name}: a full waitcnt drain inside the pipelined loop")
        if loop.count("s_barrier") != 2:
            raise InvariantError(f"{name}: {loop.count('s_barrier')} barriers in the loop (expected 2)")


def _loops(body: str) -> dict:
    """{loop header: [basic block, ...]} of the blocks the compiler annotates as belonging to a loop."""
    blocks = re.split(r"^(\.LBB\d+_\d+:.*|; %bb\.\d+:.*)$", body, flags=re.M)
    loops = {}
    for label, block in zip(blocks[1::2], blocks[2::2]):
        m = re.search(r"in Loop: Header=(BB\d+_\d+)", label)
        if not m and "Loop Header" in label:
            m = re.match(r"\.L(BB\d+_\d+):", label)
        if m:
            loops.setdefault(m.group(1), []).append(block)
    return loops


def check_gemm_canon_asm(text: str, expected_kernels: int = 20) -> None:
    parts = re.split(r"^(_ZN4wush\S*gemm_canon_kernel\S*):.*$", text, flags=re.M)
    ks = {parts[i]: parts[i + 1].split(".Lfunc_end")[0] for i in range(1, len(parts) - 1, 2)}
    if len(ks) != expected_kernels:
        raise InvariantError(f"expected {expected_kernels} gemm_canon_kernel instantiations, found {len(ks)}: {list(ks)}")
    for name, body in ks.items():
        WM, WN, RB, CB, ST = map(int, re.search(r"ILb[01]ELb[01]" + r"ELi(\d+)" * 5 + "E", name).groups())
        loads = WM * RB + WN * CB                    # direct loads per wavefront and step
        mma = RB * CB
        if "scratch_" in body:
            raise InvariantError(f"{name}: spills to scratch")
        loops = {h: b for h, b in _loops(body).items() if any("v_mfma_scale" in x for x in b)}
        if len(loops) != 2:
            raise InvariantError(f"{name}: {len(loops)} pipelined loops (expected the filling and the draining one)")
        for header, blocks in loops.items():
            where = f"{name}, loop {header}"
            whole = "".join(blocks)
            dwords = len(re.findall(r"ds_read_b32", whole)) + 2 * len(re.findall(r"ds_read2\w*_b32", whole))
            counts = (whole.count("v_mfma_scale"), whole.count("s_barrier"), whole.count("ds_read_b128"), dwords)
            if counts != (4 * mma, 1, 4 * (RB + CB), RB + CB):
                raise InvariantError(f"{where}: MFMAs, barriers, fragment and scale reads {counts} are not one step's")
            n_loads = whole.count("global_load_lds_")
            if n_loads not in (0, loads):
                raise InvariantError(f"{where}: {n_loads} direct loads (expected {loads} or none)")
            # the step's barrier: the explicit count right before it, the first issue's fragments and all scales right behind
            block = next(b for b in blocks if "s_barrier" in b)
            before, after = block.split("s_barrier")
            waits = re.findall(r"s_waitcnt ([^\n;]*)", before)
            count = (ST - 2) * loads if n_loads else 0
            if not waits or waits[-1].split() != [f"vmcnt({count})", "lgkmcnt(0)"] or "ds_read" in before:
                raise InvariantError(f"{where}: not vmcnt({count}) lgkmcnt(0), then the barrier: {waits}")
            first = len(re.findall(r"ds_read_b128", after))
            scales = len(re.findall(r"ds_read_b32", after)) + 2 * len(re.findall(r"ds_read2\w*_b32", after))
            if first < RB + CB or scales != RB + CB:
                raise InvariantError(f"{where}: a read of the step's first operands left its place behind the barrier")
            # the MFMAs: one block, no wait for loads in it, no LDS read once the last issue has begun
            multiply = [b for b in blocks if "v_mfma_scale" in b]
            pieces = "".join(multiply).split("v_mfma_scale")
            if len(multiply) != 1 or "vmcnt" in multiply[0]:
                raise InvariantError(f"{where}: the MFMAs are not one block free of waits for loads")
            if any("ds_read" in p for p in pieces[3 * mma + 1:]):
                raise InvariantError(f"{where}: an LDS read behind the last issue: it may belong to the next step")
            # full drains: with the scales' ds_write, and among the byte loads of a row's last scales
            for b in blocks:
                if "vmcnt(0)" in b and "s_barrier" not in b and "ds_write_b128" not in b and "global_load_ubyte" not in b \
                        and re.search(r"ds_read|global_load_lds", b):
                    raise InvariantError(f"{where}: a full drain of the ring")


# wait states between a matrix instruction and another kind's read of its result, by its shape: passes of four cycles + 4 (FP64: + 2)
_RESULT_WAIT = {"4x4x": 6, "16x16x128_f8f6f4": 8, "16x16x32_": 8, "32x32x64_f8f6f4": 12, "32x32x16_": 12, "f64_16x16x4": 18}
_TAKEN = 4            # what a taken branch costs at least


def _operand_regs(text: str) -> set:
    m = re.match(r"-?\|?([va])(?:\[(\d+):(\d+)\]|(\d+))", text)
    if not m:
        return set()
    lo, hi = (m.group(2), m.group(3)) if m.group(2) else (m.group(4), m.group(4))
    return {(m.group(1), r) for r in range(int(lo), int(hi) + 1)}


def _instructions(body: str):
    """[(mnemonic, operands, text)] of a kernel and {label: index of the instruction behind it}."""
    ins, labels = [], {}
    for line in body.split("\n"):
        s = line.split(";")[0].strip()
        label = re.match(r"([\w.$]+):$", s)
        if label:
            labels[label.group(1)] = len(ins)
        elif re.match(r"[a-z]", s):
            op, _, rest = s.partition(" ")
            ins.append((op, [x.strip() for x in re.split(r",\s*(?![^\[]*\])", rest)] if rest else [], s))
    return ins, labels


def check_mfma_result_waits(text: str) -> int:
    """Every path from a matrix instruction to the first other instruction that reads its result has the wait states it needs.  Returns the number
    of matrix instructions followed."""
    parts, followed = re.split(r"^(_Z\S+):.*$", text, flags=re.M), 0
    for name, body in zip(parts[1::2], parts[2::2]):
        ins, labels = _instructions(body.split(".Lfunc_end")[0])
        for at, (op, args, line) in enumerate(ins):
            if not op.startswith("v_mfma"):
                continue
            need = next((n for shape, n in _RESULT_WAIT.items() if shape in op), None)
            if need is None:
                raise InvariantError(f"{name}: no wait states known for {op}")
            result, seen, paths = _operand_regs(args[0]), {}, [(at + 1, 0)]
            while paths:
                k, waited = paths.pop()
                while k < len(ins) and waited < need and seen.get(k, need) > waited:
                    seen[k] = waited
                    o, a, s = ins[k]
                    if o == "s_endpgm":
                        break
                    if o.startswith("v_mfma"):            # interlocked; a later one's result has waits of its own
                        if _operand_regs(a[0]) & result:
                            break
                    elif not o.startswith("s_"):
                        stores = o.startswith(("ds_write", "global_store", "buffer_store", "flat_store", "scratch_store"))
                        if any(_operand_regs(x) & result for x in (a if stores else a[1:])):
                            raise InvariantError(f"{name}: {s!r} {waited} wait states behind {line!r}, {need} needed")
                    if o == "s_nop":
                        waited += int(a[0], 0) + 1
                    elif o == "s_branch":
                        k, waited = labels.get(a[0], len(ins)), waited + _TAKEN
                        continue
                    else:
                        if o.startswith("s_cbranch") and a[0] in labels:
                            paths.append((labels[a[0]], waited + _TAKEN))
                        waited += 1
                    k += 1
            followed += 1
    return followed
