"""CPU-side checks of the C-ABI library: it loads without a GPU and exports every symbol the
header declares; argument validation that needs no device returns the documented codes."""
import ctypes
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2110_13005_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _header_symbols():
    text = open(os.path.join(ROOT, "include", "axonn_stage.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(axonn_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = B.load()
    syms = _header_symbols()
    assert len(syms) >= 30
    for s in syms:
        assert hasattr(lib, s), "missing export: " + s
    assert sorted(B.EXPORTED_SYMBOLS) == syms, "binding and header disagree"


def test_half_precision_build_exports_the_same_symbols():
    """libaxonn_stage_fp16.so is the same C ABI over the other 16-bit element type."""
    from paper_2110_13005_amd import build as BLD
    lib = ctypes.CDLL(BLD.LIB_PATH_FP16)
    for s in _header_symbols():
        assert hasattr(lib, s), "missing export: " + s
    lib.axonn_element_type.restype = ctypes.c_int32
    assert lib.axonn_element_type() == 1 and B.load().axonn_element_type() == 0


def test_binding_holds_both_builds_and_routes_by_selection():
    """select_elem() switches the library that handle-free calls go to, the torch dtype and the rounding of the
    synthetic inputs; both libraries stay loaded, and each keeps an error message of its own."""
    import numpy as np
    import torch
    from paper_2110_13005_amd import inputs
    before = B.ELEM
    try:
        B.select_elem("bf16")
        lib_b = B.load()
        assert B.axonn_element_type() == 0 and B.torch_elem_dtype() == torch.bfloat16
        x = np.float32(1.0 + 2.0 ** -10)
        assert inputs.snap_elem(np.array([x]))[0] == np.float32(1.0)            # bfloat16 keeps 8 bits
        B.select_elem("fp16")
        lib_h = B.load()
        assert lib_h is not lib_b and B.load("bf16") is lib_b
        assert B.axonn_element_type() == 1 and B.torch_elem_dtype() == torch.float16
        assert inputs.snap_elem(np.array([x]))[0] == x                          # half precision keeps 11
        with pytest.raises(B.AxonnError) as e:
            B.axonn_tuning(99, 0)
        assert e.value.status == B.AXONN_EINVAL and b"99" in lib_h.axonn_last_error()
        assert b"99" not in lib_b.axonn_last_error()
        with pytest.raises(ValueError):
            B.select_elem("fp8")
    finally:
        B.select_elem(before)


def test_argument_validation_without_device():
    lib = B.load()
    assert lib.axonn_stage_create(None, None) == B.AXONN_EINVAL
    assert b"null" in lib.axonn_last_error()
    out = ctypes.c_void_p()
    cfg = B.axonn_stage_config(2, 256, 3, 1024, 128, 2, 4, 4, 1e-5, 0, 1, 0, 0)   # 256 % 3 != 0
    assert lib.axonn_stage_create(ctypes.byref(cfg), ctypes.byref(out)) == B.AXONN_EINVAL
    cfg = B.axonn_stage_config(2, 2048, 8, 8192, 128, 2, 4, 4, 1e-5, 0, 1, 0, 0)  # head dim 256
    assert lib.axonn_stage_create(ctypes.byref(cfg), ctypes.byref(out)) == B.AXONN_EUNSUPPORTED
    assert b"head dim" in lib.axonn_last_error()
    cfg = B.axonn_stage_config(2, 256, 4, 1024, 128, 2, 4, 5, 1e-5, 0, 1, 0, 0)   # pipeline_limit > M
    assert lib.axonn_stage_create(ctypes.byref(cfg), ctypes.byref(out)) == B.AXONN_EINVAL
    cfg = B.axonn_stage_config(2, 256, 4, 1024, 3, 1, 4, 4, 1e-5, 0, 1, 0, 0)     # 3 tokens
    assert lib.axonn_stage_create(ctypes.byref(cfg), ctypes.byref(out)) == B.AXONN_EUNSUPPORTED
    cfg = B.axonn_stage_config(4, 256, 4, 1024, 128, 2, 4, 4, 1e-5, 0, 1, 0, 0, 3)  # stride 3, 4 layers
    assert lib.axonn_stage_create(ctypes.byref(cfg), ctypes.byref(out)) == B.AXONN_EINVAL
    assert b"ckpt_stride" in lib.axonn_last_error()
    with pytest.raises(B.AxonnError) as e:
        B.axonn_gemm_bf16(1, 0, 0, 64, 64, 60, 1, 64, 1, 64, 1, 64)          # K % 8 != 0
    assert e.value.status == B.AXONN_EUNSUPPORTED
    with pytest.raises(B.AxonnError) as e:
        B.axonn_gemm_bf16(0, 1, 0, 64, 64, 64, 1, 64, 1, 64, 1, 64)          # layout not built
    assert e.value.status == B.AXONN_EUNSUPPORTED
    with pytest.raises(B.AxonnError) as e:
        B.axonn_gemm_wgrad_colsum(3, 64, 64, 64, 1, 64, 1, 64, 1, 64, 1, 1)     # not an accumulating epilogue
    assert e.value.status == B.AXONN_EINVAL
    with pytest.raises(B.AxonnError) as e:
        B.axonn_gemm_wgrad_colsum(5, 64, 64, 64, 1, 64, 1, 64, 1, 64, None, 1)  # no place for the column sums
    assert e.value.status == B.AXONN_EINVAL
    with pytest.raises(B.AxonnError) as e:
        B.axonn_gemm_wgrad_colsum(5, 64, 64, 64, 1, 64, 1, 56, 1, 64, 1, 1)     # ldb < N
    assert e.value.status == B.AXONN_EINVAL
    with pytest.raises(B.AxonnError) as e:
        B.axonn_adam_bucket(8, 1, 1, 1, 1, 1, 1e-3, 0.9, 0.95, 1e-8, 0.0, 0, 1.0)  # step 0
    assert e.value.status == B.AXONN_EINVAL
    with pytest.raises(B.AxonnError) as e:
        B.axonn_attention_fwd(1, 128, 4, 200, 1, 1, 1)
    assert e.value.status == B.AXONN_EUNSUPPORTED


def _llvm_tool(name):
    path = shutil.which(name) or "/opt/rocm/llvm/bin/" + name
    if not os.path.exists(path):
        pytest.skip("no " + name)
    return path


def _code_objects(lib_path, tmp_path):
    """The gfx950 code objects of a built library, as files."""
    blob = open(lib_path, "rb").read()
    magic, out = b"__CLANG_OFFLOAD_BUNDLE__", []
    at = blob.find(magic)
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", blob, at + len(magic)), at + len(magic) + 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + name_len]
            p += 24 + name_len
            if b"gfx950" in triple and size:
                out.append(tmp_path / ("code_object_%d" % len(out)))
                out[-1].write_bytes(blob[at + off:at + off + size])
        at = blob.find(magic, at + 1)
    return out


def _kernel_scratch(lib_path, tmp_path):
    """{mangled kernel name: bytes of scratch memory per lane} of a built library, from its own code objects' notes."""
    readelf, out = _llvm_tool("llvm-readelf"), {}
    for obj in _code_objects(lib_path, tmp_path):
        notes = subprocess.run([readelf, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"^ +\.name: +(_Z\S+)$", notes, flags=re.M)
        scratch = re.findall(r"^ +\.private_segment_fixed_size: +(\d+)$", notes, flags=re.M)
        assert len(names) == len(scratch)
        out.update(zip(names, map(int, scratch)))
    return out


@pytest.mark.parametrize("elem", ["bf16", "fp16"])
def test_kernels_keep_their_loops_out_of_scratch_memory(elem, tmp_path):
    """A register spilled inside a GEMM's k loop or the LayerNorm backward's row loop waits for every load in flight at
    each reload."""
    from paper_2110_13005_amd import build as BLD
    scratch = {k: v for k, v in _kernel_scratch(BLD.VARIANTS[elem][0], tmp_path).items() if "gemm_" in k or "layernorm_" in k}
    assert len(scratch) > 50
    assert not {k: v for k, v in scratch.items() if v}


@pytest.mark.parametrize("elem", ["bf16", "fp16"])
def test_attention_kernels_keep_out_of_scratch_memory(elem, tmp_path):
    """A register spilled inside an attention kernel's loop waits for every copy in flight at its reload.  No such kernel uses
    scratch memory."""
    from paper_2110_13005_amd import build as BLD
    scratch = {k: v for k, v in _kernel_scratch(BLD.VARIANTS[elem][0], tmp_path).items() if "attn_" in k}
    assert len(scratch) > 20
    assert not {k: v for k, v in scratch.items() if v}


@pytest.mark.parametrize("elem", ["bf16", "fp16"])
def test_attention_kernels_leave_room_for_their_second_workgroup(elem, tmp_path):
    """Where two workgroups of four waves share a CU (the forward and dQ kernels up to 128 columns, the dK / dV ones up to 64),
    each takes half of a SIMD's 512 registers per lane and of 160 KB of LDS at most."""
    from paper_2110_13005_amd import build as BLD
    readelf, seen = _llvm_tool("llvm-readelf"), 0
    for obj in _code_objects(BLD.VARIANTS[elem][0], tmp_path):
        notes = subprocess.run([readelf, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"^ +- \.agpr_count:", notes, flags=re.M)[1:]:
            name = re.search(r"\.name: +\S*?attn_(fwd|bwd_dq|bwd_dkdv|bwd_both)_kernelILi(\d+)E", kernel)
            if name and int(name.group(2)) <= (128 if name.group(1) in ("fwd", "bwd_dq") else 64):
                seen += 1
                assert int(re.search(r"\.vgpr_count: +(\d+)", kernel).group(1)) <= 256, name.group(0)
                assert int(re.search(r"\.group_segment_fixed_size: +(\d+)", kernel).group(1)) <= 80 * 1024, name.group(0)
    assert seen >= 12


def _registers(operand):
    m = re.match(r"^[-|]*([va])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return set()
    lo, hi = (int(m.group(2)),) * 2 if m.group(2) else (int(m.group(3)), int(m.group(4)))
    return {(m.group(1), i) for i in range(lo, hi + 1)}


@pytest.mark.parametrize("elem", ["bf16", "fp16"])
def test_attention_mfmas_keep_their_distances(elem, tmp_path):
    """The dK / dV kernels' MFMAs are inline assembly, for which the compiler keeps no distances.  In program order: two wait
    states between a vector instruction's result and an MFMA that reads it; between an MFMA's result and another kind of
    instruction that touches it two MFMAs or eleven wait states."""
    from paper_2110_13005_amd import build as BLD
    objdump, kernels, near = _llvm_tool("llvm-objdump"), 0, []
    for obj in _code_objects(BLD.VARIANTS[elem][0], tmp_path):
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*attn_bwd_(?:dkdv|both)\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, flags=re.M | re.S):
            kernels += 1
            pos = mfmas = 0
            by_vector, by_mfma = {}, {}
            for line in body.splitlines():
                op, _, rest = line.split("//")[0].strip().partition(" ")
                operands = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
                if op == "s_nop":
                    pos += int(operands[0], 0)
                elif op.startswith("v_mfma"):
                    used = set().union(*(_registers(x) for x in operands[1:]))
                    near += [(name, line) for r in used if pos - by_vector.get(r, -9) - 1 < 2]
                    for r in _registers(operands[0]):
                        by_mfma[r] = (pos, mfmas)
                        by_vector.pop(r, None)
                    mfmas += 1
                elif op.startswith(("v_", "ds_", "buffer_", "global_", "scratch_")):
                    for r in set().union(*(_registers(x) for x in operands)):
                        at, n = by_mfma.get(r, (-99, -9))
                        if pos - at - 1 < 11 and mfmas - n - 1 < 2:
                            near.append((name, line))
                    for r in _registers(operands[0]):
                        by_mfma.pop(r, None)
                        by_vector.pop(r, None)
                        if op.startswith("v_"):
                            by_vector[r] = pos
                pos += 1
    assert kernels >= 12 and not near, near[:4]


_SETTLED, _READABLE = 12, 2


def _instructions(body):
    """[(address, opcode, operands, target address or None)] of a function's listing."""
    out = []
    for text, at in re.findall(r"^\s+(\S[^\n]*?)\s*// ([0-9A-F]+):", body, flags=re.M):
        op, _, rest = text.strip().partition(" ")
        operands = [x.strip() for x in re.split(r",(?![^\[]*\])", rest)]
        at, target = int(at, 16), None
        if op.startswith(("s_branch", "s_cbranch")):
            offset = int(operands[0].split()[0], 0)
            target = at + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), op
        out.append((at, op, operands, target))
    return out


def _near_mfmas(body):
    """The instructions of a function that stand too near to what they read, along any path (jumps taken and not, loops any
    number of times): fewer than two wait states behind a vector instruction whose result an MFMA takes; fewer than twelve, and
    fewer than two MFMAs, behind an MFMA whose result another kind of instruction touches or another MFMA multiplies."""
    code = _instructions(body)
    index = {at: i for i, (at, _, _, _) in enumerate(code)}
    starts = {0} | {index[t] for _, _, _, t in code if t is not None}
    starts |= {i + 1 for i, (_, op, _, t) in enumerate(code) if t is not None or op == "s_endpgm"}
    known, todo, near = {0: ({}, {})}, [0], set()
    while todo:
        i = todo.pop()
        vector, mfma = (dict(x) for x in known[i])      # register -> states since; register -> (states, MFMAs) since
        while True:
            _, op, operands, target = code[i]
            regs = [_registers(x) for x in operands]
            states, is_mfma = 1, op.startswith("v_mfma")
            if op == "s_nop":
                states += int(operands[0], 0)
            elif is_mfma:
                near |= {i for r in set().union(*regs[1:4]) if r in vector} | {i for r in regs[1] | regs[2] if r in mfma}
            elif op.startswith(("v_", "ds_", "buffer_", "global_", "scratch_")):
                near |= {i for r in set().union(*regs) if r in mfma}
            vector = {r: n + states for r, n in vector.items() if n + states < _READABLE}
            mfma = {r: (n + states, m + is_mfma) for r, (n, m) in mfma.items() if n + states < _SETTLED and m + is_mfma < 2}
            if is_mfma or op.startswith(("v_", "ds_", "buffer_", "global_", "scratch_")):
                for r in regs[0]:
                    vector.pop(r, None)
                    mfma.pop(r, None)
                    if is_mfma:
                        mfma[r] = (0, 0)
                    elif op.startswith("v_"):
                        vector[r] = 0
            nexts = ([] if op in ("s_branch", "s_endpgm") else [i + 1]) + ([index[target]] if target is not None else [])
            if len(nexts) == 1 and nexts[0] == i + 1 and i + 1 not in starts:
                i += 1
                continue
            for n in nexts:
                old = known.get(n)
                new = (vector, mfma)
                if old:
                    new = ({r: min(x.get(r, 99) for x in (old[0], vector)) for r in old[0].keys() | vector.keys()},
                           {r: tuple(min(p) for p in zip(old[1].get(r, (99, 99)), mfma.get(r, (99, 99))))
                            for r in old[1].keys() | mfma.keys()})
                if new != old:
                    known[n] = tuple(dict(x) for x in new)
                    todo.append(n)
            break
    return [code[i] for i in sorted(near)]


def _listing(lines):
    return "".join("\t%s // %012X: 00000000\n" % (x, 4 * i) for i, x in enumerate(lines))


def test_distances_are_counted_along_every_path():
    """The scan below on listings in which the distance is one too short, or just enough: in a row, over a loop's back edge, over a
    jump around what lies between."""
    mfma, use = "v_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], v[20:23], v[0:15]", "v_mul_f32_e32 v40, v15, v15"
    def near(*lines):
        return bool(_near_mfmas(_listing(list(lines) + ["s_endpgm"])))
    assert near(mfma, "s_nop 10", use) and not near(mfma, "s_nop 11", use)
    assert near(mfma, *["s_add_i32 s0, s0, 1"] * 11, use) and not near(mfma, *["s_add_i32 s0, s0, 1"] * 12, use)
    other = "v_mfma_f32_32x32x16_bf16 a[0:15], v[16:19], v[20:23], a[0:15]"
    assert near(mfma, other, use) and not near(mfma, other, other, use)
    assert near("v_mov_b32_e32 v17, v50", "s_nop 0", mfma) and not near("v_mov_b32_e32 v17, v50", "s_nop 1", mfma)
    assert near(mfma, "s_nop 10", "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[20:23], a[0:15]")
    # the loop's first instruction reads what its last MFMA left: 12 in the first round, 2 from the second on
    assert near("s_nop 15", use, "s_nop 15", mfma, "s_nop 0", "s_cbranch_scc1 65531 <f+0x4>", "s_nop 15")
    assert not near("s_nop 15", use, "s_nop 15", mfma, "s_nop 11", "s_cbranch_scc1 65531 <f+0x4>", "s_nop 15")
    # the distance lies behind a jump around it
    assert near(mfma, "s_cbranch_scc1 1 <f+0xc>", "s_nop 11", use)
    assert not near(mfma, "s_cbranch_scc1 1 <f+0xc>", "s_nop 11", "s_nop 10", use)
    # what lies behind an unconditional jump is not reached from in front of it
    assert not near(mfma, "s_branch 1 <f+0xc>", use, "s_nop 11", use)


@pytest.mark.parametrize("elem", ["bf16", "fp16"])
def test_attention_mfma_distances_along_every_path(elem, tmp_path):
    """The dK / dV kernels' MFMAs are inline assembly, for which the compiler keeps no distances: two wait states, and twelve or two
    MFMAs (see _near_mfmas), whichever way the kernel takes.  Twelve are what the compiler itself puts between such an MFMA and
    the use of its result."""
    from paper_2110_13005_amd import build as BLD
    objdump, kernels = _llvm_tool("llvm-objdump"), 0
    for obj in _code_objects(BLD.VARIANTS[elem][0], tmp_path):
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*attn_bwd_(?:dkdv|both)\S*)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, flags=re.M | re.S):
            kernels += 1
            near = _near_mfmas(body)
            assert not near, (name, [(hex(at), op, operands) for at, op, operands, _ in near[:4]])
    assert kernels >= 12
