"""CPU-side checks of the C ABI: the library loads, exports what include/atomo.h and include/atomo_bench.h
declare, and the host-side argument validation answers without touching a GPU."""
import ctypes as C
import os
import re
import struct
import subprocess
import sys

import msgpack
import pytest

from paper_1806_04090_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols(header="atomo.h"):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(atomo_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = declared_symbols()
    assert {"atomo_encode_svd", "atomo_encode_entrywise", "atomo_probabilities", "atomo_decode"} <= set(names)
    bench = declared_symbols("atomo_bench.h")
    assert {"atomo_profile_enable", "atomo_profile_read", "atomo_measure_mfma_fp32", "atomo_last_counters"} == set(bench)
    assert not set(bench) & set(names)                       # the method's header holds no measurement call
    L = binding.lib()
    for name in names + bench:
        assert hasattr(L, name), name


def test_strerror_and_null_arguments():
    L = binding.lib()
    assert L.atomo_strerror(0) == b"ok"
    for code in (-1, -2, -3, -4, -5):
        assert L.atomo_strerror(code) not in (b"ok", b"unknown status")
    assert L.atomo_create(None, 0) == binding.ATOMO_EINVAL
    assert L.atomo_destroy(None) == binding.ATOMO_EINVAL
    assert L.atomo_reserve(None, 10) == binding.ATOMO_EINVAL
    assert L.atomo_status(None, None, None) == binding.ATOMO_EINVAL
    offs = (C.c_int64 * 2)(0, 4)
    assert L.atomo_probabilities(None, None, offs, 1, 1.0, None, None) == binding.ATOMO_EINVAL
    assert L.atomo_encode_svd(None, None, 1, 1.0, 0, 0, None, None, None, None, None) == binding.ATOMO_EINVAL
    assert L.atomo_encode_entrywise(None, None, 1.0, 0, 0, None, None, None) == binding.ATOMO_EINVAL
    assert L.atomo_decode(None, 0, None, 1, 1.0, None, 0, None) == binding.ATOMO_EINVAL


def test_workspace_queries_are_host_only():
    L = binding.lib()
    mats = (binding.atomo_mat * 2)(binding.atomo_mat(512, 4608, 4608, None), binding.atomo_mat(64, 27, 27, None))
    nbytes = C.c_size_t(0)
    assert L.atomo_svd_workspace_bytes(mats, 2, C.byref(nbytes)) == 0
    assert nbytes.value > 512 * (4608 + 512) * 4
    bad = (binding.atomo_mat * 1)(binding.atomo_mat(4096, 4096, 4096, None))
    assert L.atomo_svd_workspace_bytes(bad, 1, C.byref(nbytes)) == binding.ATOMO_EINVAL
    assert L.atomo_entrywise_workspace_bytes(11_173_962, C.byref(nbytes)) == 0
    assert nbytes.value > 70_000
    assert L.atomo_entrywise_workspace_bytes(0, C.byref(nbytes)) == binding.ATOMO_EINVAL
    assert L.atomo_entrywise_workspace_bytes(1 << 32, C.byref(nbytes)) == binding.ATOMO_EINVAL


def test_scratch_memory_of_a_short_gradient_is_for_its_records():
    # 5 MiB of atomo_encode_entrywise_noalloc hold the state of a search and the records: what a long gradient alone needs is not in there
    nbytes = C.c_size_t(0)
    for n in (16_385, 1 << 20, 1 << 24):
        assert binding.lib().atomo_entrywise_workspace_bytes(n, C.byref(nbytes)) == 0
        steps = (n + 1023) // 1024 * 4
        assert nbytes.value < 288 * steps + steps + 8 * (n // 4096 + 512) + 90_000, n     # records, counts, open draws, histograms and the rest


def test_no_fallback_without_a_gpu():
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is visible")
    with pytest.raises(RuntimeError):
        binding.Context(0)


def test_struct_layouts_match_the_header(tmp_path):
    """The ctypes mirrors in the binding against include/atomo.h as the host C compiler lays it out."""
    import shutil
    import subprocess
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no host C compiler")
    structs = [binding.atomo_mat, binding.atomo_svd_msg, binding.atomo_ew_msg, binding.atomo_lq_msg,
               binding.atomo_svd_options]
    lines = ["#include <stdio.h>", "#include <stddef.h>", '#include "atomo.h"', "int main(void) {"]
    for st in structs:
        lines.append(f'  printf("{st.__name__} size %zu\\n", sizeof({st.__name__}));')
        for name, _ in st._fields_:
            lines.append(f'  printf("{st.__name__} {name} %zu\\n", offsetof({st.__name__}, {name}));')
    lines += ["  return 0;", "}"]
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run([cc, "-std=c99", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    seen = {}
    for line in out:
        if line:
            st, field, value = line.split()
            seen[(st, field)] = int(value)
    for st in structs:
        assert seen[(st.__name__, "size")] == C.sizeof(st), st.__name__
        for name, _ in st._fields_:
            assert seen[(st.__name__, name)] == getattr(st, name).offset, (st.__name__, name)
    # and the header declares no field that the binding leaves out
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "atomo.h")).read(), flags=re.S)
    for st in structs:
        body = re.search(r"typedef struct %s \{(.*?)\} %s;" % (st.__name__, st.__name__), text, flags=re.S).group(1)
        declared = [part.replace("*", " ").split()[-1] for stmt in body.split(";") if stmt.strip()
                    for part in stmt.split(",")]
        assert declared == [name for name, _ in st._fields_], st.__name__


def test_a_call_that_runs_out_of_host_memory_returns_a_status():
    # the planners allocate; nothing may be thrown through the C interface
    code = f"""
import ctypes as C, resource
L = C.CDLL({binding.LIB_PATH!r})
n = 2_000_000
class Mat(C.Structure):
    _fields_ = [("rows", C.c_int32), ("cols", C.c_int32), ("ld", C.c_int64), ("data", C.c_void_p)]
mats = (Mat * n)()
for j in range(n):
    mats[j].rows, mats[j].cols = 64, 576
size = C.c_size_t(0)
used = [int(x.split()[1]) for x in open("/proc/self/status") if x.startswith("VmSize")][0] * 1024
resource.setrlimit(resource.RLIMIT_AS, (used + (200 << 20), resource.RLIM_INFINITY))
assert L.atomo_svd_workspace_bytes(mats, n, C.byref(size)) == {binding.ATOMO_ENOMEM}
assert L.atomo_svd_workspace_bytes(mats, 10, C.byref(size)) == 0 and size.value > 0
"""
    done = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stderr


def kernel_records():
    """What the compiler notes about each kernel of the library (the metadata notes of the code objects in it)."""
    data = open(binding.LIB_PATH, "rb").read()
    found = {}
    for note in re.finditer(rb"AMDGPU\0\0", data):
        name_size, size, kind = struct.unpack("<III", data[note.start() - 12:note.start()])
        if (name_size, kind) == (7, 32):
            for record in msgpack.unpackb(data[note.end():note.end() + size])["amdhsa.kernels"]:
                found[record[".name"]] = record
    return found


def test_the_decode_of_svd_messages_keeps_its_registers():
    # registers of these kernels that go to scratch memory are written to HBM beside the outputs that bound them
    tiles = {name: r for name, r in kernel_records().items() if "decode_svd_tiles" in name}
    assert len(tiles) == 4
    for name, r in tiles.items():
        assert r[".private_segment_fixed_size"] == 0 and r[".vgpr_spill_count"] == 0, name


def test_the_reduction_to_tridiagonal_form_keeps_its_registers():
    # the matrix lies in registers there; scratch memory of one class of sizes would be set up by every launch
    steps = {name: r for name, r in kernel_records().items() if "direct_tridiagonal" in name or "direct_tail" in name}
    assert len(steps) == 4
    for name, r in steps.items():
        assert r[".private_segment_fixed_size"] == 0 and r[".vgpr_spill_count"] == 0, name


TRANSCENDENTAL = ("v_rcp_", "v_rsq_", "v_sqrt_", "v_exp_", "v_log_", "v_sin_", "v_cos_")


def registers(operand):
    """Vector registers that an operand of a disassembled instruction names."""
    m = re.match(r"-?\|?v(?:\[(\d+):(\d+)\]|(\d+))", operand)
    return set() if not m else {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def too_early(code):
    """Of a list of (instruction, operands, address): the products with a broadcast operand, and what stands in front of each of them, on
    some path, with fewer wait states between than it takes.  Two after a vector instruction that writes the broadcast operand, five
    after one that writes EXEC, one after a transcendental one that writes any operand, 18 after a matrix instruction that does."""
    sources = {}
    for i, (op, args, addr) in enumerate(code):
        if op.startswith(("s_branch", "s_cbranch")):
            offset = int(args.split()[0])
            sources.setdefault(addr + 4 + 4 * (offset - 65536 if offset >= 32768 else offset), []).append(i)

    def in_front(i, states):
        """(instruction, wait states between it and instruction i) for all with fewer than `states`"""
        most, left = {}, [(i, 0)]
        while left:
            at, between = left.pop()
            before = list(sources.get(code[at][2], []))
            if at > 0 and code[at - 1][0] not in ("s_branch", "s_endpgm"):
                before.append(at - 1)
            for j in before:
                if between < most.get(j, states):
                    most[j] = between
                    left.append((j, between + (int(code[j][1]) + 1 if code[j][0] == "s_nop" else 1)))
        return most.items()

    found, products = [], 0
    for i, (op, args, addr) in enumerate(code):
        if op != "v_fmac_f64_dpp":
            continue
        products += 1
        operands = [registers(x.strip()) for x in args.split(" row_")[0].split(",")]
        broadcast, all_of_them = operands[1], set().union(*operands)
        for j, between in in_front(i, 18):
            what, how = code[j][0], [x.strip() for x in code[j][1].split(",")]
            if not what.startswith("v_"):
                continue
            written = registers(how[0])
            if "_swap" in what:                                  # (v_swap, v_permlane16_swap, v_permlane32_swap)
                written |= registers(how[1])
            if (between < 2 and written & broadcast or between < 5 and (what.startswith("v_cmpx") or how[0].startswith("exec"))
                    or between < 1 and what.startswith(TRANSCENDENTAL) and written & all_of_them
                    or what.startswith(("v_mfma", "v_smfma")) and written & all_of_them):
                found.append((hex(addr), op, args, code[j]))
    return found, products


def test_products_with_a_broadcast_operand_wait_for_it(tmp_path):
    """v_fmac_f64 with row_newbcast comes from inline assembly (svd_device.h), for which the compiler keeps no wait states."""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no disassembler")
    data = open(binding.LIB_PATH, "rb").read()
    products = 0
    for at in (m.start() for m in re.finditer(rb"\x7fELF\x02", data)):
        if struct.unpack_from("<H", data, at + 18)[0] != 224:    # EM_AMDGPU
            continue
        obj = tmp_path / "code.o"
        obj.write_bytes(data[at:])
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True, text=True).stdout
        if "v_fmac_f64_dpp" not in text:
            continue
        code = []
        for line in text.split("\n"):
            m = re.match(r"\s+(\S+)(.*?)// ([0-9A-F]+):", line)
            if m:
                code.append((m[1], m[2].strip(), int(m[3], 16)))
        found, here = too_early(code)
        assert not found, found[:3]
        products += here
    assert products > 100


PRODUCT = "v[0:1], -v[2:3], v[4:5] row_newbcast:3 row_mask:0xf bank_mask:0xf"


@pytest.mark.parametrize("wrong, before", [
    (True, [("v_add_f64", "v[2:3], v[6:7], v[8:9]")]),
    (True, [("v_mov_b32_e32", "v3, v9"), ("s_nop", "0")]),
    (False, [("v_mov_b32_e32", "v3, v9"), ("s_nop", "1")]),
    (False, [("v_mov_b32_e32", "v3, v9"), ("v_mov_b32_e32", "v10, v11"), ("v_mov_b32_e32", "v10, v11")]),
    (False, [("v_add_f64", "v[4:5], v[6:7], v[8:9]")]),
    (True, [("v_permlane16_swap_b32_e32", "v12, v3"), ("s_nop", "0")]),
    (True, [("v_swap_b32", "v2, v12")]),
    (False, [("v_permlane32_swap_b32_e32", "v12, v3"), ("s_nop", "1")]),
    (True, [("v_cmpx_gt_u32_e64", "exec, v20, v21"), ("s_nop", "3")]),
    (False, [("v_cmpx_gt_u32_e64", "exec, v20, v21"), ("s_nop", "4")]),
    (True, [("v_rcp_f64_e32", "v[4:5], v[6:7]")]),
    (False, [("v_rcp_f64_e32", "v[4:5], v[6:7]"), ("s_nop", "0")]),
    (True, [("v_mfma_f64_16x16x4_f64", "v[0:7], v[8:9], v[10:11], v[0:7]"), ("s_nop", "15")]),
    (True, [("v_mov_b32_e32", "v3, v9"), ("s_branch", "1"), ("v_mov_b32_e32", "v30, v31")]),    # (behind the branch: the product)
    (False, [("v_mov_b32_e32", "v3, v9"), ("s_branch", "2"), ("v_mov_b32_e32", "v30, v31")]),   # (never reached from it)
])
def test_what_is_too_early_in_front_of_a_broadcast_is_found(wrong, before):
    code = [("s_nop", "7", 0), ("s_nop", "7", 4)]
    for op, args in before + [("v_fmac_f64_dpp", PRODUCT), ("s_endpgm", "")]:
        code.append((op, args, 4 * len(code)))
    found, products = too_early(code)
    assert products == 1 and bool(found) == wrong


def test_lanes_that_exchange_values_through_lds_have_fences():
    # the wave's barrier alone does not keep the compiler from reusing what a lane stored itself, nor from moving a load over it
    csrc = os.path.join(ROOT, "paper_1806_04090_amd", "csrc")
    found = []
    for name in sorted(os.listdir(csrc)):
        text = re.sub(r"//.*", "", open(os.path.join(csrc, name)).read())
        for m in re.finditer(r"__builtin_amdgcn_wave_barrier", text):
            around = [line.strip() for line in text[:m.start()].split("\n")[-2:-1] + text[m.end():].split("\n")[1:2]]
            found.append((name, around))
    assert found
    for name, around in found:
        assert ["RELEASE" in around[0], "ACQUIRE" in around[1]] == [True, True], (name, around)
