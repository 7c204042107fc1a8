"""Builds libpeqa_hip.so (the C-ABI library) in-tree with hipcc for gfx950."""
import os
import re
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpeqa_hip.so")
SOURCES = ["peqa_api.hip", "peqa_quantize.hip", "peqa_small.hip", "peqa_gemm.hip", "peqa_gemm_r4.hip", "peqa_gemm_r6.hip",
           "peqa_gemm_r7.hip", "peqa_gemm_r8.hip", "peqa_gemv.hip", "peqa_dw.hip", "peqa_block.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-Rpass-analysis=kernel-resource-usage"]
# Kernels that queue global -> LDS DMA from inline assembly and count s_waitcnt vmcnt by hand: a
# register spill would add scratch loads and stores (also counted by vmcnt) that the hand count does
# not know about, so the build refuses any scratch use in them.
NO_SCRATCH = ("gemm_kernel", "gemm_bwd_pair_kernel", "gemm_multi_kernel", "gemv_kernel", "dw_kernel", "dw_multi_kernel")


def check_no_scratch(remarks):
    name = None
    bad = []
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split("[")[0].strip()
        elif "ScratchSize [bytes/lane]:" in line and name is not None:
            size = int(line.split("ScratchSize [bytes/lane]:")[1].split("[")[0])
            if size > 0 and any(k in name for k in NO_SCRATCH):
                bad.append("%s uses %d bytes of scratch per lane" % (name, size))
    return bad


# Wait states that gfx950 wants between an instruction that writes a register and one that reads it, where the hardware does not
# wait by itself.  The compiler keeps them between instructions that it emits itself; reads and writes in inline assembly are
# unknown to it, so the built code is looked at.  Of every rule: the readers, the writers, the registers, the wait states.
_MATRIX, _MEMORY = ("v_mfma", "v_smfmac"), ("global_", "buffer_", "flat_", "scratch_")
_RULES = (
    (lambda name: name.startswith(_MATRIX), lambda name: name.startswith("v_") and not name.startswith(_MATRIX), "va", 2),
    (lambda name: name.startswith(_MEMORY), lambda name: name.startswith("v_"), "s", 5),
    (lambda name: name.endswith("_dpp"), lambda name: name.startswith("v_") and not name.startswith(_MATRIX), "v", 2),
)
_REGISTERS = re.compile(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+)\b)")
_TARGET = re.compile(r"<(\S+?)(?:\+0x([0-9a-f]+))?>\s*$")


def _registers(operands, kinds):
    found = set()
    for operand in operands:
        for kind, lo, hi, one in _REGISTERS.findall(operand):
            if kind in kinds:
                found.update((kind, i) for i in range(int(lo or one), int(hi or one) + 1))
        if "s" in kinds and "vcc" in operand:
            found.add("vcc")
    return found


def early_reads(listing):
    """Instructions of a disassembly (llvm-objdump -d) that read a register too few wait states after it was written, on any
    path into them: one line of text each."""
    code, entry, function = [], {}, None                   # code: (function, address, mnemonic, operands, branch target)
    for line in listing.splitlines():
        label = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if label:
            function = label.group(2)
            entry[function] = int(label.group(1), 16)
        elif "//" in line and function is not None:
            text, _, tail = line.partition("//")
            mnemonic, _, operands = text.strip().partition(" ")
            target = _TARGET.search(tail) if "branch" in mnemonic else None
            code.append((function, int(tail.split(":")[0], 16), mnemonic, operands.split(","),
                         target and (target.group(1), int(target.group(2) or "0", 16))))
    index = {c[1]: i for i, c in enumerate(code)}
    jumps = {}
    for i, c in enumerate(code):
        if c[4]:
            jumps.setdefault(index[entry[c[4][0]] + c[4][1]], []).append(i)
    bad = []
    for i, (function, address, mnemonic, operands, _) in enumerate(code):
        for reads_here, writes_there, kinds, wanted in _RULES:
            if not reads_here(mnemonic):
                continue
            # everything but a destination is read (of a store or a load into LDS, the first operand too)
            reads = _registers(operands if kinds == "s" else operands[1:], kinds)
            front = [(i, 0)]                               # (instruction, wait states from its end to the reader)
            while front and reads:
                here, waited = front.pop()
                before = list(jumps.get(here, ()))
                if here > 0 and code[here - 1][0] == function and code[here - 1][2] not in ("s_branch", "s_endpgm", "s_setpc_b64"):
                    before.append(here - 1)
                for p in before:
                    _, at, name, ops, _ = code[p]
                    written = ops[:2] if "_co_" in name or "div_scale" in name else ops[:1]
                    if writes_there(name) and _registers(written, kinds) & reads:
                        bad.append("%s: %s at %x reads what %s at %x wrote, after %d wait states instead of %d" %
                                   (function, mnemonic, address, name, at, waited, wanted))
                    states = waited + (int(ops[0]) + 1 if name == "s_nop" else 1)
                    if states < wanted:
                        front.append((p, states))
    return bad


def _of_device_objects(lib, tool, *args):
    """What a tool of the toolchain prints of every code object in a library built here."""
    tools = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
    with tempfile.TemporaryDirectory() as tmp:
        name = os.path.basename(lib)
        shutil.copy(lib, tmp)
        subprocess.run([os.path.join(tools, "llvm-objdump"), "--offloading", name], cwd=tmp, check=True, stdout=subprocess.DEVNULL)
        objects = [f for f in sorted(os.listdir(tmp)) if "amdgcn" in f]
        return [subprocess.run([os.path.join(tools, tool), *args, f], cwd=tmp, check=True, stdout=subprocess.PIPE, text=True).stdout
                for f in objects]


def device_listings(lib):
    """Disassembly of every code object in a library built here."""
    return _of_device_objects(lib, "llvm-objdump", "-d")


def kernel_registers(lib):
    """Vector registers of a lane, accumulators among them, of every kernel in a library built here: {mangled name: number}."""
    found, name = {}, None
    for text in _of_device_objects(lib, "llvm-readelf", "--notes"):
        for line in text.splitlines():
            key, _, value = line.strip().partition(":")
            if key == ".name" and value.strip().startswith("_Z"):
                name = value.strip()
            elif key == ".vgpr_count":
                found[name] = int(value)
    return found


def _quiet(text):
    return "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l and "remark:" not in l)


def build(verbose=False, extra=(), jobs=None):
    """Every source is compiled (always: no time stamps are consulted) to an object of its own, in
    parallel, then the objects are linked into the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    if os.path.exists(LIB):
        os.remove(LIB)

    def compile_one(src):
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        cmd = [hipcc] + FLAGS + list(extra) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        return src, obj, r

    jobs = jobs or min(len(SOURCES), int(os.environ.get("MAX_JOBS", "8")), os.cpu_count() or 1)
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        results = list(pool.map(compile_one, SOURCES))
    remarks = ""
    for src, _, r in results:
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, _quiet(r.stdout)))
        remarks += r.stdout
    with open(os.path.join(OBJ, "remarks.txt"), "w") as f:     # registers, LDS and occupancy of every kernel
        f.write(remarks)
    bad = check_no_scratch(remarks)
    if bad:
        raise RuntimeError("register spills in kernels that count vmcnt by hand:\n" + "\n".join(bad))
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + [obj for _, obj, _ in results] + ["-o", LIB]
    if verbose:
        print(" ".join(link), flush=True)
    r = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + _quiet(r.stdout))
    early = [b for text in device_listings(LIB) for b in early_reads(text)]
    if early:
        os.remove(LIB)
        raise RuntimeError("reads too close behind the writes they depend on:\n" + "\n".join(early))
    out = _quiet(remarks)
    if verbose and out.strip():
        print(out)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
