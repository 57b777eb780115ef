"""Build libburstattn.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libburstattn.so")
SOURCES = ["api.hip", "fwd.hip", "bwd.hip", "elementwise.hip", "lm_head.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffast-math", "-fno-finite-math-only",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def check_resources(remarks, src):
    """The kernels are written to live in registers: a kernel that spills vector registers or touches
    scratch memory (a dynamically indexed struct does that silently) runs several times slower, so
    the build refuses it.  `remarks` is hipcc's -Rpass-analysis=kernel-resource-usage output."""
    name = None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split("[")[0].strip()
        for what in ("ScratchSize [bytes/lane]:", "VGPRs Spill:"):
            if what in line and int(line.split(what)[1].split("[")[0]) != 0:
                raise RuntimeError(f"{src}: kernel {name} has {line.split('remark:')[1].strip()}")


def _scalar_registers(operand):
    """The 32-bit scalar registers that an operand names."""
    m = re.fullmatch(r"s(\d+)|s\[(\d+):(\d+)\]", operand)
    if m:
        return {f"s{i}" for i in range(int(m[1] or m[2]), int(m[1] or m[3]) + 1)}
    return {"vcc_lo", "vcc_hi"} if operand == "vcc" else {operand} if operand in ("vcc_lo", "vcc_hi", "m0") else set()


def check_load_addresses(assembly, src):
    """A memory instruction may read a scalar register five wait states after a vector instruction wrote it, and load to LDS one
    after m0 was written.  The compiler keeps these distances between its own instructions and does not look into assembly
    statements, which the direct loads to LDS are: the build refuses a load that could come too early on any path, instead of
    leaving a tile read from a stale address."""
    code = []                       # (operation, operands), labels as (None, name)
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            code.append((None, line[:-1]))
        elif line and not line.startswith("."):
            op, *rest = line.split(None, 1)
            code.append((op, [x.strip() for x in rest[0].split(",")] if rest else []))
    jumps = {}                      # label: the branches that go there
    for i, (op, args) in enumerate(code):
        if op and op.startswith(("s_branch", "s_cbranch")):
            jumps.setdefault(args[0], []).append(i)

    def early(start, address, m0, states):
        """Whether one of the instructions before `start`, of which `states` wait states are over, is too near."""
        for i in range(start - 1, -1, -1):
            if states >= 5 or not (address or m0):
                break
            op, args = code[i]
            if op is None:
                if any(early(j + 1, address, m0, states) for j in jumps.get(args, ())):
                    return True
                continue
            if op in ("s_branch", "s_endpgm") and i + 1 < start:
                break               # (what stands behind it is reached through its label only)
            written = _scalar_registers(args[0]) if args and not op.startswith(("s_cmp", "s_bitcmp")) else set()
            if len(args) > 1 and ("_co_" in op or op.startswith(("v_mad_u64", "v_mad_i64", "v_div_scale"))):
                written |= _scalar_registers(args[1])
            if op.startswith("v_") and written & address or m0 and "m0" in written:
                return True
            if op.startswith("s_"):
                address = address - written    # (the scalar unit waits for a vector instruction's result by itself)
            m0 = False
            states += 1 + int(args[0], 0) if op == "s_nop" else 1
        return False

    found = 0
    for i, (op, args) in enumerate(code):
        if op and op.startswith("global_load_lds"):
            found += 1
            address = _scalar_registers(args[1].split()[0])
            if early(i, address, True, 0):
                raise RuntimeError(f"{src}: a vector instruction writes the address of a load to LDS less than five wait states "
                                   f"before it, or m0 is written right before: {op} {', '.join(args)}")
    return found


def build(verbose=False, extra_flags=(), out_path=None, tag=""):
    """Compile every source to an object (in parallel) and link the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build", tag) if tag else os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    temps = tempfile.TemporaryDirectory()   # the compiler's assembly, for check_load_addresses
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-Rpass-analysis=kernel-resource-usage", "--save-temps", *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, obj, subprocess.Popen(cmd, cwd=temps.name, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                                 text=True)))
    objs = []
    for src, obj, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if not os.environ.get("BURST_ALLOW_SPILLS"):   # experiments only: the committed build must not spill
            check_resources(out, src)
        with open(os.path.join(temps.name, src.replace(".hip", "-hip-amdgcn-amd-amdhsa-gfx950.s"))) as f:
            check_load_addresses(f.read(), src)
        if verbose and out.strip():
            print(out)
        objs.append(obj)
    temps.cleanup()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", out_path or LIB_PATH]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}")
    return out_path or LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
