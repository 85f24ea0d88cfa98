"""Compile the HIP sources under csrc/ for gfx950 into paper_2402_17764_amd/libbitnet_hip.so.

hipcc cross-compiles without a GPU.  Objects go to paper_2402_17764_amd/_build/ (not committed);
the shared library sits next to this file so that it travels with the tree.
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbitnet_hip.so")

SOURCES = ["api.hip", "quant_weights.hip", "quant_acts.hip", "linear_ref.hip", "linear_gemv.hip", "linear_decode.hip", "linear_skinny.hip", "linear_ksplit.hip", "linear_gemm.hip", "trit5.hip", "static_scratch.hip"]
SOURCES += ["decode%s_%s.hip" % (k, t) for k in ("", "_norm", "_pair", "_norm_pair") for t in ("bf16", "f32")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                       # every rounding step of the quantizers is explicit
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the leading kernel arguments arrive in scalar registers with the wave: no load, cold in a chain of launches that stream
    # weights through the L2, stands before a kernel's first address (3B decode stack 639 -> 623 us with nothing else changed)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wextra", "-Wno-unused-parameter", "-Wno-unknown-attributes",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Kernels that count the vector-memory loads in flight (explicit s_waitcnt vmcnt(n)): a register spill would
# add scratch loads to that count, so the build fails if the compiler gives any of them scratch memory.
NO_SCRATCH = {"linear_skinny.hip": ("linear_skinny_2bit", "linear_skinny_ws_2bit"), "linear_ksplit.hip": ("linear_ksplit_2bit",)}


def _check_no_scratch(src, stderr):
    """stderr holds -Rpass-analysis=kernel-resource-usage remarks: 'Function Name: <mangled>' ... 'ScratchSize ...: n'."""
    name, bad = None, []
    for line in stderr.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
        elif "ScratchSize" in line and name and any(k in name for k in NO_SCRATCH[src]):
            if int(line.split("]:")[1].split()[0]) != 0:
                bad.append(name)
    if bad:
        raise RuntimeError("%s: kernels that count loads in flight must not spill: %s" % (src, ", ".join(bad)))


def skinny_instantiations(source_text, macro="SKINNY"):
    """The linear_skinny_2bit<kMT, kR, kW, kS, kD, kLx> instantiations that the launcher dispatches: every
    `SKINNY(a, b, c, d, e, f)` use in the source (SKINNY_WS: those of the form with a loader wave)."""
    return sorted({tuple(int(v) for v in m.groups())
                   for m in re.finditer(r"\b%s\((\d+), (\d+), (\d+), (\d+), (\d+), (\d+)\)" % macro, source_text)})


def check_issue_order(asm_text, expected):
    """linear_skinny_2bit waits for a step's LDS copies with a count of the younger loads (s_waitcnt vmcnt(n)), which
    holds only if each step's copies are issued before the weight loads that follow them in the source.  Scheduling
    fences in the kernel pin that; this reads the device assembly the object is assembled from and raises if a
    compiler ever ignores them: between barriers a wave must issue kC = 4 kMT / kW copies ("buffer_load ... lds") and
    then kR weight loads, and the prologue kD such groups; the last kD steps, behind the loop, request nothing but the
    copies of the kD - kLx steps that are still missing.  Every instantiation in `expected` must be present and pass;
    an instantiation in the assembly that is not expected is an error too (it would ship unchecked by the dispatch
    tests).  Returns the instantiations checked."""
    cur, segs, checked = None, [""], []
    for line in asm_text.splitlines():
        m = re.match(r"^_ZN6bitnet18linear_skinny_2bitILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E\S*:", line)
        if m:
            cur, segs = tuple(int(v) for v in m.groups()), [""]
            continue
        if cur is None:
            continue
        if "buffer_load_dwordx4" in line:
            segs[-1] += "L" if re.search(r"\blds\b", line) else "W"
        elif "s_barrier" in line:
            segs.append("")
        elif "s_endpgm" in line:
            kMT, kR, kW, kS, kD, kLx = cur
            unit = "L" * (4 * kMT // kW) + "W" * kR
            loops = [g for g in segs[1:] if g]
            last = ["L" * (4 * kMT // kW)] * (kD - kLx)
            if last and loops[-len(last):] == last:
                loops = loops[:-len(last)]
            if segs[0] != unit * kD or not loops or any(g != unit for g in loops):
                raise RuntimeError("linear_skinny_2bit<%s>: loads are not issued in source order (%s), the counted "
                                   "waits would be wrong" % (", ".join(map(str, cur)), " | ".join(segs)))
            checked.append(cur)
            cur = None
    if cur is not None:
        raise RuntimeError("linear_skinny_2bit<%s>: the kernel's end was not found in the assembly" % ", ".join(map(str, cur)))
    missing = sorted(set(expected) - set(checked))
    extra = sorted(set(checked) - set(expected))
    if missing or extra or len(checked) != len(set(checked)):
        raise RuntimeError("linear_skinny_2bit: issue order unchecked for %s; not dispatched but built: %s" % (missing, extra))
    return checked


def lds_reads_at_barriers(asm_text):
    """For every batched-decode kernel in the assembly the most LDS reads that can be outstanding at one of its barriers, over all
    paths: {(has a loader wave, parameters): reads}.  A ds_read adds one, s_waitcnt lgkmcnt(n) leaves n at most."""
    found = {}
    for m in re.finditer(r"^_ZN6bitnet\d+linear_skinny(_ws)?_2bitI((?:Li\d+E)+)E\S*:[^\n]*\n(.*?)^\.Lfunc_end", asm_text, re.M | re.S):
        code = []                              # (kind, operand)
        for line in m.group(3).splitlines():
            line = line.split(";")[0].strip()
            label, op = re.match(r"(\.LBB\w+):", line), line.split(" ")[0].split("\t")[0]
            wait = re.search(r"lgkmcnt\((\d+)\)", line)
            if label:
                code.append(("label", label.group(1)))
            elif op.startswith("ds_read"):
                code.append(("read", None))
            elif op == "s_waitcnt" and wait:
                code.append(("wait", int(wait.group(1))))
            elif op == "s_barrier":
                code.append(("barrier", None))
            elif op in ("s_branch", "s_endpgm") or op.startswith("s_cbranch"):
                code.append((op[2:], line.split()[-1]))
        at = {operand: i for i, (kind, operand) in enumerate(code) if kind == "label"}
        entry, work, most = {0: 0}, [0], 0
        while work:                            # states grow up to the counter's limit: this ends
            i = work.pop()
            n = entry[i]
            while i < len(code):
                kind, operand = code[i]
                n = min(n + 1, 15) if kind == "read" else min(n, operand) if kind == "wait" else n
                most = max(most, n) if kind == "barrier" else most
                if "branch" in kind and entry.get(at[operand], -1) < n:
                    entry[at[operand]] = n
                    work.append(at[operand])
                if kind in ("branch", "endpgm"):
                    break
                i += 1
                if i < len(code) and code[i][0] == "label":
                    if entry.get(i, -1) >= n:
                        break
                    entry[i] = n
        found[(bool(m.group(1)), tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(2))))] = most
    return found


def check_lds_reads(asm_text, plain, loader):
    """A barrier of the batched-decode kernels gives the LDS stage that was read in front of it to the next copy: no read of it may
    be outstanding there, in any dispatched instantiation."""
    found = lds_reads_at_barriers(asm_text)
    missing = {(False, p) for p in plain} | {(True, p) for p in loader}
    if set(found) != missing:
        raise RuntimeError("batched decode: LDS reads checked for %s, dispatched %s" % (sorted(found), sorted(missing)))
    bad = sorted(k for k, n in found.items() if n)
    if bad:
        raise RuntimeError("batched decode: LDS reads outstanding at a barrier that frees their stage: %s" % bad)
    return found


def ksplit_instantiations(source_text):
    """The linear_ksplit_2bit<kMT, kR, kW, kS, kQ> instantiations that the launcher dispatches: KSPLIT(kMT, kR, kW, kS, kLx) uses, kQ
    slots of 16 tokens a wave."""
    found = {tuple(int(v) for v in m.groups()) for m in re.finditer(r"\bKSPLIT\((\d+), (\d+), (\d+), (\d+), (\d+)\)", source_text)}
    return sorted((mt, r, w, s, (lx + 1) * mt // w) for mt, r, w, s, lx in found)


def check_ksplit_order(asm_text, expected):
    """linear_ksplit_2bit waits for a tile's LDS copies with a count of the younger loads, of which there are at least that many only if the
    loads are issued as in the source: the weights of the first step (W, kR kW of them) and the copies (L, four a tile) of the
    first kQ tiles; in the loop a step's weights, then for each of its kMT tiles a wait that leaves the copies of kQ - 1 tiles and one step's
    weights in flight, the tile's four reads (R), and the copies that take its slot, no read outstanding; behind the loop the steps that the slots
    still reach, each wait with the copies of the tiles behind it alone.  Raises unless the assembly of every instantiation reads so up to
    its first barrier, with no read of LDS elsewhere."""
    checked = []
    for m in re.finditer(r"^_ZN6bitnet\d+linear_ksplit_2bitI((?:Li\d+E)+)E\S*:[^\n]*\n(.*?)^\.Lfunc_end", asm_text, re.M | re.S):
        p = tuple(int(v) for v in re.findall(r"Li(\d+)E", m.group(1)))
        kMT, kR, kW, _, kQ = p
        rows, got, limit, reading = kR * kW, "", None, False
        for line in m.group(2).splitlines():
            line = line.split(";")[0]
            wait = re.search(r"vmcnt\((\d+)\)", line)
            if "s_barrier" in line:
                break
            if re.search(r"lgkmcnt\(0\)", line):
                reading = False
            if wait:                           # the strictest of the waits in front of a tile's first read
                limit = int(wait.group(1)) if limit is None else min(limit, int(wait.group(1)))
            elif "buffer_load_dwordx4" in line:
                copy = re.search(r"\blds\b", line)
                got += ("!" if copy and reading else "") + ("L" if copy else "W")
                limit = None
            elif re.search(r"\bds_read", line):
                got += ("" if limit is None else "<%d>" % limit) + "R"
                limit, reading = None, True
            if "v_mfma" in line:
                limit = None
        ahead = -(-kQ // kMT)
        want = "W" * rows + "LLLL" * kQ + "W" * rows + ("<%d>RRRRLLLL" % (4 * (kQ - 1) + rows)) * kMT
        for e in range(ahead - 1, -1, -1):
            want += "W" * rows if e else ""
            for t in range(kMT):
                left = e * kMT + kMT - 1 - t
                want += "<%d>RRRR" % (4 * min(left, kQ - 1)) + ("LLLL" if left >= kQ else "")
        if got != want:
            raise RuntimeError("linear_ksplit_2bit<%s>: loads, waits and reads (!: a copy over a slot that is being read) are %s, not %s"
                               % (", ".join(map(str, p)), got, want))
        checked.append(p)
    if sorted(checked) != sorted(expected):
        raise RuntimeError("linear_ksplit_2bit: checked %s, dispatched %s" % (sorted(checked), sorted(expected)))
    return checked


def _check_issue_order(src):
    """Runs the checks on the assembly that -save-temps left next to the object: the very text the device code of the
    shipped object was assembled from."""
    asm = open(os.path.join(BUILD, os.path.splitext(src)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")).read()
    source = open(os.path.join(CSRC, src)).read()
    if src == "linear_ksplit.hip":
        check_ksplit_order(asm, ksplit_instantiations(source))
        return
    expected = skinny_instantiations(source)
    if not expected:
        raise RuntimeError("%s: no SKINNY(...) dispatch found: the issue-order check has nothing to go by" % src)
    check_issue_order(asm, expected)
    check_lds_reads(asm, expected, skinny_instantiations(source, "SKINNY_WS"))


# Host code with the undefined-behaviour sanitizer compiled in as traps (no runtime library to load): signed overflow,
# bad shifts, out-of-range enum and integer conversions, misaligned and null accesses in the validation and dispatch
# code end the process.  The device code is built as usual; only host-side calls are meant to run against this build.
SANITIZE_HOST = ["-Xarch_host", "-fsanitize=undefined,integer", "-Xarch_host", "-fsanitize-trap=all", "-Xarch_host",
                 "-fno-sanitize=unsigned-integer-overflow,unsigned-shift-base,implicit-conversion"]


def _compile_sanitized(src, out_dir):
    obj = os.path.join(out_dir, os.path.splitext(src)[0] + ".o")
    flags = [f for f in FLAGS if f != "-O3"] + ["-O1", *SANITIZE_HOST]
    r = subprocess.run([HIPCC, *flags, "-c", os.path.join(CSRC, src), "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc (host-sanitized) failed on %s:\n%s" % (src, r.stderr))
    return obj


def build_library_sanitized() -> str:
    """libbitnet_hip_ubsan.so under _build/ubsan: for the CPU test that runs the host-side tests against it."""
    out_dir = os.path.join(BUILD, "ubsan")
    os.makedirs(out_dir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile_sanitized(s, out_dir), SOURCES))
    lib = os.path.join(out_dir, "libbitnet_hip_ubsan.so")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", lib])
    return lib


def _compile(src):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if src in NO_SCRATCH:
        cmd += ["-Rpass-analysis=kernel-resource-usage", "-save-temps=obj"]      # the device assembly stays next to the object
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    lines = [l for l in r.stderr.splitlines() if noise not in l]
    if src in NO_SCRATCH:                      # drop the resource remarks and the source excerpts printed under them
        lines = [l for l in lines if "remark:" not in l and not re.match(r"^\s*\d*\s*\|", l)]
    err = "\n".join(lines)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    if src in NO_SCRATCH:
        _check_no_scratch(src, r.stderr)
        _check_issue_order(src)
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_library(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


def build_floors(verbose: bool = False) -> str:
    """libbitnet_floors.so: the read-only and the MFMA-only kernel that bench.py and read_floor.py time next to the product
    (no part of the BitLinear library)."""
    lib = os.path.join(HERE, "libbitnet_floors.so")
    tmp = lib + ".tmp.%d" % os.getpid()
    r = subprocess.run([HIPCC, *FLAGS, "-shared", os.path.join(CSRC, "floors.hip"), os.path.join(CSRC, "prefill_ladder.hip"), "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on floors.hip / prefill_ladder.hip:\n" + r.stderr)
    os.replace(tmp, lib)
    if verbose:
        print("built", lib)
    return lib


def build_call(verbose: bool = False) -> str:
    """_call.so: the native argument marshalling of binding.py (host code only, against torch's headers and libraries)."""
    import sysconfig
    from torch.utils import cpp_extension as ext
    lib = os.path.join(HERE, "_call.so")
    tmp = lib + ".tmp.%d" % os.getpid()
    libdir = ext.library_paths()[0]
    cmd = [HIPCC, "-O2", "-std=c++17", "-fPIC", "-shared", "-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-Wno-deprecated-declarations"]
    cmd += [f for p in ext.include_paths("cuda") + [sysconfig.get_paths()["include"]] for f in ("-isystem", p)]
    cmd += ["-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "call.cpp"), "-o", tmp, "-L", libdir, "-Wl,-rpath," + libdir,
            "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on call.cpp:\n" + r.stderr)
    os.replace(tmp, lib)
    if verbose:
        print("built", lib)
    return lib


if __name__ == "__main__":
    build_library(verbose=True)
    build_call(verbose=True)
    build_floors(verbose=True)
