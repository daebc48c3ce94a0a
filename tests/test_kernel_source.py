"""What the kernels' source has to keep to for the compiled code to be right."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_24010_amd", "csrc")


def _functions(text):
    """(declaration, body) of every function that starts at the first column."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"^(?:template <[^\n]*>\n)?[^\n#}]*\b__(?:device|global)__[^;{]*\{\n(.*?)^\}", text, re.S | re.M):
        yield text[m.start():m.start(1)], m.group(1)


def test_readers_of_the_kernel_arguments_are_inlined_into_a_kernel():
    """__builtin_amdgcn_kernarg_segment_ptr() is null in a function that is not: its callers
    (touch_args and push_args, and those that call them) are kernels or forced inline."""
    fns = list(_functions(open(os.path.join(CSRC, "gs_kernels.hip")).read()))
    reads, seen = {"__builtin_amdgcn_kernarg_segment_ptr"}, set()
    while reads - seen:
        name = (reads - seen).pop()
        seen.add(name)
        callers = [decl for decl, body in fns if re.search(r"\b%s\b" % name, body)]
        assert callers, name
        for decl in callers:
            if "__global__" in decl:
                continue
            assert "__forceinline__" in decl, decl
            reads.add(re.search(r"(\w+)\(", decl.split("__forceinline__")[1]).group(1))
    assert {"push_args", "flush_seg", "close_seg", "push_piece", "push_tail_emit"} <= reads


def test_injection_remembers_nothing_between_calls():
    """A launch attribute set once per process is missing on a second device, and a smaller
    one set later by another thread takes a larger one's place."""
    src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "gs_kernels.hip")).read())
    body = re.search(r"static hipError_t inject_t\(.*?^\}", src, re.S | re.M).group(0)
    assert "hipFuncSetAttribute" in body and "static" not in body.split("\n", 1)[1]


def test_the_pushs_chunk_loop(tmp_path):
    """The compiled loop over full chunks (binary32, one vector a thread): nothing is waited
    for between the loop's top and the next chunk's loads; and in round-robin order, whose
    passes end with a wait, the absorbed ions' stores go out before the particles' own."""
    from paper_2603_24010_amd import build as B
    out = str(tmp_path / "push.s")
    flags = [f for f in B.FLAGS if f != "-Wall"]
    cmd = [B.HIPCC, *flags, "-w", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-DGS_PUSH_PART=4",
           "--cuda-device-only", "-S", os.path.join(B.CSRC, "gs_kernels.hip"), "-o", out]
    subprocess.run(cmd, check=True)
    text = open(out).read()
    seen = 0
    for m in re.finditer(r"^_ZN2gs6k_push\w*Li4ELb1ELb([01])E\w*:(.*?)^\.Lfunc_end", text, re.S | re.M):
        lines = m.group(2).splitlines()
        store = next(i for i, ln in enumerate(lines) if "global_store_dwordx4" in ln and ln.rstrip().endswith(" nt"))
        loads = [i for i in range(store) if "global_load_dwordx4" in lines[i] and lines[i].rstrip().endswith(" nt")][-2:]
        top = max(i for i in range(loads[0]) if re.match(r"\.LBB.*Parent Loop BB\d+_\d+ Depth=1", lines[i]))
        assert loads[1] - top < 60, "the chunk loop's top"
        assert not any("vmcnt" in ln for ln in lines[top:loads[0]])
        queued = any("v_cvt_f64_f32" in ln for ln in lines[top:store])  # the absorbed ions' velocities
        assert queued == (m.group(1) == "1")
        seen += 1
    assert seen == 8  # workgroups of 256, 512, 768 and 1024, contiguous and round robin
