"""Where device code may ask for the kernel's argument segment."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2505_17368_amd", "csrc")


def _functions():
    """(qualifiers, name, body) of every device function; bodies run to the
    closing brace in the first column."""
    out = []
    for f in sorted(os.listdir(CSRC)):
        src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())
        for m in re.finditer(r"^[^\n#}]*__(?:device|global)__[^;{]*\{.*?^\}", src, re.M | re.S):
            head, body = m[0].split("{", 1)
            quals = re.sub(r"__attribute__\(\(.*?\)\)\)?|__launch_bounds__\([^)]*\)", "", head)
            name = re.search(r"(\w+)\s*\(", quals)
            if name:
                out.append((quals, name[1], body))
    return out


def test_argument_segment_is_read_in_kernels_only():
    """The compiler gives a kernel's argument segment to kernels alone: in a
    called function __builtin_amdgcn_kernarg_segment_ptr is null.  So it is
    used in a kernel, or in functions forced inline all the way into one."""
    funcs = _functions()
    assert {"k_search", "search_one", "search_kernel_body"} <= {f[1] for f in funcs}
    todo, seen = ["__builtin_amdgcn_kernarg_segment_ptr"], set()
    while todo:
        callee = todo.pop()
        users = [f for f in funcs if re.search(r"\b%s\b" % callee, f[2]) and f[1] != callee]
        assert users, callee
        for quals, name, _ in users:
            if "__global__" in quals or name in seen:
                continue
            assert "__forceinline__" in quals, f"{name} uses {callee} and may be a called function"
            seen.add(name)
            todo.append(name)
