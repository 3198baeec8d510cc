"""Words that a kernel reads through the scalar cache as constants (const_ld) are not written by the same
launch: the compiler may repeat such a load after a store to the word.  Read from the source: each kernel
with the device functions it reaches."""
import os
import re

from paper_2501_07465_amd import build as B


def _functions(text):
    """name -> bodies of the functions defined at the left margin"""
    out = {}
    for m in re.finditer(r"^\{\n(.*?)^\}", text, re.S | re.M):
        head = text[:m.start()].rsplit("\n\n", 1)[-1]
        names = re.findall(r"\b(\w+)\(", re.sub(r"__attribute__\(\(.*?\)\)\)|__launch_bounds__\(.*?\)", "", head))
        if names:
            out.setdefault(names[0], []).append((head, m.group(1)))
    return out


def test_no_kernel_writes_what_it_reads_as_constant():
    text = open(os.path.join(B.CSRC, "pic_kernels.inc")).read()
    text = re.sub(r"//[^\n]*", "", text)
    fn = _functions(text)
    kernels = [n for n, bodies in fn.items() if any("__global__" in h for h, _ in bodies)]
    assert {"k_particles", "k_fields", "k_tensor_u", "k_tensor_fold"} <= set(kernels)
    read = set()
    for k in kernels:
        seen, todo = set(), [k]
        while todo:
            f = todo.pop()
            if f in seen:
                continue
            seen.add(f)
            code = " ".join(b for _, b in fn[f])
            todo += [g for g in fn if g not in seen and re.search(r"\b%s\b" % g, code)]
        code = "\n".join(b for f in seen for _, b in fn[f])
        consts = set(re.findall(r"const_ld\(\s*&?\s*(?:S|sims\[\w+\])\.(\w+)", code))
        written = set(re.findall(r"(?:S|sims\[\w+\])\.(\w+)\s*\[[^;=]*\]\s*[-+|]?=(?!=)", code))
        written |= set(re.findall(r"\*\s*(?:glb<\w+>\()?(?:S|sims\[\w+\])\.(\w+)\)?\s*=(?!=)", code))
        written |= set(re.findall(r"atomic\w+\([^;]*?(?:S|sims\[\w+\])\.(\w+)", code))
        print(k, "reads as constant", sorted(consts), "writes", sorted(written))
        assert not consts & written, (k, consts & written)
        read |= consts
        if k == "k_fields":
            assert {"fmask", "step_p"} <= consts and {"fdirty", "step_f", "series"} <= written
        if k == "k_particles":
            assert {"step_f", "n_units"} <= consts and {"step_p", "partials", "over_count"} <= written
    assert read
