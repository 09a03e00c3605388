"""What the compiler does not see in inline assembly, checked on the kernel sources."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_23406_amd", "csrc")

# scalar instructions that leave SCC as it is; every other s_* ALU instruction writes it
KEEPS_SCC = re.compile(r"s_(mov|cmov|mul_i32|mul_hi|nop|waitcnt|barrier|sleep|setprio|brev|ff0|ff1|flbit|sext|"
                       r"bitset|bfm|pack|movk|cselect|cbranch|branch|load|buffer|dcache|endpgm|sethalt)")


def asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read()).replace("\\\n", "\n")
        for m in re.finditer(r"\basm\s*(volatile)?\s*\(", text):
            depth, i, quoted = 1, m.end(), False
            while depth:
                c = text[i]
                quoted ^= c == '"' and text[i - 1] != "\\"
                depth += 0 if quoted else (c == "(") - (c == ")")
                i += 1
            yield os.path.basename(path), text[m.end():i - 1]


def test_scalar_condition_code_is_declared():
    """An asm statement with an instruction that writes SCC names it as clobbered: otherwise the
    compiler may carry a scalar compare across the statement."""
    seen = 0
    for path, body in asm_statements():
        words = [w for lit in re.findall(r'"((?:[^"\\]|\\.)*)"', body) for w in re.findall(r"\bs_\w+", lit)]
        writes = [w for w in words if not KEEPS_SCC.match(w)]
        if writes:
            seen += 1
            assert re.search(r'"scc"', body), (path, writes)
    assert seen > 0


def test_gemm_assembly_reads_no_vector_registers():
    """The GEMM's values come straight from the matrix cores: its inline assembly is waits and
    barriers only."""
    bodies = [body for path, body in asm_statements() if path == "hq_gemm.hip"]
    assert bodies
    for body in bodies:
        assert not re.search(r'"[=+&]*[va]"\s*\(', body), body
