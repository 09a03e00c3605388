"""What the compiler does not see in inline assembly, checked on the kernel sources."""
import glob
import os
import re
import subprocess

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
            yield os.path.basename(path), text[m.end():i - 1].replace("\\n", " ").replace("\\t", " ")


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


PROBE = r"""
#include "hq_device.h"
__global__ __launch_bounds__(256, 2) void by_asm(const uint32_t* c, float* o) {
  const MfmaRht m(threadIdx.x & 63);
  const uint32_t p[4] = {c[4 * threadIdx.x], c[4 * threadIdx.x + 1], c[4 * threadIdx.x + 2], c[4 * threadIdx.x + 3]};
  float y[8];
  m.small(p, y);
  for (int j = 0; j < 8; ++j) o[8 * threadIdx.x + j] = y[j];
}
__global__ __launch_bounds__(256, 2) void by_compiler(const v8h_t* c, float* o) {
  const v4f_t r = __builtin_amdgcn_mfma_f32_16x16x32_f16(c[threadIdx.x], c[threadIdx.x + 64], (v4f_t){}, 0, 0, 0);
  o[threadIdx.x] = r[0] * 3.0f;
}
"""


def wait_states(body):
    """Wait states between each matrix instruction and the first instruction, inline or not, that has
    one of its result registers among its operands."""
    pending, now, out = [], 0, []
    for line in body.split("\n"):
        t = line.split(";")[0].strip()
        if not t or t.endswith(":") or t.startswith("."):
            continue
        if t.startswith("s_nop"):
            now += int(t.split()[1]) + 1
            continue
        regs = set()
        for b, lo, hi, b1, r1 in re.findall(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", t):
            regs |= {(b1, int(r1))} if b1 else {(b, i) for i in range(int(lo), int(hi) + 1)}
        for at, res in [p for p in pending if p[1] & regs]:
            out.append(now - at)
            pending.remove((at, res))
        now += 1
        if t.startswith("v_mfma"):
            b, lo, hi = re.match(r"\S+\s+([va])\[(\d+):(\d+)\]", t).groups()
            pending.append((now, {(b, i) for i in range(int(lo), int(hi) + 1)}))
    assert not pending
    return out


def test_matrix_results_wait_before_inline_assembly(tmp_path):
    """The transform's inline assembly reads matrix-core results no sooner than the compiler lets its
    own instructions read them, also where they are not copied between register files first."""
    from paper_2606_23406_amd import build
    src, s = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run([build.HIPCC] + flags + ["-w", "-I", CSRC, "-S", "--offload-device-only", "-o", str(s), str(src)],
                   check=True, timeout=120)
    text = s.read_text()
    body = {k: re.search(r"\n_Z\d+%s\w*:(.*?)s_endpgm" % k, text, re.S).group(1) for k in ("by_asm", "by_compiler")}
    (need,) = wait_states(body["by_compiler"])
    got = wait_states(body["by_asm"])
    assert need >= 4 and len(got) == 2
    assert min(got) >= need, (got, need)


def test_gemm_keeps_products_in_plain_registers(tmp_path):
    """No GEMM kernel copies its products between register files or spills them."""
    from paper_2606_23406_amd import build
    s = tmp_path / "gemm.s"
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run([build.HIPCC] + flags + ["-w", "-S", "--offload-device-only", "-o", str(s),
                                            os.path.join(CSRC, "hq_gemm.hip")], check=True, timeout=300)
    text = s.read_text()
    assert text.count("v_mfma") > 100
    assert "v_accvgpr" not in text and not re.search(r"scratch_(load|store)", text)


def test_gemm_assembly_reads_no_vector_registers():
    """The GEMM's values come straight from the matrix cores: its inline assembly is waits and
    barriers only."""
    bodies = [body for path, body in asm_statements() if path == "hq_gemm.hip"]
    assert bodies
    for body in bodies:
        assert not re.search(r'"[=+&]*[va]"\s*\(', body), body


def test_scalar_operands_wait():
    """A vector instruction in inline assembly with a scalar register operand has the two wait states
    in front that it needs behind a vector instruction that wrote the register; those with a carry are
    looked at below, as compiled."""
    seen = 0
    for path, body in asm_statements():
        ops = re.findall(r"\b(v_\w+)", body)
        if not ops or not re.search(r'"s"\s*\(', body) or all(o.startswith(("v_addc", "v_subb")) for o in ops):
            continue
        seen += 1
        assert re.match(r'\s*"s_nop [1-9]', body), (path, body)
    assert seen > 0


CARRY_PROBE = r"""
#include "hq_device.h"
__global__ __launch_bounds__(256) void probe(const float* w, int32_t* o) {
  float v[8];
  int32_t h[8], cb;
  for (int j = 0; j < 8; ++j) v[j] = w[8 * threadIdx.x + j];
  e8_nearest(v, h, cb);
  for (int j = 0; j < 8; ++j) o[9 * threadIdx.x + j] = h[j];
  o[9 * threadIdx.x + 8] = cb;
}
"""


def test_carry_masks_come_from_scalar_logic(tmp_path):
    """The lane masks that the E8 decision's inline assembly takes as carries are last written by scalar
    instructions, or two wait states before."""
    from paper_2606_23406_amd import build
    src, s = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(CARRY_PROBE)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run([build.HIPCC] + flags + ["-w", "-I", CSRC, "-S", "--offload-device-only", "-o", str(s), str(src)],
                   check=True, timeout=120)
    body = re.search(r"\n_Z\d+probe\w*:(.*?)s_endpgm", s.read_text(), re.S).group(1)

    def pairs(t):
        return {i for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", t) for i in (int(lo), int(hi))} | (
            {"vcc"} if re.search(r"\bvcc\b", t) else set())
    lines = [t for t in (line.split(";")[0].strip() for line in body.split("\n")) if t and t[0] != "."]
    seen = 0
    for n, t in enumerate(lines):
        if not re.match(r"v_(addc|subb)_co_u32", t):
            continue
        mask, states = pairs(t.split(",")[-1]), 0
        assert mask
        seen += 1
        for u in reversed(lines[:n]):
            if u.startswith("s_nop"):
                states += int(u.split()[1]) + 1
                continue
            written = pairs(u.split(",")[1] if re.match(r"v_\w+_co_", u) else u.split(",")[0])
            if written & mask:
                assert u.startswith("s_") or states >= 2, (u, t)
                break
            states += 1
    assert seen >= 16
