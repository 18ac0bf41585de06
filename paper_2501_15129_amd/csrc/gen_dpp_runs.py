"""Writes dpp_runs.inc: the inline-assembly runs of DPP row-broadcast multiply-adds used by the
register-resident binary32 rollout kernels (run `python gen_dpp_runs.py` in this folder after a change).

Inline assembly needs its instruction text and operand numbers as literals, so the runs for every
(accumulators, inputs per row) pair the kernels use are spelled out here instead of by hand."""
from pathlib import Path

DOT = [(q, n) for q in (1, 2, 4) for n in (3, 4, 5, 8, 12, 16)]     # (accumulators, inputs per row)
CHAIN = (3, 4, 5, 8, 12, 16)                                    # one accumulator, no partial sums
ROTATE = (4, 8, 16)                                             # rotations of a row
MAC = (3, 4, 6, 8, 16)                                          # accumulate-into runs (the action term)
TAIL = ' row_mask:0xf bank_mask:0xf bound_ctrl:1\\n\\t"'
# ends a run whose accumulators a row swap may read at once: the compiler keeps one of the two wait states behind inline assembly
SWAP = '\n      "s_nop 0\\n\\t"'


def ins(op, acc, h, w, j):
    return f'"{op} %{acc}, %{h}, %{w} row_newbcast:{j}{TAIL}'


def operands(n, per=10):
    items = [f'"v"(w[{k}])' for k in range(n)]
    return ",\n".join("          " + ", ".join(items[a:a + per]) for a in range(0, n, per))


def dot_block(q, n, swapped=False):
    """q accumulators x n inputs: o[a] = sum_j w[n a + j] * bcast_j(h); with one accumulator the sum is split into
    up to four interleaved partial sums."""
    lines = []
    if q == 1:
        parts = min(4, n)
        for j in range(n):
            a = j % parts
            lines.append(ins("v_mul_f32_dpp" if j < parts else "v_fmac_f32_dpp", a, parts, parts + 1 + j, j))
        outs = ", ".join(f'"=&v"(p{a})' for a in range(parts))
        body = "      " + "\n      ".join(lines)
        total = " + ".join(f"p{a}" for a in range(parts)) if parts < 4 else "(p0 + p1) + (p2 + p3)"
        return (f"    float {', '.join(f'p{a}' for a in range(parts))};\n"
                f'    asm volatile("s_nop 1\\n\\t"\n{body}\n        : {outs}\n        : "v"(h),\n{operands(n)});\n'
                f"    o[0] = {total};\n")
    for j in range(n):
        lines.append(" ".join(ins("v_mul_f32_dpp" if j == 0 else "v_fmac_f32_dpp", a, q, q + 1 + n * a + j, j) for a in range(q)))
    outs = ", ".join(f'"=&v"(o[{a}])' for a in range(q))
    body = "      " + "\n      ".join(lines) + (SWAP if swapped else "")
    return f'    asm volatile("s_nop 1\\n\\t"\n{body}\n        : {outs}\n        : "v"(h),\n{operands(q * n)});\n'


def dot_add_block(q, n):
    """as dot_block, added to o"""
    lines = [" ".join(ins("v_fmac_f32_dpp", a, q, q + 1 + n * a + j, j) for a in range(q)) for j in range(n)]
    outs = ", ".join(f'"+v"(o[{a}])' for a in range(q))
    body = "      " + "\n      ".join(lines) + SWAP
    return f'    asm volatile("s_nop 1\\n\\t"\n{body}\n        : {outs}\n        : "v"(h),\n{operands(q * n)});\n'


def mac_block(n):
    lines = [ins("v_fmac_f32_dpp", 0, 1, 2 + j, j) for j in range(n)]
    body = "      " + "\n      ".join(lines)
    return f'    asm volatile("s_nop 1\\n\\t"\n{body}\n        : "+v"(acc)\n        : "v"(h),\n{operands(n)});\n'


def chain_block(n):
    """one accumulator: a dependent multiply-add issues as fast as an independent one, so partial sums would only cost their additions"""
    lines = [ins("v_mul_f32_dpp" if j == 0 else "v_fmac_f32_dpp", 0, 1, 2 + j, j) for j in range(n)]
    body = "      " + "\n      ".join(lines)
    return f'    asm volatile("s_nop 1\\n\\t"\n{body}\n        : "=&v"(p)\n        : "v"(h),\n{operands(n)});\n'


def rotate_block(n):
    """the first rotation is none: a plain multiply, which is also one of the two wait states"""
    lines = ['"v_mul_f32_e32 %0, %1, %2\\n\\t"'] + [f'"v_fmac_f32_dpp %0, %1, %{2 + j} row_ror:{j}{TAIL}' for j in range(1, n)]
    body = "      " + "\n      ".join(lines)
    return f'    asm volatile("s_nop 0\\n\\t"\n{body}\n        : "=&v"(p)\n        : "v"(h),\n{operands(n)});\n'


def main():
    out = ["// Generated by gen_dpp_runs.py - do not edit.",
           "//",
           '// "v_fmac_f32_dpp acc, h, w row_newbcast:j" adds w * (lane j of h\'s 16-lane row) to acc: the input element is',
           "// broadcast within each row by the DPP modifier, fused into the multiply-add - one instruction per multiply-add,",
           "// no scalar hop.  The compiler folds a DPP move into v_mul / v_add but not into v_fmac, hence inline assembly.",
           "// Its hazard checks do not look inside inline assembly: a vector ALU write of `h` must be two wait states away",
           "// from the first DPP read, hence the s_nop that leads every run.  The same distance lies before a row swap (v_permlane16_swap,",
           "// v_permlane32_swap): behind inline assembly the compiler leaves one wait state, so a run of two accumulators, which are swapped with one",
           "// another as they are, ends with the other.  Of four accumulators the pair that is swapped first ends one instruction earlier; a single one is",
           "// copied before it is swapped with itself, and the copy's distance is the compiler's.  tests/test_wait_states.py reads the distances out",
           "// of the built code.  A run starts with multiplies (no zeroed",
           "// accumulators) and interleaves its accumulators, so that consecutive instructions never depend on each other.",
           "",
           "// o[a] = sum_{j < N} w[N a + j] * (lane j of h's row), a < Q.  SWAPPED: the two accumulators may be swapped with one another next",
           "template <int Q, int N, bool SWAPPED = Q == 2>",
           "__device__ __forceinline__ void row_bcast_dot(float (&o)[Q], float h, const float (&w)[Q * N]) {"]
    first = True
    for q, n in DOT:
        out.append(f"  {'if' if first else 'else if'} constexpr (Q == {q} && N == {n}) {{")
        if q == 2:
            out += ["    if constexpr (SWAPPED) {", dot_block(q, n, True).rstrip("\n"), "    } else {", dot_block(q, n).rstrip("\n"), "    }"]
        else:
            out.append(dot_block(q, n).rstrip("\n"))
        out.append("  }")
        first = False
    out.append('  else static_assert(Q < 0, "no run of this shape: add it to gen_dpp_runs.py");')
    out.append("}")
    out.append("")
    out.append("// o[a] += sum_{j < 16} w[16 a + j] * (lane j of h's row), a < 2")
    out.append("__device__ __forceinline__ void row_bcast_dot_add(float (&o)[2], float h, const float (&w)[32]) {")
    out.append(dot_add_block(2, 16).rstrip("\n"))
    out.append("}")
    out.append("")
    out.append("// acc + sum_{j < N} w[j] * (lane j of h's row)")
    out.append("template <int N>")
    out.append("__device__ __forceinline__ float row_bcast_mac(float acc, float h, const float (&w)[N]) {")
    first = True
    for n in MAC:
        out.append(f"  {'if' if first else 'else if'} constexpr (N == {n}) {{")
        out.append(mac_block(n).rstrip("\n"))
        out.append("  }")
        first = False
    out.append('  else static_assert(N < 0, "no run of this length: add it to gen_dpp_runs.py");')
    out.append("  return acc;")
    out.append("}")
    for name, doc, sizes, block in (
            ("row_bcast_chain", "// sum_{j < N} w[j] * (lane j of h's row), in one accumulator", CHAIN, chain_block),
            ("row_rotate_chain", "// sum_{j < N} w[j] * (lane (c - j) mod 16 of h's row) in column c, in one accumulator", ROTATE, rotate_block)):
        out += ["", doc, "template <int N>", f"__device__ __forceinline__ float {name}(float h, const float (&w)[N]) {{", "  float p;"]
        for k, n in enumerate(sizes):
            out.append(f"  {'if' if k == 0 else 'else if'} constexpr (N == {n}) {{")
            out.append(block(n).rstrip("\n"))
            out.append("  }")
        out += ['  else static_assert(N < 0, "no run of this length: add it to gen_dpp_runs.py");', "  return p;", "}"]
    Path(__file__).with_name("dpp_runs.inc").write_text("\n".join(out) + "\n")


if __name__ == "__main__":
    main()
