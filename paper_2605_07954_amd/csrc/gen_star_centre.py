"""Writes star_centre.h and star_rows.h.  star_centre.h: the centre-row taps of a star footprint as one inline-asm block per
(radius, columns per lane), with the side columns read from the neighbouring lanes by DPP operand
shifts of the FMAs themselves instead of separate lane moves.

star_rows.h: the same taps on several rows at once (register tiles), so that the wait states at the
block's head are paid once.

    python paper_2605_07954_amd/csrc/gen_star_centre.py   # rewrites both beside it
"""
import os

HERE = os.path.dirname(os.path.abspath(__file__))
DPP = "row_mask:0xf bank_mask:0xf bound_ctrl:1"


def block(R, V):
    # operands: %0..%V-1 accumulators (read-write), %V..%2V-1 the lane's own centre-row columns,
    # %2V..%2V+2R-1 the weights of dx = -R..-1, 1..R
    lines = ["s_nop 4"]  # wait states for an earlier EXEC or VGPR write that a DPP operand reads
    dxs = [d for d in range(-R, R + 1) if d != 0]
    for wi, dx in enumerate(dxs):
        w = 2 * V + wi
        for c in range(V):
            k = c + dx
            if k < 0:
                lines.append(f"v_fmac_f32_dpp %{c}, %{V + k + V}, %{w} wave_shr:1 {DPP}")
            elif k >= V:
                lines.append(f"v_fmac_f32_dpp %{c}, %{V + k - V}, %{w} wave_shl:1 {DPP}")
            else:
                lines.append(f"v_fmac_f32_e32 %{c}, %{V + k}, %{w}")
    return "\\n\"\n        \"".join(lines)


def rows_block(R, V, N):
    # operands: %0..%NV-1 accumulators (row-major), %NV..%2NV-1 the rows' own columns, then the weights of
    # dx = -R..-1, 1..R
    lines = ["s_nop 4"]
    for wi, dx in enumerate(d for d in range(-R, R + 1) if d != 0):
        w = 2 * N * V + wi
        for n in range(N):
            for c in range(V):
                k, x = c + dx, N * V + n * V
                if k < 0:
                    lines.append(f"v_fmac_f32_dpp %{n * V + c}, %{x + k + V}, %{w} wave_shr:1 {DPP}")
                elif k >= V:
                    lines.append(f"v_fmac_f32_dpp %{n * V + c}, %{x + k - V}, %{w} wave_shl:1 {DPP}")
                else:
                    lines.append(f"v_fmac_f32_e32 %{n * V + c}, %{x + k}, %{w}")
    return "\\n\"\n        \"".join(lines)


def write_rows():
    out = ['// Generated by gen_star_centre.py; do not edit.  The centre-row taps of a star footprint on N rows',
           '// of V columns per lane at once (R <= V): o[n][c] += w[dx] * x[n][c + dx] for dx = -R..-1, then 1..R,',
           '// in that order for every cell; columns beyond the lane are read from the neighbouring lanes by DPP',
           '// operands, lanes at the wave\'s ends read 0.', '#pragma once', '', 'namespace st {', 'namespace block {', '',
           'template <int R, int V, int N>', 'struct StarRows {', '    static constexpr bool exists = false;', '};', '']
    for R, V, N in ((1, 1, 8), (1, 1, 4), (1, 2, 4), (2, 2, 4), (1, 4, 2), (2, 4, 2), (3, 4, 2), (4, 4, 2)):
        outs = ", ".join(f'"+v"(o[{n}][{c}])' for n in range(N) for c in range(V))
        ins = ", ".join([f'"v"(x[{n}][{c}])' for n in range(N) for c in range(V)] + [f'"v"(w[{i}])' for i in range(2 * R)])
        out += ['template <>', f'struct StarRows<{R}, {V}, {N}> {{', '    static constexpr bool exists = true;',
                f'    __device__ __forceinline__ static void apply(float (*o)[{V}], const float (*x)[{V}], const float* w) {{',
                f'        asm("{rows_block(R, V, N)}"', f'            : {outs}', f'            : {ins});', '    }', '};', '']
    out += ['}  // namespace block', '}  // namespace st', '']
    with open(os.path.join(HERE, "star_rows.h"), "w") as f:
        f.write("\n".join(out))


def main():
    write_rows()
    out = ['// Generated by gen_star_centre.py; do not edit.  The centre-row taps of a star footprint,',
           '// dx = -R..-1 then 1..R, each applied to the lane\'s V columns: o[c] += w[dx] * x[c + dx], where',
           '// x[k] for k < 0 is column k + V of the previous lane (wave_shr:1) and for k >= V column k - V of',
           '// the next lane (wave_shl:1); lanes at the wave\'s ends read 0 (bound_ctrl), which only feeds',
           '// outputs that are never stored.  One FMA per tap and column in the canonical order.',
           '#pragma once', '', 'namespace st {', 'namespace march {', '',
           'template <int R, int V>', 'struct StarCentre;', '']
    for V in (4, 8):
        for R in range(1, 5):
            outs = ", ".join(f'"+v"(o[{c}])' for c in range(V))
            ins = ", ".join([f'"v"(x[{c}])' for c in range(V)] + [f'"v"(w[{i}])' for i in range(2 * R)])
            out += ['template <>', f'struct StarCentre<{R}, {V}> {{',
                    f'    __device__ __forceinline__ static void apply(float (&o)[{V}], const float* x, const float* w) {{',
                    f'        asm volatile("{block(R, V)}"', f'                     : {outs}', f'                     : {ins});',
                    '    }', '};', '']
    out += ['}  // namespace march', '}  // namespace st', '']
    with open(os.path.join(HERE, "star_centre.h"), "w") as f:
        f.write("\n".join(out))


if __name__ == "__main__":
    main()
