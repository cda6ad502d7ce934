"""Build step: writes tables.inc, the constant tables compiled into the HIP code object.

* kTw4096   float2[4096]  exp(-2 pi i m / 4096), each component correctly rounded to float32
                          from its double value (FFT twiddles for sizes 512..4096).
* kTwRows<N>  float2[R][N/R]  exp(-2 pi i r j / N) at [r][j], the same values in the order in which
                          the lanes j of a radix-R pass read them (whole lines; kTw4096 itself would
                          be up to 64 lines a load)
* kHann<N>  float[N]      periodic Hann window 0.5 - 0.5 cos(2 pi n / N), rounded once from the
                          float32 cosine
* kCos4096  double[4096]  cos(2 pi m / 4096)  (EQ spectrum on the 4096-point FFT grid)
* kCos2047  double[2047]  cos(2 pi m / 2047)  (EQ FIR design, N = 2047)

Values are emitted as hexadecimal floating literals, so the compiled tables hold exactly the
rounded values computed here.
"""
import math
import os
import struct
import sys


def f32(x: float) -> float:
    return struct.unpack("<f", struct.pack("<f", x))[0]


def hexf(x: float, single: bool) -> str:
    if x == 0.0:
        return "0.0f" if single else "0.0"
    return float.hex(x) + ("f" if single else "")


def main(out_path: str) -> None:
    lines = ["// generated by gen_tables.py -- do not edit", "#pragma once", ""]
    tw, cos4096 = [], []
    for m in range(4096):
        a = -2.0 * math.pi * m / 4096.0
        # exact values at the multiples of pi/4 avoid tiny non-zero residues
        c, s = math.cos(a), math.sin(a)
        if m % 1024 == 0:
            c, s = [(1.0, 0.0), (0.0, -1.0), (-1.0, 0.0), (0.0, 1.0)][m // 1024]
        cos4096.append(c)
        tw.append("{%s, %s}" % (hexf(f32(c), True), hexf(f32(s), True)))
    lines.append("__device__ const float2 kTw4096[4096] = {")
    for i in range(0, 4096, 4):
        lines.append("  " + ", ".join(tw[i:i + 4]) + ",")
    lines.append("};")
    for n, radix in ((64, 8), (128, 8), (256, 16), (512, 8), (1024, 8), (2048, 8), (4096, 16)):
        rows = [tw[r * j * (4096 // n)] for r in range(radix) for j in range(n // radix)]
        lines.append("__device__ const float2 kTwRows%d[%d] = {" % (n, n))
        for i in range(0, n, 4):
            lines.append("  " + ", ".join(rows[i:i + 4]) + ",")
        lines.append("};")
    for n in (512, 1024, 2048):
        win = [hexf(f32(0.5 - 0.5 * f32(cos4096[m * (4096 // n)])), True) for m in range(n)]
        lines.append("__device__ const float kHann%d[%d] = {" % (n, n))
        for i in range(0, n, 8):
            lines.append("  " + ", ".join(win[i:i + 8]) + ",")
        lines.append("};")
    for name, n in (("kCos4096", 4096), ("kCos2047", 2047)):
        vals = []
        for m in range(n):
            c = math.cos(2.0 * math.pi * m / n)
            if n % 4 == 0 and m % (n // 4) == 0:  # exact at the multiples of pi/2
                c = [1.0, 0.0, -1.0, 0.0][m // (n // 4)]
            vals.append(hexf(c, False))
        lines.append("")
        lines.append("__device__ const double %s[%d] = {" % (name, n))
        for i in range(0, n, 4):
            lines.append("  " + ", ".join(vals[i:i + 4]) + ",")
        lines.append("};")
    text = "\n".join(lines) + "\n"
    if os.path.exists(out_path) and open(out_path).read() == text:
        return
    with open(out_path, "w") as f:
        f.write(text)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else
         os.path.join(os.path.dirname(os.path.abspath(__file__)), "tables.inc"))
