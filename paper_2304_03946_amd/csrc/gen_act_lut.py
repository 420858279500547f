"""Writes act_lut_data.inc: the GELU residual tables of the bf16 expert-FFN epilogues as constant data.

Both GELU forms are z*F(z) with F(z) + F(-z) = 1, so on the bf16 magnitudes a = 2^-24 .. 8
    GELU(z)  = max(z, 0) + r(|z|),            r(a) = -a F(-a)
    GELU'(z) = [z >= 0] + sign(z) * q(|z|),    q(a) = a F'(a) - F(-a)
Entry i belongs to the magnitude with bf16 bits kLutLo + i (clamped to kLutHi), computed here in double precision and
stored in fp32: first the erf form (F = standard normal CDF), then the tanh form, of each a table of r and one of q.
The layout constants must agree with ffn_bf16_tile.h (a static_assert there checks the entry count).
Run by build.py before the HIP sources are compiled; the output is a build artefact.
"""
import math
import struct
import sys

LUT_LO = 103 << 7          # bf16 bits of 2^-24
LUT_HI = 130 << 7          # bf16 bits of 8.0
LUT_BYTES = 14 * 1024
ENTRIES = LUT_BYTES // 4


def bf16_value(bits: int) -> float:
    return struct.unpack("<f", struct.pack("<I", bits << 16))[0]


def entry(form: int, a: float):
    if form == 0:
        f_neg = 0.5 * math.erfc(a * math.sqrt(0.5))
        d_f = math.exp(-0.5 * a * a) / math.sqrt(2.0 * math.pi)
    else:
        c = math.sqrt(2.0 / math.pi)
        th = math.tanh(c * (a + 0.044715 * a ** 3))
        f_neg = 0.5 * (1.0 - th)
        d_f = 0.5 * (1.0 - th * th) * c * (1.0 + 3.0 * 0.044715 * a * a)
    return -a * f_neg, a * d_f - f_neg


def f32_hex(v: float) -> str:
    # C99 hexadecimal float literal of the value rounded to fp32 (exact, no decimal round trip)
    return float.hex(struct.unpack("<f", struct.pack("<f", v))[0]) + "f"


def main(path: str) -> None:
    with open(path, "w") as out:
        out.write("// generated by gen_act_lut.py -- do not edit\n")
        out.write(f"// {ENTRIES} entries per table\n")
        for form in (0, 1):
            pairs = [entry(form, bf16_value(min(LUT_LO + i, LUT_HI))) for i in range(ENTRIES)]
            out.write("{\n")
            for which in (0, 1):
                out.write("{\n")
                for pair in pairs:
                    out.write(f32_hex(pair[which]) + ",\n")
                out.write("},\n")
            out.write("},\n")


if __name__ == "__main__":
    main(sys.argv[1])
