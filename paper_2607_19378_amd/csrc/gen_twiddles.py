"""Write twiddles.inc: fp32 twiddle tables computed in fp64 on the host.

Tables (all values exp(-2 pi i j / n) rounded once to float32):
  kTwCoarse[j] = exp(-2 pi i j / 4096),  j < 4096
  kTwFine[j]   = exp(-2 pi i j / 2^24),  j < 4096
  kCos32/kSin32[j] = cos/sin(2 pi j / 32), j < 32 (radix-<=32 butterfly constants)
  kTwDelta[j]  = exp(-2 pi i j / 32768) - 1,  j < 1024 (weights near 1, to full relative accuracy)
  kCos64/kSin64[j] = cos/sin(2 pi j / 64), j < 16 (shifted radix-16 passes)
  kCos32Lo, kSin32Lo, kCos64Lo, kSin64Lo: what the rounding of those leaves
  kPassTw_<log2 NS>_<log2 R>: for every Stockham pass shape (NS, R) with
    NS * R <= 8192, the twiddles exp(-2 pi i jm r / (NS R)) laid out
    [r - 1][jm] (r in 1..R-1, jm in 0..NS-1), so lanes holding consecutive jm
    read consecutive entries; pass_table<log2 NS, log2 R>() returns it.
Any exp(-2 pi i a / 2^s) with s <= 24 is kTwCoarse[b >> 12] * kTwFine[b & 4095]
with b = a << (24 - s); for s <= 12 it is kTwCoarse[a << (12 - s)] alone.

Usage: python gen_twiddles.py [output path]
"""
import math
import os
import struct
import sys


def f32(x: float) -> float:
    return struct.unpack("<f", struct.pack("<f", x))[0]


def lit(x: float) -> str:
    x = f32(x)
    if x == 0.0:
        return "0.0f" if math.copysign(1.0, x) > 0 else "-0.0f"
    return float.hex(x) + "f"


def table(name: str, n: int, count: int) -> str:
    out = [f"static __device__ const float2 {name}[{count}] = {{"]
    for j in range(count):
        a = 2.0 * math.pi * j / n
        # cos/sin of the reduced angle in fp64, then one rounding to fp32
        out.append(f"  {{{lit(math.cos(a))}, {lit(-math.sin(a))}}},")
    out.append("};")
    return "\n".join(out)


def main():
    path = sys.argv[1] if len(sys.argv) > 1 else os.path.join(os.path.dirname(os.path.abspath(__file__)),
                                                              "twiddles.inc")
    parts = ["// Generated by gen_twiddles.py: fp64 values rounded once to fp32. Do not edit.",
             "#pragma once",
             table("kTwCoarse", 4096, 4096),
             table("kTwFine", 1 << 24, 4096)]
    rows = []
    for j in range(1024):
        a = 2.0 * math.pi * j / 32768
        rows.append(f"  {{{lit(-2.0 * math.sin(a / 2) ** 2)}, {lit(-math.sin(a))}}},")
    parts.append("static __device__ const float2 kTwDelta[1024] = {\n" + "\n".join(rows) + "\n};")
    # Stockham pass tables: one array per pass shape, so that a translation
    # unit holds only the shapes its kernels use
    parts.append("template <int LNS, int LR>\n__device__ __forceinline__ const float2* pass_table();")
    for lns in range(1, 13):
        for lr in range(1, 5):
            NS, R = 1 << lns, 1 << lr
            if NS * R > 8192:
                continue
            n = NS * R
            entries = []
            for r in range(1, R):
                for jm in range(NS):
                    a = 2.0 * math.pi * ((jm * r) % n) / n
                    entries.append((math.cos(a), -math.sin(a)))
            body = ",\n".join(f"  {{{lit(c)}, {lit(sn)}}}" for c, sn in entries)
            name = f"kPassTw_{lns}_{lr}"
            parts.append(f"static __device__ const float2 {name}[{len(entries)}] = {{\n{body}\n}};")
            parts.append(f"template <>\n__device__ __forceinline__ const float2* pass_table<{lns}, {lr}>() "
                         f"{{ return {name}; }}")
    cos32 = ", ".join(lit(math.cos(2 * math.pi * j / 32)) for j in range(32))
    sin32 = ", ".join(lit(math.sin(2 * math.pi * j / 32)) for j in range(32))
    parts.append(f"constexpr float kCos32[32] = {{{cos32}}};")
    parts.append(f"constexpr float kSin32[32] = {{{sin32}}};")
    cos64 = ", ".join(lit(math.cos(2 * math.pi * j / 64)) for j in range(16))
    sin64 = ", ".join(lit(math.sin(2 * math.pi * j / 64)) for j in range(16))
    parts.append(f"constexpr float kCos64[16] = {{{cos64}}};")
    parts.append(f"constexpr float kSin64[16] = {{{sin64}}};")
    for name, fn, n, count in (("kCos32Lo", math.cos, 32, 32), ("kSin32Lo", math.sin, 32, 32),
                               ("kCos64Lo", math.cos, 64, 16), ("kSin64Lo", math.sin, 64, 16)):
        exact = [fn(2 * math.pi * j / n) for j in range(count)]
        parts.append(f"constexpr float {name}[{count}] = {{{', '.join(lit(x - f32(x)) for x in exact)}}};")
    text = "\n".join(parts) + "\n"
    tmp = path + ".tmp"
    with open(tmp, "w") as f:
        f.write(text)
    os.replace(tmp, path)


if __name__ == "__main__":
    main()
