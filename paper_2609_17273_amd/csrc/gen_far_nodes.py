"""Writes far_nodes.h: Chebyshev nodes and the node-to-coefficient matrices of
the tile expansions: 12 and 20 nodes (FP32 and FP64 forms), 6 and 12 for the
tiles that window ends cut.

    python gen_far_nodes.py > far_nodes.h
"""
import math


def main():
    print("// Generated by gen_far_nodes.py: for P Chebyshev nodes x_q = cos((q + 1/2) pi / P)")
    print("// the nodes, and the matrix D[q][m] with c_m = sum_q D[q][m] f(x_q), the")
    print("// coefficients of the interpolant sum_m c_m T_m(x).")
    print("#pragma once")
    for p in (6, 12, 20):
        x = [math.cos((q + 0.5) * math.pi / p) for q in range(p)]
        print(f"#define XS_FAR_X{p} {{" + ", ".join(f"{v:.17g}" for v in x) + "}")
        rows = []
        for q in range(p):
            for m in range(p):
                # the angle reduced exactly: m (2q + 1) modulo 4p
                a = (m * (2 * q + 1)) % (4 * p)
                rows.append(math.cos(a * math.pi / (2 * p)) * (1.0 if m == 0 else 2.0) / p)
        print(f"#define XS_FAR_D{p} {{" + ", ".join(f"{v:.17g}" for v in rows) + "}")


if __name__ == "__main__":
    main()
