"""Coefficients of the FP64 sine polynomial of dev_math.h.

sin(2 pi b) on |b| <= 1/4 as b p(b^2) with p of degree 8: p interpolates
sin(2 pi sqrt(z)) / sqrt(z) at the 9 Chebyshev nodes of z in [0, 1/16], in 60
digits.  Prints the coefficients rounded to FP64 and the largest error of
b p(b^2) with those, evaluated exactly."""
import mpmath as mp

mp.mp.dps = 60
TERMS, END = 9, mp.mpf(1) / 4


def main():
    top = END * END
    nodes = [top / 2 * (1 + mp.cos(mp.pi * (2 * k + 1) / (2 * TERMS))) for k in range(TERMS)]
    A, y = mp.matrix(TERMS, TERMS), mp.matrix(TERMS, 1)
    for i, z in enumerate(nodes):
        for j in range(TERMS):
            A[i, j] = z ** j
        y[i] = mp.sin(2 * mp.pi * mp.sqrt(z)) / mp.sqrt(z)
    c = [mp.mpf(float(v)) for v in mp.lu_solve(A, y)]
    for k, v in enumerate(c):
        print(f"    {float(v).hex()},  // b^{2 * k + 1}")
    err = max(abs(sum(v * b ** (2 * k + 1) for k, v in enumerate(c)) - mp.sin(2 * mp.pi * b))
              for b in (END * j / 4000 for j in range(1, 4001)))
    print("// largest error", mp.nstr(err, 3))


if __name__ == "__main__":
    main()
