"""Times of the products and of attention in every form the library has for them, on the GPU at hand.

`python -m tests.product_times > tests/golden/product_times.txt` takes the table that test_product_choice.py holds the library's choices against
(a few minutes).  A line: kind, epilogue, rows, columns, contraction, columns of a second product, rows per slice, then form:us; for attention head
dim, heads, rows per slice, tokens per slice, slices, order of summation, then queries per wave:us.  Every product is timed among
other kernels and with cold weights (epd_op_gemm_bf16_us): behind a norm that writes its operand, with the next of as many weight matrices as a
GiB holds.  Of a pair, form 0 is the two products in a launch each, each as the library picks it.
"""
import ctypes

import torch

from paper_2501_05460_amd import binding as B

# encoder width, MLP width, epilogue of FC1, (rows per slice, slices) of a call
ENCODERS = [
    (1024, 4096, 1, [(1024, n) for n in (1, 2, 3, 4, 5, 6, 7, 8, 10, 13, 16, 20, 26, 39, 52, 78, 104)] + [(1032, n) for n in (1, 3, 5, 8, 16, 32)]
     + [(576, 3), (576, 9), (264, 6), (256, 3), (256, 7), (256, 22), (256, 40)]),
    (1152, 4304, 2, [(1024, n) for n in (1, 2, 3, 4, 5, 6, 8, 10, 14, 20, 26, 40, 64)] + [(736, n) for n in (1, 4, 8, 23, 64)]
     + [(448, 3), (448, 20), (256, 6)]),
    (3200, 12800, 1, [(1024, n) for n in (1, 2, 4, 8, 12, 20, 32, 40)] + [(576, 2), (576, 4), (256, 3)]),
]
# projectors: rows per slice, input width, inner and output width, slices
PROJECTORS = [(256, 4096, 4096, (1, 3, 5, 8, 13, 26, 52, 104)), (1024, 1152, 3584, (1, 2, 5, 10, 20, 64)), (256, 12800, 5120, (1, 4, 6, 12, 32))]
# head dim, heads, (rows per slice, tokens of them, slices)
ATTENTION = [
    (64, 16, [(1024, 1024, n) for n in (1, 2, 3, 4, 5, 6, 8)] + [(1088, 1025, n) for n in (1, 2, 3, 4, 5)] + [(576, 576, n) for n in (1, 3, 5, 6, 7, 9)]
     + [(256, 256, n) for n in (4, 12, 20)] + [(64, 64, 52), (192, 192, 17), (320, 320, 12), (448, 448, 9)]),
    (72, 16, [(1024, 1024, n) for n in (1, 2, 3, 4, 5, 8)] + [(768, 729, n) for n in (1, 3, 4, 6)] + [(576, 576, n) for n in (1, 3, 5, 6, 9)]
     + [(256, 256, n) for n in (4, 12)] + [(192, 192, 20), (448, 448, 9), (576, 576, 7)]),
    (96, 12, [(1024, 1024, n) for n in (1, 2, 3, 4, 5, 8)] + [(1088, 1025, n) for n in (1, 3, 4)] + [(576, 576, n) for n in (3, 7, 8, 9)]
     + [(320, 320, n) for n in (4, 12, 13, 16)] + [(192, 192, 23), (448, 448, 12)]),
    (128, 25, [(1024, 1024, n) for n in (1, 2, 3, 4)] + [(1088, 1025, n) for n in (1, 2, 3)] + [(576, 576, n) for n in (1, 2, 3, 4, 6)]
     + [(768, 768, n) for n in (1, 2, 3)] + [(192, 192, 11), (320, 320, 7), (448, 448, 5)]),
]


def round_up(n, m):
    return (n + m - 1) // m * m


def products():
    """(epilogue, rows, columns, contraction, columns of a second product, rows per slice)"""
    seen = []
    for D, F, act, calls in ENCODERS:
        for tok, n in calls:
            M, Kf = tok * n, round_up(F, 128)
            seen += [(0, M, 2 * D, D, D, tok), (0, M, 2 * D, D, 0, tok), (5, M, D, D, 0, tok), (3, M, D, D, 0, tok), (act, M, F, D, 0, tok),
                     (3, M, D, Kf, 0, tok)]
    for tok, pin, mid, slices in PROJECTORS:
        for n in slices:
            seen += [(1, tok * n, mid, pin, 0, tok), (0, tok * n, mid, mid, 0, tok)]
    return seen


def bf16_forms(epi, M, N, n2):
    few = (M + 127) // 128 * ((N + 127) // 128 + (n2 + 127) // 128) <= 8 * 256
    forms = [11, 13, 14] if few else []
    if n2:
        return forms + [9, 15, 16, 17] + ([12] if N % 192 == 0 and n2 % 192 == 0 else [])
    forms += [1, 10 if epi == 3 else 9, 5]
    if epi in (1, 2, 3):
        forms.append(15)
    if epi == 3:
        forms += ([12] if N % 192 == 0 else []) + ([18] if 0 < N % 256 <= 128 else [])
    return forms


class Pools:
    """Operands, as many elements as the largest product takes: random ones where a product reads them."""

    def __init__(self):
        g = torch.Generator(device="cuda").manual_seed(5)
        self.x = torch.randn(540_000_000, device="cuda", generator=g)
        self.A = torch.zeros(540_000_000, dtype=torch.bfloat16, device="cuda")
        self.W = torch.randn(540_000_000, device="cuda", generator=g).mul_(0.02).bfloat16()
        self.W8 = torch.randint(0x28, 0x40, (1_080_000_000,), device="cuda", dtype=torch.uint8, generator=g)
        self.W8 |= torch.randint(0, 2, (1_080_000_000,), device="cuda", dtype=torch.uint8, generator=g) << 7
        self.SW = torch.full((40_000_000,), 0x75757575, dtype=torch.int32, device="cuda")
        self.SW2 = self.SW.clone()
        self.SA = torch.zeros(5_000_000, dtype=torch.int32, device="cuda")
        self.ones = torch.ones(32768, device="cuda")
        self.bias = torch.randn(32768, device="cuda", generator=g)
        self.C, self.V = (torch.empty(540_000_000, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        self.R = torch.zeros(140_000_000, device="cuda")
        self.Cq = torch.empty(540_000_000, dtype=torch.uint8, device="cuda")
        self.SC = torch.empty(20_000_000, dtype=torch.int32, device="cuda")

    def check(self, M, N, K, n2, epi):
        Mp = round_up(M, 256)
        assert Mp * K <= len(self.x) and Mp * round_up(N, 256) <= (len(self.R) - 256 if epi == 3 else len(self.C)) and M * n2 <= len(self.V)
        assert Mp * K // 128 <= len(self.SA) and Mp * round_up(N, 256) // 128 <= len(self.SC)

    def bf16(self, epi, M, N, K, n2, n_tok, form):
        """us, or None where the form is not one for this product"""
        self.check(M, N, K, n2, epi)
        step = ((round_up(N, 256) if N > 128 else 128) + round_up(n2, 256)) * K
        reps = max(4, min(30, int(6e3 / (2e-9 * M * (N + n2) * K + 8))))
        us = ctypes.c_float()
        s = B.lib().epd_op_gemm_bf16_us(self.x.data_ptr(), self.ones.data_ptr(), self.A.data_ptr(), self.W.data_ptr(), len(self.W) // step, self.bias.data_ptr(),
                                        self.C.data_ptr(), self.V.data_ptr(), self.R.data_ptr(), M, N, n2, K, epi, n_tok, form, reps, ctypes.byref(us),
                                        torch.cuda.current_stream().cuda_stream)
        if s == B.EPD_OK:
            return us.value
        assert form in (5, 18), (B.lib().epd_last_error(None).decode(), epi, M, N, K, n2, form)
        return None

    def mx(self, epi, M, N, K, n2, n_tok, tile):
        self.check(M, N, K, n2, epi)
        Np, n2p = round_up(N, 256), round_up(n2, 256)
        n_w = min(len(self.W8) // ((Np + n2p) * K), len(self.SW) // (K // 128 * max(Np, n2p)))
        reps = max(4, min(30, int(6e3 / (1e-9 * M * (N + n2) * K + 8))))
        us = ctypes.c_float()
        s = B.lib().epd_op_mx_gemm_us(self.x.data_ptr(), self.ones.data_ptr(), self.A.data_ptr(), self.SA.data_ptr(), self.W8.data_ptr(), self.SW.data_ptr(),
                                      self.SW2.data_ptr(), n_w, self.bias.data_ptr(), self.ones.data_ptr(), self.C.data_ptr(), self.V.data_ptr(), self.R.data_ptr(),
                                      self.Cq.data_ptr(), self.SC.data_ptr(), M, N, n2, K, epi, n_tok, tile, reps, ctypes.byref(us),
                                      torch.cuda.current_stream().cuda_stream)
        assert s == B.EPD_OK, (B.lib().epd_last_error(None).decode(), epi, M, N, K, n2, tile)
        return us.value


def line(*fields, times):
    print(*fields, " ".join("%s:%.1f" % (f, t) for f, t in times.items() if t is not None), flush=True)


def attention(hd, heads, n_tok, keys, n, paired):
    g = torch.Generator(device="cuda").manual_seed(7)
    D = hd * heads
    rows = n * n_tok + 64   # a last key block is read past its slice
    qk = torch.randn((rows, 2 * D), device="cuda", generator=g)
    qk[:, :D] *= 1.4427 / hd ** 0.5   # the factor the library folds into its q projection
    qk = qk.bfloat16()
    vt = torch.randn(n * D * n_tok + 64, device="cuda", generator=g).bfloat16()
    o = torch.empty((rows, D), dtype=torch.bfloat16, device="cuda")
    us = ctypes.c_float()
    times = {}
    for queries in (16, 32):
        s = B.lib().epd_op_attention_us(qk.data_ptr(), qk.data_ptr() + 2 * D, vt.data_ptr(), o.data_ptr(), n, n_tok, keys, heads, hd, 2 * D, paired, queries, 100,
                                        ctypes.byref(us), torch.cuda.current_stream().cuda_stream)
        assert s == B.EPD_OK, B.lib().epd_last_error(None).decode()
        times[queries] = us.value
    return times


def main():
    attention(64, 16, 1024, 1024, 40, 0)   # clocks up
    for hd, heads, calls in ATTENTION:
        for n_tok, keys, n in calls:
            for paired in (0, 1):
                line("attention", hd, heads, n_tok, keys, n, paired, times=attention(hd, heads, n_tok, keys, n, paired))
    pools = Pools()
    times = {}
    for case in products():
        epi, M, N, K, n2, n_tok = case
        if case in times:
            continue
        t = {f: pools.bf16(*case, f) for f in bf16_forms(epi, M, N, n2)}
        if n2:
            t[0] = pools.bf16(0, M, N, K, 0, n_tok, 0) + pools.bf16(5, M, n2, K, 0, n_tok, 0)
        times[case] = t
        line("bf16", *case, times=t)
    for case in dict.fromkeys(p for p in products() if not (p[2] == p[3] and p[0] == 0) and (p[2], p[3]) not in [(m, k) for _, k, m, _ in PROJECTORS]):
        epi, M, N, K, n2, n_tok = case
        t = {tile: pools.mx(*case, tile) for tile in ((1, 2, 3) if epi == 3 else (1, 2))}
        if n2:
            t[0] = pools.mx(0, M, N, K, 0, n_tok, 0) + pools.mx(5, M, n2, K, 0, n_tok, 0)
        line("mx", *case, times=t)


if __name__ == "__main__":
    main()
