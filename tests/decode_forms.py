"""Calls of decode_verify and the kernel that each one reaches (n = 64, noise of 9
terms): checked against the launches on the host and against the oracle on a GPU."""

# m, ry, columns, repetitions, challenge terms, Y over Yhat, kernel
FORMS = [
    # 13 columns and more of up to 8192 positions with one or two repetitions, where
    # the decode role takes four columns a lane; one column or one repetition to
    # the other side, no four columns a lane (m = 4097; 15 columns of 4096)
    (5000, 1, 13, 1, 31, False, "decode_verify_syn<16, 4>"),
    (4096, 2, 16, 2, 31, False, "decode_verify_syn<16, 4>"),
    (5464, 1, 12, 1, 31, False, "decode_verify_dot<16, 16>"),
    (5464, 1, 15, 2, 31, False, "decode_verify_dot<16, 16>"),
    (4096, 2, 16, 3, 31, False, "decode_verify_dot<16, 16>"),
    (4096, 2, 15, 1, 31, False, "decode_verify_dot<16, 16>"),
    (4097, 1, 16, 1, 31, False, "decode_verify_dot<16, 16>"),
    (4100, 2, 16, 1, 31, False, "decode_verify_dot<24, 16>"),
]
