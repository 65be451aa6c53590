"""Calls of decode_verify and the kernel that each one reaches (n = 64, noise of 9
terms): checked against the launches on the host and against the oracle on a GPU."""

# m, ry, columns, repetitions, challenge terms, Y over Yhat, kernel
FORMS = [
    # the challenge syndromes in the same launch, every tile size of the syndrome and
    # both widths of the decode role: more than 4 repetitions, more than 64 terms,
    # Y over Yhat; four columns a lane (only the two smaller tiles are resident then)
    (1000, 4, 2, 5, 31, False, "decode_verify_syn<8, 1>"),
    (1000, 4, 2, 2, 65, False, "decode_verify_syn<8, 1>"),
    (4096, 2, 1, 5, 31, False, "decode_verify_syn<16, 1>"),
    (4096, 2, 2, 3, 65, False, "decode_verify_syn<16, 1>"),
    (2049, 2, 2, 2, 31, True, "decode_verify_syn<16, 1>"),
    (4096, 3, 2, 16, 31, False, "decode_verify_syn<24, 1>"),
    (2731, 3, 3, 2, 31, True, "decode_verify_syn<24, 1>"),
    (4096, 4, 1, 5, 31, False, "decode_verify_syn<32, 1>"),
    (4096, 4, 1, 2, 65, False, "decode_verify_syn<32, 1>"),
    (4096, 4, 2, 2, 31, True, "decode_verify_syn<32, 1>"),
    (15000, 1, 1, 6, 31, False, "decode_verify_syn<32, 1>"),
    (4096, 1, 16, 2, 31, False, "decode_verify_syn<8, 4>"),
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
    # one column a lane: 15 columns of at least 960 rows with one repetition
    (1366, 3, 15, 1, 31, False, "decode_verify_syn<16, 1>"),
    (960, 8, 16, 1, 31, False, "decode_verify_syn<16, 1>"),
    (1366, 3, 14, 1, 31, False, "decode_verify_dot<16, 16>"),
    (959, 8, 16, 1, 31, False, "decode_verify_dot<16, 16>"),
    (1366, 3, 15, 2, 31, False, "decode_verify_dot<16, 16>"),
    # neither: the syndromes before, in a launch of their own
    (4096, 3, 17, 2, 31, False, "decode_verify_fused"),
]
