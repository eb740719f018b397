"""Batches that reach every form the staged gather is built with: (tau, lanes a token, token slots) where token ranges are divided
over the workgroups, and (d_out, tau, tokens, slots allowed, slots taken) where whole chunks are."""

SLOTS = (4, 6, 7, 8, 10, 12, 13, 14, 16)

# (tau, lanes): copy rounds a table 1, 2, 4 of 128-byte and of 64-byte slices
WIDTHS = ((7, 8), (8, 8), (9, 8), (8, 4), (9, 4), (10, 4))
RANGES = tuple((tau, lanes, slots) for tau, lanes in WIDTHS for slots in SLOTS if lanes == 8 or slots >= 6)
TABLES = 8  # four stages and more: both buffers, the prefetch of the third ahead, every step of the multi-probe form's lag


def width(lanes):
    """Seven slices, the last a part: four workgroups to each slice of an eighth of the tokens."""
    return 200 if lanes == 8 else 104


def tokens(lanes, slots):
    """The last chunk of every range short of `slots` full ones."""
    return 8 * 4 * (1024 // lanes) * slots - 77


def has_probes(tau, lanes):
    return lanes == (8 if tau <= 8 else 4)  # the multi-probe form is built for these


CHUNKS = ((224, 7, 32943, 4, 4), (352, 7, 26993, 6, 6), (352, 7, 33643, 8, 7), (224, 7, 66235, 8, 8), (352, 8, 48267, 10, 10),
          (352, 8, 53364, 12, 12), (352, 7, 62046, 14, 13), (352, 7, 66986, 14, 14), (352, 8, 76011, 16, 16),
          (176, 9, 57497, 6, 6), (176, 9, 65841, 8, 7), (176, 9, 79721, 8, 8), (288, 9, 63088, 10, 10), (288, 9, 78034, 12, 12),
          (384, 10, 67109, 13, 13), (384, 10, 72852, 14, 14), (384, 10, 82852, 16, 16))
