"""The host's rules for the position sweeps' kernels (make_pos_args,
line_tiles_supported, pair_mode, launch_position), restated for tests that have
to know which of them a grid reaches."""


def position_route(n, nu, axis, prec_scaled, max_shift, forward=True):
    """(kernel, lines per thread) of a position sweep: 'tiles', 'pair',
    'gathered' or 'walk'.  max_shift: largest |shift| in cells; forward: the
    upper half of the velocity cells moves up."""
    Nu = nu[0] * nu[1] * nu[2]
    O, I = 1, Nu
    for a in range(axis):
        O *= n[a]
    for a in range(axis + 1, 3):
        I *= n[a]
    M, nuz = n[axis], nu[2]
    pst = (nu[1] * nuz, nuz, 1)[axis]
    V = 1 if axis == 2 else (4 if nuz % 4 == 0 else 2 if nuz % 2 == 0 else 1)
    if O * I < 1024 * 64 * V:                # less than a wave for each SIMD
        V = 1
    if nuz in (16, 32, 64) and M in (16, 32, 64) and I % 64 == 0:
        if axis == 2 and (M != 64 or max_shift >= 1):
            return "tiles", V
        if pst == nuz and axis < 2 and (nuz == 16 or (nuz == 32 and M != 64 and prec_scaled
                                                    and max_shift >= 1)):
            return "tiles", V
    if axis == 2 and prec_scaled and M == 64 and nuz in (16, 32, 64) and (I // 2) % 64 == 0 \
            and max_shift < 1 and forward:
        return "pair", V
    if axis == 1 and V == 4 and pst % 256 and 256 % nuz == 0 and (I // 4) % 256 == 0 and nu[1] % 4 == 0:
        R = 256 // nuz
        if R > 1 and nu[0] % R == 0 and O * (I // Nu) * (nu[0] // R) % 8 == 0 \
                and (not prec_scaled or nuz >= 64):
            return "gathered", V
    return "walk", V
