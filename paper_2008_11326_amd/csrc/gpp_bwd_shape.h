// gpp_bwd_shape.h -- how the adjoint's pairs kernel deals bands out to the
// waves that share a tile (host and device code).
#pragma once

namespace gpp {

// Where part k of `total` items in `parts` equal parts begins.  The product
// is formed in 64 bits: four times a band count passes 2^31 from 2^29 bands.
constexpr int share_begin(int total, int k, int parts) { return (int)((long)total * k / parts); }

// First band of part k of the unoccupied bands [nocc, nb), in whole groups of
// `group` bands (the last one may be ragged); part `parts` begins at nb.
constexpr int share_first_band(int nb, int nocc, int group, int k, int parts)
{
    const int groups = (nb - nocc + group - 1) / group;
    const int at = nocc + share_begin(groups, k, parts) * group;
    return at < nb ? at : nb;
}

}  // namespace gpp
