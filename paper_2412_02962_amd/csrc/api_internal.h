// Host-side helpers shared by the C ABI translation units.
#pragma once

#include <stdint.h>

#include "../../include/pcpp.h"
#include "kernels.h"

namespace pcpp {

// Eq. 1 geometry of one validated call.
struct Geo {
    int32_t h;      // band height H / n
    int32_t up;     // context rows from the band above
    int32_t dn;     // context rows from the band below
    int32_t nq;     // queries per image: h * W
    int32_t n_kv;   // context keys per image: (up + h + dn) * W
    int32_t C;      // heads * head_dim
    int32_t esize;  // bytes per element
};

int validate_geom(const pcpp_geom_t* g, Geo* out);
int validate_geom_hops(const pcpp_geom_t* g, bool multi_hop, Geo* out);
KvSource make_kv_source(const pcpp_geom_t* g, const Geo& r, const void* k_fresh, const void* v_fresh,
                        const void* k_up, const void* v_up, const void* k_dn, const void* v_dn);
AttnParams make_attn_params(const pcpp_geom_t* g, const Geo& r, const void* q, void* out,
                            const KvSource& kv);
// Argument checks of pcpp_partial_attention (geometry, dtype, head_dim,
// pointers, 16-byte alignment); PCPP_OK or the status to return.
int check_attention(const pcpp_geom_t* g, Geo* r, const void* q, const void* k_fresh, const void* v_fresh,
                    const void* k_up, const void* v_up, const void* k_dn, const void* v_dn, const void* out);

}  // namespace pcpp

// pcpp_conv3x3_export with a limit on the looks that the pieces of a split
// tile take at each other (GemmParams::max_polls; < 0: the library's own).
// Exported for the tests of the pieces that give up waiting; not part of the C
// ABI.
extern "C" __attribute__((visibility("default"))) int pcpp_internal_conv3x3(
    const pcpp_conv_geom_t* g, const void* x, const void* row_up, const void* row_dn, const void* w, const void* bias,
    void* y, void* first_out, void* last_out, void* workspace, size_t ws_bytes, int32_t max_polls, void* stream);
