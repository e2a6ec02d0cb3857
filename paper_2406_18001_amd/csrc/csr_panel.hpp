// Dense-panel CSR product (csr_panel.hip), used by the CSR dispatch.
#pragma once

#include "common.hpp"

namespace kdcd {

// Chunks of lpr sampled rows against a panel of cap rows (lpr 0: no panel).
// sure: no chunk can have more than cap distinct columns; otherwise every
// chunk's product is followed by a kernel that needs no panel, gated on the
// build's overflow flag.  fits: chunks of average rows have not.
struct CsrPanelPlan {
    int lpr;
    uint32_t cap;
    bool sure;
    bool fits;
};
bool csr_long_rows(const kdcd_matrix *A);                   // rows long enough for this path
CsrPanelPlan csr_panel_plan(const KBlockArgs &a);
int64_t csr_panel_groups(const kdcd_matrix *A);             // row groups of the product
int32_t csr_panel_fallback_groups(const kdcd_matrix *A);    // of the gated broadcast launch
size_t csr_dense_panel_min_bytes(int64_t n);
size_t csr_dense_panel_full_bytes(const kdcd_matrix *A);
hipError_t launch_csr_dense_panel_init(const kdcd_matrix *A, void *panel, hipStream_t st);
const int32_t *csr_panel_gate(const void *panel);
hipError_t launch_csr_panel_chunk(const KBlockArgs &a, const CsrPanelPlan &p, int32_t j0, int32_t nj,
                                  bool timed, hipStream_t st);

}  // namespace kdcd
