// Attention variant: tables and launchers shared by its host side (attn_layer.cpp) and its kernels (kernels_attn.hip).
#pragma once
#include "common.h"

namespace hgnn {

struct AttnPtrs {   // attention vectors (storage type) or their gradients (fp32), per relation
  const void *a_src[kMaxR];
  const void *a_dst[kMaxR];
};
// Merged rows by relation, and tiles that do not cross a relation.
struct RelRows {
  int32_t tile_off[kMaxR + 1];   // tiles before relation r (set by the launcher)
  int32_t row_off[kMaxR + 1];    // merged rows before relation r
  int32_t zdst[kMaxR];           // projected row of the first destination vertex of relation r
  int32_t gdst[kMaxR];           // output row of the same vertex
  uint8_t dst[kMaxR];
  int32_t n;
};
// Destination rows by type, and tiles that do not cross a type.
struct TypeTiles {
  int32_t tile_off[kMaxT + 1], row_off[kMaxT + 1];
  int32_t n;
};
// relations grouped by destination type
struct RelsOfType {
  uint16_t first[kMaxT + 1];
  uint8_t rel[kMaxR];
};
struct SemBwd {
  int32_t n_dw, dw_rows;   // blocks of the dW_s part and the merged rows each of them takes
};

hgnn_status launch_attn_proj(hipStream_t s, int dtype, const TypeTab &tt, const PtrTab &w_type_as_root, int H, const void *x, float *z,
                             double *wsum);
hgnn_status launch_attn_agg(hipStream_t s, int dtype, const LayerDev &L, RelRows rr, const AttnPtrs &ap, int H, int heads,
                            const float *z, float *mout, float *mx, float *ls);
hgnn_status launch_attn_sem(hipStream_t s, int dtype, RelRows rr, int H, const float *mbuf, const void *w_sem, const void *b_sem,
                            const void *q_sem, float *tbuf, double *wsum);
hgnn_status launch_attn_fuse(hipStream_t s, int dtype, const TypeTab &tt, const RelRows &rr, const PtrTab &pt, int H, int relu,
                             const float *mbuf, const double *wsum, float *beta, void *h);
hgnn_status launch_attn_zero(hipStream_t s, float *const *ptrs, const int64_t *counts, int n);
hgnn_status launch_attn_mask_dbeta(hipStream_t s, int dtype, const TypeTab &tt, const RelRows &rr, const GradPtrTab &gt, int H, int relu,
                                   const void *g, const void *h, void *gp, const float *mbuf, float *dbeta);
hgnn_status launch_attn_sem_bwd(hipStream_t s, int dtype, const RelRows &rr, int H, const float *mbuf, const float *tbuf, const void *w_sem,
                                const void *q_sem, const void *gp, const float *beta, const float *dbeta, float *dm, float *dws, float *dq,
                                float *dbs);
hgnn_status launch_attn_agg_bwd(hipStream_t s, int dtype, const LayerDev &L, const TypeTab &tt, RelRows rr, const AttnPtrs &ap,
                                const AttnPtrs &dap, int H, int heads, const float *z, const float *dm, const float *mx, const float *ls,
                                void *edge_ad, float *xsum, float *dsum, void *dz, float *partial);

}  // namespace hgnn
