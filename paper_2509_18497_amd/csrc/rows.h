// Host launchers of the FP32 row products (rows.hip): the bounce, its
// adjoint and the sampled products behind dL/dF and dL/drho, for one scene
// or for the scenes of a batch.
#pragma once

#include <vector>

#include "trace_api.h"

namespace gsrad {

// One scene of a launch: its rows of F, the first column index of its block,
// where its [n][C] block of values starts, and its stored entries.
struct RowScene {
    int64_t row0 = 0, n = 0;
    int64_t vbase = 0;
    int32_t C = 0;
    int64_t nnz = 0;
};

// The scenes of a batch, grouped by the kernel that takes them, and where the
// groups' tables lie in one block of device memory.
struct RowTable {
    // scenes of one launch: RowScene[count] and their first workgroups,
    // int64_t[count], at byte offsets of the block
    struct Part {
        int g = 0, lanes = 0, cp = 1, per = 0, chunks = 1;
        int count = 0;
        size_t tab = 0, first = 0;
        int64_t blocks = 0;
    };
    const char *base = nullptr;      // the block; every scene, in order, at its start
    int scenes = 0;
    int64_t vals = 0;
    bool whole = false;              // scenes that 16 lanes per row may suit hold most of the work
    std::vector<Part> rows[3];       // row products with 16, 32 and 64 lanes per row
    std::vector<Part> sampled;       // sampled products of the smaller scenes
    std::vector<RowScene> alone;     // the others, one by one
};
// t of the scenes, and the block's contents, at most rows_table_bytes
void rows_table(const std::vector<RowScene> &scenes, RowTable *t, std::vector<char> *image);
size_t rows_table_bytes(size_t scenes);

// Bout = E + rho * (F Bin)
gsrad_status rows_bounce(const Csr &F, const RowScene &s, const float *Bin, const float *E, const float *rho,
                         float *Bout, hipStream_t st);
// lam = F^T p with p = rho * lam_in, given FT = transpose(F); gE += lam;
// lam and p_out = rho * lam are written where not NULL
gsrad_status rows_adjoint(const Csr &FT, const RowScene &s, const float *p, const float *rho, float *lam,
                          float *p_out, float *gE, hipStream_t st);
// the same over a batch's scenes, lanes per row forced to 16, 32 or 64
gsrad_status rows_bounce_batch(const Csr &F, const RowTable &t, int lanes, const float *Bin, const float *E,
                               const float *rho, float *Bout, hipStream_t st);
gsrad_status rows_adjoint_batch(const Csr &FT, const RowTable &t, int lanes, const float *p, const float *rho,
                                float *lam, float *p_out, float *gE, hipStream_t st);
// The adjoint's start for a whole F or a batch: lam = gE = grad_B (grad_B may be
// gE) and p = rho * grad_B
gsrad_status rows_seed(const RowScene &s, const float *grad_B, const float *rho, float *lam, float *gE, float *p,
                       hipStream_t st);
gsrad_status rows_seed_batch(const RowTable &t, const float *grad_B, const float *rho, float *lam, float *gE, float *p,
                             hipStream_t st);
// grad_F[e] and grad_rho of one scene's rows, or a batch's, from the forward
// tape B^(k) and the adjoint tape lambda^(k+1), slot k at k * stride
gsrad_status rows_sddmm(const Csr &F, const RowScene &s, int nb, int64_t stride, const float *Btape,
                        const float *Ltape, const float *rho, float *grad_F, float *grad_rho, hipStream_t st);
gsrad_status rows_sddmm_batch(const Csr &F, const RowTable &t, int nb, const float *Btape, const float *Ltape,
                              const float *rho, float *grad_F, float *grad_rho, hipStream_t st);

}  // namespace gsrad
