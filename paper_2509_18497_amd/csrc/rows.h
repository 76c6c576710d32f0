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

// The scenes of a batch: on the device those with more than four
// coefficients, tab[count], and for 16, 32 and 64 lanes per row the first
// workgroup of each (first[.][count], blocks[.] in all); the others in few.
struct RowTable {
    const RowScene *all = nullptr;   // on the device: every scene, in order
    int scenes = 0;
    int64_t vals = 0;
    const RowScene *tab = nullptr;
    int count = 0;
    const int64_t *first[3] = {nullptr, nullptr, nullptr};
    int64_t blocks[3] = {0, 0, 0};
    std::vector<RowScene> few;
    bool whole = false;   // scenes of rows_whole hold most of the work
};
// whether a scene of C columns goes to few, and the workgroups it takes
// with `lanes` lanes per row
bool rows_few(int C);
// whether less than 64 lanes per row may be the faster ones for the scene
bool rows_whole(const RowScene &s);
int64_t rows_blocks(int64_t n, int C, int lanes);

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
// grad_F[e] and grad_rho of one scene's rows from the forward tape B^(k) and
// the adjoint tape lambda^(k+1), slot k at k * stride
gsrad_status rows_sddmm(const Csr &F, const RowScene &s, int nb, int64_t stride, const float *Btape,
                        const float *Ltape, const float *rho, float *grad_F, float *grad_rho, hipStream_t st);

}  // namespace gsrad
