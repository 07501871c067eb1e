// Once-refined meshes with hanging nodes: argument block and launchers
// (kernels in amr.hip, tables built on the host by vpp_amr_create).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "blas.h"
#include "common.h"

namespace vpp {

struct AmrArgs {
    MeshArgs mc;                  // coarse lattice (cell size h)
    MeshArgs mf;                  // fine lattice over the whole box (h / 2)
    int64_t nc;                   // coarse lattice entries; the fine lattice follows
    int64_t n;                    // vector length (coarse + fine lattice)
    const int* cells;             // active cells: coarse index c >= 0, or -(1 + fine index)
    int ncells;
    const int* fkind;             // per fine node: -1 free, -2 unused, else its constraint list
    const int* cptr;              // constraint lists: terms cptr[i] .. cptr[i+1]
    const int* ccol;              // coarse vector entry of each term
    const double* cw;             // its weight
    const unsigned char* ident;   // per entry: 1 = identity row (not a free unknown, or Dirichlet)
    // The packed vector ext: the nfree free unknowns (entry fent[i] of the full
    // vector; pidx is the inverse, -1 on identity rows), one entry that stands
    // for all identity rows in the solver, the ncon constrained nodes (in the
    // order of the constraint lists), a zero.
    int nfree, ncon;
    const int* fent;
    const int* pidx;
    const int* cpk;               // packed index of each constraint term, -1 for an identity row
    double* ext;
    double* invd;                 // packed inverse diagonal (nfree + 1 entries)
    // Cells kernel: thread t of workgroup b (amr_cells_per_block cells each) has
    // its x-plane's packed indices, coefficient factors and result slots at
    // (b (k+1)^2 + q) 256 + t.
    const int* cidx;
    double* coef;
    double* scratch;              // the slots (and the diagonal's, below)
    // the slots of free unknown i: fidx[fptr[i] .. fptr[i+1]); of constrained
    // node m: sidx[sptr[m] ..]; the nsrc unknowns src[k] that constrained nodes
    // draw on (flagged in issrc), and those nodes with weights: tcon, tw[tptr[k] ..]
    const int* fptr;
    const unsigned* fidx;
    const int* sptr;
    const unsigned* sidx;
    int nsrc;
    const int* src;
    const unsigned char* issrc;
    const int* tptr;
    const int* tcon;
    const double* tw;
    double* csum;                 // per constrained node: the sum of its slots
    // The diagonal in two launches: cell e's free nodes at scratch[q * ncells + e]
    // and, for every coarse node a fine cell reaches through constraints (in the
    // order the cell meets them), e^T K_e e at scratch[nfree_slots + soff[e] + i];
    // entry g of diag sums scratch[didx[j]] for j in [dptr[g], dptr[g+1]).
    const int* soff;
    const int* dptr;
    const int* didx;
    int64_t nfree_slots;
};

// CG workspace on the packed vector (nfree + 1 entries each).
struct AmrCg {
    CgState* st;
    double* red;      // 2 nred partials
    int nred;         // amr_red_blocks
    double* dot;      // amr_dot_partials entries
    double* idpart;   // nred: partials of the identity rows' residual
    double* rho;      // its norm
    double* x;
    double* r;
};

int amr_cells_per_block(int k);
int amr_dot_partials(int k, const AmrArgs& a);
int amr_red_blocks(const AmrArgs& a);
// The stored coefficient for a nodal phi on both lattices.
hipError_t launch_amr_coef(int k, const AmrArgs& a, const double* phi, hipStream_t s);
// y = A x; every entry of y is written.
hipError_t launch_amr_apply(int k, const AmrArgs& a, const double* x, double* y, hipStream_t s);
// diag(A) with 1 on identity rows, its FP64 / FP32 inverses and the packed one.
hipError_t launch_amr_diag(int k, const AmrArgs& a, const double* phi, double* diag, double* inv64, float* inv32,
                           hipStream_t s);
// CG: initial residual and direction from b and x (rr_last, rz[0] in w.st); one
// iteration of parity par; the solution back into the full x.
hipError_t launch_amr_cg_init(int k, const AmrArgs& a, const AmrCg& w, const double* b, const double* x, hipStream_t s);
hipError_t launch_amr_cg_step(int k, const AmrArgs& a, const AmrCg& w, int par, hipStream_t s);
hipError_t launch_amr_unpack(const AmrArgs& a, const AmrCg& w, const double* b, double* x, hipStream_t s);

}  // namespace vpp
