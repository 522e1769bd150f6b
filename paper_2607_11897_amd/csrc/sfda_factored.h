// The factored chunk evaluation: what a 16-token block does to the state depends on the
// block's q, k, alpha, theta and beta only through a few small operands.  With S the state
// entering the block (in the frame of its 64-token step, below), the block relations of
// sfda_chunk_bf16.hip
//   Delta = N D_beta (conj(V) - (conj(K) G) S),   N = (I + D_beta L)^{-1}
//   O^*   = (conj(Q) G) S + A Delta,   S_out = |D| S + (K Q)^T Delta
// read, with T = N D_beta (Thm 4.2's D_beta M), W = T (conj(K) G) and Z = conj(Q) G - A W,
//   Delta = X conj(V) - W S,   O^* = Y conj(V) + Z S,   S_out = |D| S + (K Q)^T Delta,
// with X = T and Y = A T.  The write-decoupled variant (erase rows k with eta, write rows r with
// beta; L_r, A_r its k-r and q-r Gram blocks, T = N D_eta) has the same form with
// X = -T L_r D_beta, Y = A_r D_beta + A X and one more term, (R Q)^T D_beta conj(V), in S_out.
//
// So the work splits in two: a preparing kernel forms every block's operands at once (one
// workgroup per head and 64-token step, one wave per block), and a scan over the blocks that
// only holds the products with the state.  Where the state-dependent chain of a chunk used to
// wait for the chunk's loads, Gram products and inverse, it now waits for two products.
//
// Operand record of a 16-token block (in the caller's workspace, per head and step): left
// operands of the matrix cores as the scans' lanes read them.  A fragment covers 16 rows x 16
// complex K indices: lane (c, g) = (lane % 16, lane / 16) holds row c, K indices 4g .. 4g + 3;
// one 16-byte word per lane as bf16 pairs (1 KiB), or two 16-byte halves per lane as fp32
// (half 0 of every lane, then half 1: 2 KiB).  Channel blocks kb = 0 .. nkb - 1, nkb =
// ceil(m / 16):
//   -W  [nkb]  rows tokens,   K channels of kb         Z  [nkb]  the same
//   K Q [nkb]  rows channels of kb, K tokens            (R Q) D_beta [nkb]  (decoupled)
//   X, Y       rows tokens, K tokens
//   |D| [64] fp32; e^{i phi} of the step's whole phase [64] complex fp32 (in every block; the
//   scans read block 0's)
// Phases are relative to the step's first token; the scans rotate the state by the step's
// phase after its last block.  Decay magnitudes are relative to the block, as in the bf16
// kernel, and a block whose decay falls below 2^-126 has NaN operands.
#pragma once

#include "sfda_device.h"
#include "sfda_launch.h"

namespace sfda {
namespace fac {

constexpr int CP = 64;               // tokens per step (one workgroup of the preparing kernel)
constexpr int NB = CP / 16;          // blocks per step

// what the records serve: the forward, the write-decoupled forward, the backward's scans
enum Kind { FWD = 0, DEC = 1, BWD = 2 };

// bytes of one block's record and of its parts
struct RecLayout {
    int nkb, frag, z, kq, rq, x, y, dm, rot, block;
    __host__ __device__ RecLayout(int m, bool bf16, bool dec) {
        nkb = (m + 15) / 16;
        frag = bf16 ? 1024 : 2048;
        z = nkb * frag;
        kq = 2 * z;
        rq = 3 * z;
        x = (dec ? 4 : 3) * z;
        y = x + frag;
        dm = y + frag;
        rot = dm + 256;
        block = rot + 512;
    }
};

// The backward's records.  The frame is the block's own: phases relative to the block's first
// token, and K Q turned to its end, so that S_out = g S + (K Q)^T Delta with g = |D| e^{i phi} of
// the block (complex), and the adjoint of the block (G = dL/dS_out, G_R = conj(dL/do)) is
//   X' = conj(K Q) G,   dL/dS = conj(g) G - W^* X' + Z^* G_R,
//   G_F = N^* (X' + A^* G_R)     (the adjoint of the solve's right-hand side, before D_beta)
// Fragments, in the order of the forward's record: -W [kb] and T (rows tokens), K Q [kb] (rows
// channels) for the states; conj(K Q) [kb] (rows tokens), -W^* [kb] and Z^* [kb] (rows channels),
// N^* and (A N)^* (rows tokens) for the adjoint; g [64] complex fp32.
struct BwdLayout {
    int nkb, frag, kq, kr, ws, zs, x, ns, an, gc, block;
    __host__ __device__ BwdLayout(int m, bool bf16) {
        nkb = (m + 15) / 16;
        frag = bf16 ? 1024 : 2048;
        kq = nkb * frag;
        kr = 2 * kq;
        ws = 3 * kq;
        zs = 4 * kq;
        x = 5 * kq;
        ns = x + frag;
        an = ns + frag;
        gc = an + frag;
        block = gc + 512;
    }
};

// What the backward's scans leave for the gradient kernel, per head:
//   states: S entering and dL/dS leaving every grad_blocks() blocks, fp32.  bf16 operands: as
//     right operands over the value columns, [channel block][column block of 16][lane (c, g)][4]
//     complex, channel c, columns 4g .. 4g + 3 (the scan turns them through LDS); fp32: [channel][column]
//     (its scan writes 8 columns of a channel at a time: half lines, quarter lines in the other order);
//   rows: Delta and G_F of every block, fp32.  bf16 operands: in the accumulator's order
//     [column block][half][lane (c, g)][2] complex, column c, tokens 4g + 2 half + {0, 1} (whole lines
//     by an instruction); fp32: [token][column].
// The gradient kernel walks from a run's ends to its blocks, three matrix products per block.  In
// fp32 (32 cycles an instruction, and the SIMD issues nothing beside it) that costs more than
// recording every block.  bf16, B8 H16 T4096 m n 64 (with rows of 16 bits): runs of 1, 2, 4 blocks:
// scans 1150, 795, 615 us (what they write), gradients 720, 670, 1060-1570 (four blocks' sums do not
// fit the registers).
__host__ __device__ constexpr int grad_blocks(bool bf16) { return bf16 ? 2 : 1; }
struct GradLayout {
    int nkb, ncb, recs;                  // recs: state records per head
    int state, rows;                     // bytes of a state record, of a block's rows
    long blocks;                         // blocks per head (whole 64-token steps)
    __host__ __device__ GradLayout(int T, int m, int n, bool bf16) {
        nkb = (m + 15) / 16;
        ncb = (n + 15) / 16;
        blocks = (static_cast<long>(T) + CP - 1) / CP * NB;
        recs = static_cast<int>(blocks / grad_blocks(bf16));
        state = nkb * ncb * 2048;
        rows = ncb * 2048;
    }
    __host__ __device__ size_t bytes(long heads) const {
        return static_cast<size_t>(heads) * 2 * (static_cast<size_t>(recs) * state + static_cast<size_t>(blocks) * rows);
    }
};

}  // namespace fac
}  // namespace sfda
