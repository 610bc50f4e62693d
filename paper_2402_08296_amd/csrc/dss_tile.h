// The FP64 and FP32 DSS forward in launches of one message-passing block each,
// over tiles of 16 nodes (dss_tile.hip): weight blobs and launchers. Host part
// in plain C++.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "device.h"

namespace ddmgnn {

constexpr int VT_TILE = 16;   // nodes of a tile (the N dimension of the matrix instructions)
constexpr int VT_BLOCK = 256; // threads of the setup kernels
constexpr int64_t VT_MAX_FP32 = 60 * 1024;  // most tiles of an FP32 launch in this form (runs_tiled)
constexpr int VT_ROWS = 8;    // edge rows read at a time (the array is padded by as many)

// Values per lane of one block's blob: matrix operands, then per-lane constants.
// The blobs are stored in chunks of 16 bytes per lane ([chunk][lane][16 bytes]).
template <typename T>
struct VtLayout;
template <>
struct VtLayout<double> {
    // Psi's hidden layer (h and c, deg: 3 steps; message sums: 5) and output layer, operands of
    // the 4-row product (16 values each), three per step: 10 places of 64 values;
    // receiver part of the first message layers (units 0-3 of every lane, unit 4)
    static constexpr int HID = 0, OUT = 24, N_QUAD = 33;
    static constexpr int P16 = 10, P4 = 13, CP = 16, CP4 = 20, CH = 21, CO = 24, WN = 27, N_MAIN = 32;
    static_assert((N_QUAD + 1) / 2 * 32 <= P16 * 64, "the 4-row operands fit before the others");
    // sender part
    static constexpr int Q16 = 0, Q4 = 3, N_Q = 6;
    static constexpr int N_OPS = CP, N_QOPS = N_Q;  // operands; the rest are constants of a group
    // decoder
    static constexpr int DH = 0, DO = 3, CDH = 6, CDO = 9, N_DEC = 10;
};
template <>
struct VtLayout<float> {
    // as above, with the second message layers (FO, FI) and the coordinate weights (WX, WY)
    static constexpr int P16 = 0, P4 = 3, FO = 6, FI = 9, HID = 12, OUT = 21;
    static constexpr int CP = 24, CP4 = 28, WX = 29, WY = 34, WN = 39, CCO = 44, CCI = 47, CH = 50, CO = 53,
                         N_MAIN = 56;
    static constexpr int Q16 = 0, Q4 = 3, QX = 6, QY = 11, N_Q = 16;
    static constexpr int N_OPS = CP, N_QOPS = QX;
    static constexpr int DH = 0, DO = 3, CDH = 6, CDO = 9, N_DEC = 12;
};

// A blob of n values per lane on the device, where it is read from LDS: the first n_ops,
// operands, are held per lane; the others are constants of a lane's group and follow as
// four rows (a quarter of the constants' LDS, which limits the wavefronts in flight). Whole KB.
template <typename T>
struct VtBlob {
    static constexpr int PER = 16 / (int)sizeof(T);
    static constexpr int ops(int n_ops) { return (n_ops + PER - 1) / PER * PER * 64; }
    // (padded by 16 bytes: the four rows start on different banks)
    static constexpr int row(int n, int n_ops) { return n > n_ops ? (n - n_ops + 2 * PER - 1) / PER * PER : 0; }
    static constexpr int size(int n, int n_ops) {
        return (ops(n_ops) + 4 * row(n, n_ops) + 64 * PER - 1) / (64 * PER) * (64 * PER);
    }
};
// Device weights: kbar main blobs, kbar sender blobs, one decoder blob, back to back.
template <typename T>
struct VtBlobs {
    static constexpr size_t MAIN = VtBlob<T>::size(VtLayout<T>::N_MAIN, VtLayout<T>::N_OPS),
                            Q = VtBlob<T>::size(VtLayout<T>::N_Q, VtLayout<T>::N_QOPS),
                            DEC = (size_t)VtLayout<T>::N_DEC * 64;
    static size_t size(int kbar) { return (size_t)kbar * (MAIN + Q) + DEC; }
};
// theta: kbar blocks of the width-10 model (Table II layout).
void build_vt_blobs(const float* theta, int kbar, std::vector<double>& b64, std::vector<float>& b32);

// The FP32 main, sender and decoder blobs of one block given by its TRAIN_NWB values
// (training passes positions instead of weights and gathers by them).
void build_vt_maps(const float* one_block, std::vector<float>& main, std::vector<float>& sender,
                   std::vector<float>& dec);

// Tile of a problem: first slot of its sub-mesh, first position of the tile in
// it, first edge row, edge rows (the tile's largest in-degree).
using VtTile = int4;
// Fills the nodes (slot or -1, in-degree) of every tile and the slots' tile lanes (P's
// base arrays from *tab); the edge records (sentinel sender: 16 n_tiles) in one
// precision (the other null).
hipError_t launch_vt_nodes(const DevProb* tab, const VtTile* info, int n_tiles, int2* node, int32_t* pos,
                           hipStream_t s);
hipError_t launch_vt_edges(const DevProb* tab, const VtTile* info, int n_tiles, const int2* node, const int32_t* pos,
                           VtRec<float>* rec32, VtRec<double>* rec64, hipStream_t s);
// Fills n values with v (the sentinel rows and the padding).
hipError_t launch_vt_fill(double* p, int64_t n, double v, hipStream_t s);
hipError_t launch_vt_fill(float* p, int64_t n, float v, hipStream_t s);

// One DSS forward over n_tiles tiles of the sub-meshes in subs: the restriction
// (apply) with the first sender rows, kbar block launches. tiles: (problem,
// tile, first edge row, edge rows). solo: every item is of problem 0.
template <typename T>
hipError_t launch_dss_tiles(const DevProb* tab, const int2* subs, int n_subs, const int4* tiles, int n_tiles,
                            bool solo, int kbar, double alpha, int apply, const T* blobs, hipStream_t s, bool check);

}  // namespace ddmgnn
