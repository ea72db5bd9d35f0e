// Mesh passes of the axis lengths of group d (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(20) X(40) X(144) X(240) X(432)
QEQ_LEN_GROUP(mesh_len_d, LENGTHS)
