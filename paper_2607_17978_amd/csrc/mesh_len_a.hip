// Mesh passes of the axis lengths of group a (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(60) X(120) X(192) X(512)
QEQ_LEN_GROUP(mesh_len_a, LENGTHS)
